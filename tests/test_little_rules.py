"""CPU checks of the little solve's host rules (csrc/little_rules.h), built as plain
C++ under the address and undefined-behaviour sanitizers: when the host looks at
the norms.  On residuals that fall by a constant factor no step is run beyond the
one that converged, save up to the first look of a solve that gains more than a
digit a step, and looks are no more than one in four steps and two.  How a product
is split: every tile taken once, a workgroup's four waves on one tile as long as
the tiles do not fill the device and on a tile each beyond (a wave alone in its
workgroup made large products slower than they had been)."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1605_00564_amd", "csrc")
FLAGS = ["-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
         "-fno-omit-frame-pointer"]


def _run(tmp_path, source, lines):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "check")
    r = subprocess.run(["g++", *FLAGS, "-I", CSRC, os.path.join(ROOT, "tests", source), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], input="".join(lines), capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    return [[int(v) for v in line.split()] for line in r.stdout.splitlines()]


def test_looks(tmp_path):
    cases = [(tol, rate) for tol in (0.9, 0.5, 0.3, 0.1, 0.03, 1e-2, 1e-3, 1e-4, 1e-6, 1e-10)
             for rate in (0.01, 0.05, 0.2, 0.5, 0.8, 0.95)]
    out = _run(tmp_path, "little_rules_check.cpp", [f"{t} {r}\n" for t, r in cases])
    assert len(out) == len(cases)
    for (tol, rate), (need, steps, looks) in zip(cases, out):
        assert need <= steps <= (need if rate >= 0.1 else max(need, 4)), (tol, rate, need, steps)
        assert looks <= -(-need // 4) + 2, (tol, rate, need, looks)
        if tol >= 0.1:
            assert steps == need, (tol, rate, need, steps)


def test_row_tiles(tmp_path):
    cases = [(r, ns, n) for r in (1, 7, 8, 16, 128, 648, 1296, 2592, 8192) for ns in (1, 12, 16, 17, 20, 40)
             for n in (1, 8, 9, 16, 17, 24, 25, 40)]
    out = _run(tmp_path, "row_tiles_check.cpp", [f"{r} {s} {n}\n" for r, s, n in cases])
    assert len(out) == len(cases)
    for (r, ns, n), (waves, nmt, ng, ok) in zip(cases, out):
        assert ok, (r, ns, n)
        assert waves == (4 if r * nmt * ng <= 2048 else 1), (r, ns, n)
