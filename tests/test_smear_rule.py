"""CPU check of the rule that splits Gaussian smearing over its two kernels
(csrc/smear_rules.h): one launch a step on small lattices, whatever the number of
vectors (two of them took up to 1.8 times as long), groups of four first on large
ones."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1605_00564_amd", "csrc")


def test_groups(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "check")
    r = subprocess.run(["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined",
                        "-fno-sanitize-recover=all", "-I", CSRC,
                        os.path.join(ROOT, "tests", "smear_rule_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    cases = [(V, n) for V in (256, 4096, 32768, 32768 + 256, 65536, 2097152) for n in range(1, 26)]
    r = subprocess.run([exe], input="".join(f"{V} {n}\n" for V, n in cases), capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
    got = [int(v) for v in r.stdout.split()]
    assert len(got) == len(cases)
    for (V, n), g in zip(cases, got):
        rest = n - 4 * g
        launches = (g > 0) + (rest > 0)
        assert rest >= 0 and launches >= 1, (V, n, g)
        assert launches == 1 if V <= 32768 else rest < 4, (V, n, g)
