"""CPU check of the canonical-vector stencil's tiles (csrc/block_tables.h): they divide
the lattice into parts of blocks or whole blocks, and block shapes whose tiles
leave more than half of a workgroup idle (an extent of twice a prime above 128) are
not put on that stencil: it took up to 4.5 times as long there as the one between
conversions."""

import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1605_00564_amd", "csrc")
FLAGS = ["-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
         "-fno-omit-frame-pointer"]
EVEN = [b for b in range(2, 33, 2)]
SMALL = [(a, b, c, d) for a in EVEN for b in EVEN for c in (2, 4, 6) for d in (2, 4)]
# (block, whether its tiles are used)
LARGE = [((2, 2, 2, 134), True), ((2, 6, 2, 134), True), ((4, 4, 4, 262), True), ((2, 2, 2, 254), True),
         ((4, 4, 2, 262), False), ((2, 2, 6, 262), False), ((2, 2, 2, 262), False), ((262, 2, 2, 2), False)]


def test_tiles(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "check")
    r = subprocess.run(["g++", *FLAGS, "-I", CSRC, os.path.join(ROOT, "tests", "tile_rule_check.cpp"), "-o", exe],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    cases = [(b, True) for b in SMALL] + LARGE
    sizes = [(b[0] * b[1] * b[2] * b[3] // 2, nb) for b, _ in cases for nb in (16, 48, 2592)]
    r = subprocess.run([exe], input="".join(f"{v} {nb}\n" for v, nb in sizes), capture_output=True, text=True,
                       timeout=60)
    assert r.returncode == 0, r.stderr
    got = [tuple(int(v) for v in line.split()) for line in r.stdout.splitlines()]
    assert len(got) == len(sizes)
    for i, ((vbh, nb), (P, used)) in enumerate(zip(sizes, got)):
        block, expect = cases[i // 3]
        assert 0 < P <= 128 and (vbh % P == 0 or (P % vbh == 0 and nb % (P // vbh) == 0)), (block, P)
        assert bool(used) == expect == (P >= 64), (block, P)
