"""CPU check of qcd_field_ape_smear when an allocation or a launch fails
(tests/ape_failure_check.cpp: the host code of csrc/smear.hip with stand-ins for
the device): a handle without smeared links still has none, and later calls say
so instead of using memory that nothing wrote; one with links keeps them."""

import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1605_00564_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")


def test_a_failed_smearing_leaves_the_handle_as_it_was(tmp_path):
    if not os.path.exists(HIPCC):
        pytest.skip("hipcc not available")
    obj, exe = str(tmp_path / "check.o"), str(tmp_path / "check")
    for cmd in ([HIPCC, "-x", "hip", "--offload-arch=gfx950", "--cuda-host-only", "-O1", "-std=c++17", "-Wno-unused-result",
                 "-I", CSRC, "-I", os.path.join(ROOT, "include"), "-c",
                 os.path.join(ROOT, "tests", "ape_failure_check.cpp"), "-o", obj],
                # the device code is not there: only its address is left open
                ["g++", obj, "-o", exe, "-no-pie", "-Wl,--unresolved-symbols=ignore-all"]):
        r = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
        assert r.returncode == 0, r.stderr
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0, r.stderr
