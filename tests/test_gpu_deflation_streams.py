"""A deflation handle is complete when the call that built it returns, so that it
can be used on another stream than the one that built it: nothing is left queued
on that stream, and a solve on a second stream finds the same folded couplings,
bit for bit, as one on the first."""

import pytest

import synth

pytestmark = pytest.mark.gpu

# large enough that its last kernels take some hundred microseconds
DIMS, BLOCK, NS = (16, 16, 16, 16), (2, 2, 2, 2), 20


def test_handle_is_complete_on_return():
    import torch
    import paper_1605_00564_amd as dfl
    fld = dfl.Field(DIMS, BLOCK, 0.120, 1.0, synth.gauge_field(DIMS, 0.3, 2))
    torch.cuda.synchronize()
    build, use = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(build):
        d = dfl.Deflation(fld, Ns=NS, ninv=1, seed=21)
    assert build.query()
    with torch.cuda.stream(use):
        v = torch.randn((2, d.Nb, NS), dtype=torch.complex128, device="cuda")
        other, _ = d.little_solve(v, tol=1e-10)
    torch.cuda.synchronize()
    with torch.cuda.stream(build):
        own, _ = d.little_solve(v, tol=1e-10)
    torch.cuda.synchronize()
    assert torch.equal(own, other)
    phi = d.get_phi()
    torch.cuda.synchronize()
    with torch.cuda.stream(build):
        d.set_phi(phi)
    assert build.query()
    with torch.cuda.stream(use):
        again, _ = d.little_solve(v, tol=1e-10)
    torch.cuda.synchronize()
    # the subspace read back in FP32 is the one that was there
    res = (d.little_apply(again) - v).flatten(1).norm(dim=1) / v.flatten(1).norm(dim=1)
    assert torch.equal(again, own) and float(res.max()) <= 1e-10 + 1e-12
    d.close()
    fld.close()
