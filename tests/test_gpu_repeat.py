"""The same inputs give the same bits: the little operator rebuilt from one
set of fields, and solves on two handles built alike.

A store whose data registers were overwritten too early once changed single
elements by 1e-10 to 1e-7 from run to run."""

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_1605_00564_amd as dfl  # noqa: E402
import synth  # noqa: E402

DIMS, BLOCK = (16, 16, 16, 16), (4, 4, 4, 4)


def test_little_operator_rebuilt_alike():
    fld = dfl.Field(DIMS, BLOCK, 0.124, 1.5, synth.gauge_field(DIMS, 0.4, 1))
    d = dfl.Deflation(fld, Ns=12, ninv=2, seed=7)
    phi = d.get_phi()
    gen = torch.Generator(device="cuda").manual_seed(5)
    v = torch.view_as_complex(torch.randn((2, d.Nb, d.Ns, 2), dtype=torch.float64, device="cuda", generator=gen))
    first = d.little_apply(v).clone()
    for _ in range(4):
        d.set_phi(phi)
        assert torch.equal(d.little_apply(v), first)
    # and the rebuilt operator is Phi^+ M Phi to FP64 rounding (2 V_b Ns terms an entry)
    w = d.restrict(dfl.dirac_apply(fld, d.prolong(v), storage=dfl.F64))
    assert float((w - first).norm() / w.norm()) < 1e-13


@pytest.mark.parametrize("n", [1, 2])
def test_deflated_solves_on_two_handles(n):
    U = synth.gauge_field(DIMS, 0.4, 1)
    b = torch.from_numpy(np.stack([synth.point_source(DIMS, synth.seeded_site(DIMS, 1), k) for k in range(n)])).cuda()
    out = []
    for _ in range(2):
        fld = dfl.Field(DIMS, BLOCK, 0.124, 1.5, U)
        d = dfl.Deflation(fld, Ns=8, ninv=2, seed=7)
        p = dfl.GcrParams(nkv=8, nmx=60, res=1e-10, sap=dfl.SapParams(5, 4, dfl.F32), dfl=d, little_tol=1e-10)
        out.append(dfl.gcr_solve(fld, b, p)[0])
    assert torch.equal(out[0], out[1])
