"""Restriction and prolongation at the edges of their launch rules: tiles of
right-hand sides (1, 4, 5, 8, 9, 16, 17, 25), one and two tiles of fields
(N_s = 20 > 16), blocks small enough for four waves (2^4: 96 elements) and
larger ones, deflation blocks of several Schwarz blocks, runs that are not a
multiple of the stride (2 x 6 x 2 x 2: 12 sites per parity).

Reference: the exported basis in FP64 (torch).  FP64 vectors: sums of at most
24 x 256 terms in another order, 1e-12; FP32 vectors: FP32 products and sums,
1e-5 as in the other restriction tests, prolongation rounded once, 1e-6.
"""

import pytest

import synth

pytestmark = pytest.mark.gpu

CASES = [((8, 8, 8, 8), (2, 2, 2, 2), None), ((8, 8, 8, 8), (2, 2, 2, 2), (4, 4, 2, 2)),
         ((8, 8, 8, 8), (4, 4, 4, 4), None), ((4, 12, 4, 4), (2, 6, 2, 2), None)]


def to_blocks(v, dims, block):
    """(n, V, 4, 3) lexicographic -> (Nb, n, Vb 12)"""
    n = v.shape[0]
    shape = [n]
    for L, b in zip(dims, block):
        shape += [L // b, b]
    v = v.reshape(*shape, 12).permute(1, 3, 5, 7, 0, 2, 4, 6, 8, 9)
    nb = v.shape[0] * v.shape[1] * v.shape[2] * v.shape[3]
    return v.reshape(nb, n, -1)


@pytest.mark.parametrize("case", range(len(CASES)))
@pytest.mark.parametrize("Ns", [3, 20])
def test_restrict_and_prolong(case, Ns):
    import torch
    import paper_1605_00564_amd as dfl
    dims, block, dblock = CASES[case]
    fld = dfl.Field(dims, block, 0.120, 1.0, synth.gauge_field(dims, 0.3, 2))
    d = dfl.Deflation(fld, Ns=Ns, ninv=0, seed=5, block=dblock)
    db = dblock or block
    phi = d.get_phi().reshape(d.Nb, Ns, -1)
    g = torch.Generator(device="cuda").manual_seed(9)
    for n in (1, 4, 5, 8, 9, 16, 17, 25):
        v = torch.randn((n, fld.V, 4, 3), dtype=torch.complex128, device="cuda", generator=g)
        for dt, tol in ((torch.complex128, 1e-12), (torch.complex64, 1e-5)):
            vb = to_blocks(v.to(dt).to(torch.complex128), dims, db)
            want = torch.stack([(phi.conj() * vb[:, r, None, :]).sum(-1) for r in range(n)])
            got = d.restrict(v.to(dt))
            assert float((got - want).norm() / want.norm()) <= tol, (n, dt)
            ptol = 1e-12 if dt == torch.complex128 else 1e-6
            back = to_blocks(d.prolong(want, dt).to(torch.complex128), dims, db)
            for r in range(n):
                ref = (want[r][:, :, None] * phi).sum(1)
                assert float((back[:, r] - ref).norm() / ref.norm()) <= ptol, (n, dt, r)
    d.close()
    fld.close()
