"""Little operator and its solve at the edges of their launch rules: one and
two tiles of N_s (20 > 16), narrow, wide and several tiles of right-hand
sides (8, 9, 17, 25), one workgroup per right-hand side and many, four waves
per row and one (more than 3072 tiles: 1024 blocks, N_s = 20, 25 right-hand
sides).

The product with many right-hand sides is compared with one at a time (pinned
to the oracle elsewhere): sums of at most 9 x 20 terms in FP64 in another
order, 1e-13 of the norm.  The solve is judged by its residual: the tolerance
plus the rounding of the product, 1e-12; with a tolerance below the rounding it
goes through a restart after 24 steps.
"""

import pytest

import synth

pytestmark = pytest.mark.gpu

SMALL, MANY = ((8, 8, 8, 8), (4, 4, 4, 4)), ((16, 16, 8, 8), (2, 2, 2, 2))
_fields = {}


def deflation(geometry, Ns):
    import paper_1605_00564_amd as dfl
    if geometry not in _fields:
        dims, block = geometry
        _fields[geometry] = dfl.Field(dims, block, 0.120, 1.0, synth.gauge_field(dims, 0.3, 2))
    return dfl.Deflation(_fields[geometry], Ns=Ns, ninv=2, seed=21)


@pytest.mark.parametrize("geometry,Ns,n", [
    (SMALL, 1, 1), (SMALL, 12, 8), (SMALL, 16, 9), (SMALL, 20, 17), (SMALL, 20, 25),
    (MANY, 5, 1), (MANY, 12, 16), (MANY, 20, 24), (MANY, 20, 25)])
def test_little_product_and_solve(geometry, Ns, n):
    import torch
    d = deflation(geometry, Ns)
    g = torch.Generator(device="cuda").manual_seed(3)
    v = torch.randn((n, d.Nb, Ns), dtype=torch.complex128, device="cuda", generator=g)
    both = d.little_apply(v)
    for r in (0, n // 2, n - 1):
        one = d.little_apply(v[r:r + 1])[0]
        assert float((both[r] - one).norm() / one.norm()) <= 1e-13
    for tol in (1e-4, 1e-10):
        w, iters = d.little_solve(v, tol=tol)
        res = (d.little_apply(w) - v).flatten(1).norm(dim=1) / v.flatten(1).norm(dim=1)
        assert float(res.max()) <= tol + 1e-12 and 0 < iters < 500
        # the last step was needed
        w, fewer = d.little_solve(v, tol=tol, maxit=max(1, iters - 1))
        res = (d.little_apply(w) - v).flatten(1).norm(dim=1) / v.flatten(1).norm(dim=1)
        assert fewer == max(1, iters - 1) and (iters == 1 or float(res.max()) > tol - 1e-12)
    w, iters = d.little_solve(v, tol=1e-30, maxit=53)
    assert 24 < iters <= 53   # the recurrence's own residual may get there after the restart
    res = (d.little_apply(w) - v).flatten(1).norm(dim=1) / v.flatten(1).norm(dim=1)
    assert float(res.max()) <= 1e-12
    d.close()
