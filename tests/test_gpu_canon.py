"""The Dirac operator on the caller's canonical vectors against the same
operator staged in the internal layout (whose kernels the oracle tests cover
through the launch knobs): every tile shape, storage and the edges of the rule
that chooses between them.

Both evaluate the same products and sums per site, apart from which product of
a complex multiplication is fused: some 10^2 roundings a component."""

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

import paper_1605_00564_amd as dfl  # noqa: E402
import synth  # noqa: E402

F = dfl.Field
TOL = {dfl.F64: 1e-14, dfl.F32: 1e-6, dfl.F16: 1e-6, dfl.BF16: 1e-6}
# tiles of a whole block, several blocks, half a block, a sixth of a block (108
# of 128 positions), a block of 96 positions, the whole lattice
SHAPES = [((8, 8, 8, 16), (4, 4, 4, 4)), ((8, 8, 8, 8), (2, 2, 2, 2)), ((16, 8, 8, 8), (8, 4, 4, 4)),
          ((12, 12, 12, 12), (6, 6, 6, 6)), ((8, 8, 8, 12), (4, 4, 4, 6)), ((4, 4, 4, 4), (2, 2, 2, 2))]


def staged(fld, x, storage):
    fld.tune(F.TUNE_STENCIL_ORDER, 0)
    try:
        return dfl.dirac_apply(fld, x, storage=storage)
    finally:
        fld.tune(F.TUNE_STENCIL_ORDER, 1)


def vectors(n, V, storage, seed=3):
    dt = torch.complex128 if storage == dfl.F64 else torch.complex64
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn((n, V, 4, 3), dtype=dt, device="cuda", generator=gen)


@pytest.mark.parametrize("dims,block", SHAPES)
@pytest.mark.parametrize("storage", [dfl.F64, dfl.F32, dfl.F16, dfl.BF16])
@pytest.mark.parametrize("n", [1, 5])
def test_canonical_equals_staged(dims, block, storage, n):
    fld = dfl.Field(dims, block, 0.124, 1.5, synth.gauge_field(dims, 0.4, 1))
    x = vectors(n, fld.V, storage)
    y, z = dfl.dirac_apply(fld, x, storage=storage), staged(fld, x, storage)
    assert float((y - z).norm() / z.norm()) < TOL[storage]
    assert float((y - z).abs().max() / z.abs().max()) < 10 * TOL[storage]


@pytest.mark.parametrize("dims,block", [SHAPES[0], SHAPES[3]])
@pytest.mark.parametrize("storage", [dfl.F16, dfl.BF16])
def test_operator_held_in_registers(dims, block, storage):
    """Enough tile passes (8192) for the variant that loops over right-hand
    sides, with a last chunk that is not full."""
    fld = dfl.Field(dims, block, 0.124, 1.5, synth.gauge_field(dims, 0.4, 1))
    x = vectors(257, fld.V, storage)
    y = dfl.dirac_apply(fld, x, storage=storage)
    z = staged(fld, x, storage)
    assert float((y - z).norm() / z.norm()) < TOL[storage]
    few = dfl.dirac_apply(fld, x[250:], storage=storage)      # the other variant
    assert float((y[250:] - few).norm() / few.norm()) < TOL[storage]


@pytest.mark.parametrize("storage", [dfl.F64, dfl.F32])
def test_unaligned_and_overlapping_vectors_are_staged(storage):
    dims = (8, 8, 8, 8)
    fld = dfl.Field(dims, (4, 4, 4, 4), 0.124, 1.5, synth.gauge_field(dims, 0.4, 1))
    x = vectors(2, fld.V, storage)
    ref = staged(fld, x, storage)
    # 8 bytes past a 16-byte boundary (a view of a real buffer)
    real = torch.zeros(2 * x.numel() + 16, dtype=torch.float64 if storage == dfl.F64 else torch.float32, device="cuda")
    off = 1 if storage == dfl.F64 else 2
    u = torch.view_as_complex(real[off:off + 2 * x.numel()].view(-1, 2)) if storage == dfl.F32 else None
    if u is not None:
        u = u.view(x.shape)
        u.copy_(x)
        assert u.data_ptr() % 16 == 8
        assert torch.equal(dfl.dirac_apply(fld, u, storage=storage), ref)
        out = torch.view_as_complex(torch.empty_like(real)[off:off + 2 * x.numel()].view(-1, 2)).view(x.shape)
        assert torch.equal(dfl.dirac_apply(fld, x, storage=storage, out=out), ref)
    # input and output one vector apart in one buffer: staged, as before
    buf = torch.cat([x, x[:1]])
    y = dfl.dirac_apply(fld, buf[:2], storage=storage, out=buf[1:])
    assert torch.equal(y, ref)
