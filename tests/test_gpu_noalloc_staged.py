"""dirac_apply_noalloc where the vectors do pass through the static device array: io
and vector precision differ, vectors off a 16-byte boundary, input and output one
vector apart in one buffer, a stencil chosen on the handle.  Each time two calls in
a row, the second with fewer right-hand sides and on a smaller lattice, so that
what the first left in the array would show.  dirac_apply stages the same vectors
in work space, through the same kernels: the outputs are identical.  No work space
is taken, and calls beyond the array are refused whichever way they would go."""

import pytest

import synth

pytestmark = pytest.mark.gpu

F64, F32, F16, BF16 = 0, 1, 2, 3
CASES = [((8, 8, 8, 16), 6), ((8, 8, 8, 8), 2)]     # second call: smaller input


def _gpu():
    import torch
    import paper_1605_00564_amd as dfl
    return torch, dfl


def _vectors(torch, V, n, dtype, off=0, seed=3):
    """n random vectors, `off` real numbers past the start of their buffer."""
    real = torch.float64 if dtype == torch.complex128 else torch.float32
    g = torch.Generator(device="cuda").manual_seed(seed)
    buf = torch.zeros(24 * V * n + 16, dtype=real, device="cuda")
    x = torch.view_as_complex(buf[off:off + 24 * V * n].view(-1, 2)).view(n, V, 4, 3)
    x.copy_(torch.randn((n, V, 4, 3), dtype=dtype, device="cuda", generator=g))
    return x


def _no_work_space(dfl, fld, call):
    fld.trim()
    dfl.workspace_trim()
    call()
    fld.trim()
    assert dfl.workspace_cached(0) == 0


@pytest.mark.parametrize("what", ["mixed", "unaligned", "overlap", "tuned", "converted"])
@pytest.mark.parametrize("storage", [F64, F32, F16, BF16])
def test_staged_calls_match_dirac_apply(what, storage):
    torch, dfl = _gpu()
    own = torch.complex128 if storage == F64 else torch.complex64
    other = torch.complex64 if storage == F64 else torch.complex128
    dt, off = (other if what == "mixed" else own), (2 if what == "unaligned" and own == torch.complex64 else 0)
    for dims, n in CASES:
        fld = dfl.Field(dims, (4, 4, 4, 4), 0.124, 1.5, synth.gauge_field(dims, 0.4, 1))
        if what == "tuned":
            fld.tune(dfl.Field.TUNE_STENCIL_BLOCK, 0)
        if what == "converted":
            fld.tune(dfl.Field.TUNE_DIRAC_CANON, 2)
        if what == "overlap":
            both = _vectors(torch, fld.V, n + 1, dt)
            x, out = both[:n], both[1:]
            ref = dfl.dirac_apply(fld, x.clone(), storage=storage, out=torch.empty_like(x))
            tol = 1e-14 if storage == F64 else 1e-6     # the reference is not staged
        else:
            x, out = _vectors(torch, fld.V, n, dt, off), _vectors(torch, fld.V, n, dt, off, seed=4)
            ref = dfl.dirac_apply(fld, x, storage=storage)
            tol = 0.0
        assert off == 0 or x.data_ptr() % 16 == 8
        _no_work_space(dfl, fld, lambda: dfl.dirac_apply_noalloc(fld, x, out, storage=storage))
        torch.cuda.synchronize()
        assert float((out - ref).norm() / ref.norm()) <= tol, (dims, n)
        fld.close()


def test_the_limit_does_not_depend_on_the_route():
    """22 FP32 vectors of 16384 sites need 2 x 22 x 16384 x 96 bytes = 69.2 MB > 64 MiB."""
    torch, dfl = _gpu()
    dims = (16, 16, 8, 8)
    fld = dfl.Field(dims, (4, 4, 4, 4), 0.124, 1.5, synth.gauge_field(dims, 0.4, 1))
    for n, fits in ((21, True), (22, False)):
        x = torch.zeros((n, fld.V, 4, 3), dtype=torch.complex64, device="cuda")
        for canon in (1, 2):
            fld.tune(dfl.Field.TUNE_DIRAC_CANON, canon)
            if fits:
                dfl.dirac_apply_noalloc(fld, x, torch.empty_like(x), storage=F32)
            else:
                with pytest.raises(dfl.DflError) as e:
                    dfl.dirac_apply_noalloc(fld, x, torch.empty_like(x), storage=F32)
                assert e.value.code == -1
    fld.close()
