"""qcd_field_ape_smear when the device has room for one of its two buffers only: the
call fails, and the handle still says that it has no smeared links instead of
handing out memory that nothing wrote.  With the room back the call succeeds."""

import pytest

pytestmark = pytest.mark.gpu

DIMS, BLOCK = (32, 32, 32, 32), (4, 4, 4, 4)


def test_a_failed_first_smearing_leaves_no_links():
    import torch
    import paper_1605_00564_amd as dfl
    V = 32 ** 4
    U = torch.eye(3, dtype=torch.complex128, device="cuda").expand(V, 4, 3, 3).contiguous()
    fld = dfl.Field(DIMS, BLOCK, 0.124, 1.0, U)
    x = torch.zeros((1, V, 4, 3), dtype=torch.complex64, device="cuda")
    torch.cuda.synchronize()
    dfl.workspace_trim()
    torch.cuda.empty_cache()
    each = 27 * 16 * V                       # the links, and the scratch of the steps
    free, _ = torch.cuda.mem_get_info()
    hog = [torch.empty(free - 3 * each // 2, dtype=torch.uint8, device="cuda")]
    # the free count leaves out a reserve: take that in quarters, then give six back
    for _ in range(64):
        try:
            hog.append(torch.empty(each // 4, dtype=torch.uint8, device="cuda"))
        except torch.OutOfMemoryError:
            break
    else:
        pytest.skip("the device's memory has no end here")
    del hog[-6:]
    torch.cuda.empty_cache()
    with pytest.raises(dfl.DflError) as e:
        fld.ape_smear(0.5, 2)
    assert e.value.code == -3             # out of memory
    del hog
    torch.cuda.empty_cache()
    for use in (fld.ape_links, lambda: dfl.gauss_smear(fld, x, 0.2, 1)):
        with pytest.raises(dfl.DflError) as e:
            use()
        assert e.value.code == -7            # not set
    fld.ape_smear(0.5, 2)
    # unit links stay unit links
    assert float((fld.ape_links() - U[:, 1:]).abs().max()) <= 1e-15
    fld.close()
