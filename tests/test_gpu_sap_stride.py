"""Schwarz sweeps on both sides of the rule for a fixed stride of the exchange
buffers (more than 384 sites per parity and at most 744): blocks of 384, 448,
720 and 768, against the quantised oracle with the bounds of the other
Schwarz tests (FP32 storage 1e-6; BF16 storage with FP16 vectors
n_cy 2^-11).
"""

import numpy as np
import pytest

import synth
from tests.test_gpu_ops import BF16, F16, F32, SAP_TOL, SAP_TOL_V16, Case, rel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,block", [
    ((8, 8, 12, 16), (4, 4, 6, 8)), ((8, 8, 8, 28), (4, 4, 4, 14)),
    ((8, 12, 12, 20), (4, 6, 6, 10)), ((8, 8, 8, 48), (4, 4, 4, 24))])
def test_sap_blocks_around_the_stride_rule(dims, block):
    import torch
    import paper_1605_00564_amd as dfl
    c = Case(dims, block, 0.3, 0.120, 1.0)
    eta = synth.gaussian_spinor(dims, 1, 1011).astype(np.complex64)
    for storage, vecs, tol in ((F32, F32, SAP_TOL[F32]), (BF16, F16, SAP_TOL_V16)):
        psi = dfl.sap_precond(c.field, torch.from_numpy(eta).cuda(), dfl.SapParams(5, 4, storage, vecs)).cpu().numpy()
        ref = c.qop(storage).sap(eta.astype(np.complex128), block, 5, 4)
        assert rel(psi[0], ref[0]) <= tol, (storage, rel(psi[0], ref[0]))
    c.field.close()
