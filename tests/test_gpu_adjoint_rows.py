"""The adjoint's row bands: one, two or four groups of 16 cotangent rows, at
the resolutions where the number changes, against the oracle.  The bound is
that of the other adjoint tests (1e-5 of the largest magnitude of a block)."""
import numpy as np
import pytest
import torch

import fa_inputs as fi
import oracle
from gpu_util import check_normwise, mixed_batch, models, oracle_blocks

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mask", [1, 6, 15])
@pytest.mark.parametrize("rz", [16, 13])  # rows of whole 16-byte vectors, and not
@pytest.mark.parametrize("ry", [2, 15, 16, 17, 31, 32, 33, 64])
def test_row_bands(ry, rz, mask):
    import paper_2409_00184_amd as fa
    res, nblocks = (11, ry, rz), 5
    b = mixed_batch(500 + ry, nblocks, ncp_hi=20)
    m = models(b)
    g = fi.rng(ry).normal(size=(nblocks, bin(mask).count("1")) + res).astype(np.float32)
    G = torch.full_like(m.ctrl, 777.0)
    fa.decode_backward(m, res, torch.as_tensor(g).cuda(), mask, grad_ctrl=G)
    got = G.cpu().numpy()
    ref = oracle.decode_adjoint(oracle_blocks(b), res, g.astype(np.float64), mask)
    for k in range(nblocks):
        o, n = int(b.ctrl_off[k]), int(np.prod(b.ncp[k]))
        check_normwise(got[None, None, o:o + n], ref[None, None, o:o + n], what=f"block {k} {b.ncp[k]}")
