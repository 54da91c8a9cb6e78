"""The adjoint's forms: every set of channels, rows that are and are not
whole 16-byte vectors, micro-models split between workgroups (few blocks) or
not (many), lattices with and without a copy of their planes per chunk, and
planes that no grid position touches."""
import numpy as np
import pytest
import torch

import fa_inputs as fi
import oracle
from gpu_util import check_normwise, mixed_batch, models, oracle_blocks

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mask", [1, 2, 4, 8, 9, 6, 14, 15])
@pytest.mark.parametrize("res,nblocks,ncp_hi", [
    ((20, 18, 22), 3, 20),   # ragged rows
    ((33, 64, 63), 2, 40),   # tiles and bands of every width
    ((64, 16, 16), 1, 9),    # one block: eight segments of a small lattice
    ((7, 5, 3), 4, 12),      # more functions than positions; rows below one vector
    ((9, 12, 8), 300, 6),    # one workgroup per block
    ((200, 17, 33), 5, 33),  # slices beyond one 64-bit word of the span table
], ids=str)
def test_adjoint_against_oracle(mask, res, nblocks, ncp_hi):
    import paper_2409_00184_amd as fa
    b = mixed_batch(100 + nblocks, nblocks, ncp_hi=ncp_hi)
    m = models(b)
    nch = bin(mask).count("1")
    g = fi.rng(7).normal(size=(nblocks, nch) + res).astype(np.float32)
    # a sentinel shows a plane left out and a value written outside a lattice
    G = torch.full_like(m.ctrl, 777.0)
    fa.decode_backward(m, res, torch.as_tensor(g).cuda(), mask, grad_ctrl=G)
    got = G.cpu().numpy()
    again = fa.decode_backward(m, res, torch.as_tensor(g).cuda(), mask, grad_ctrl=torch.full_like(G, 777.0))
    assert np.array_equal(again.cpu().numpy(), got)  # deterministic
    ref = oracle.decode_adjoint(oracle_blocks(b), res, g.astype(np.float64), mask)
    inside = np.zeros(got.size, bool)
    for k in range(nblocks):
        o, n = int(b.ctrl_off[k]), int(np.prod(b.ncp[k]))
        inside[o:o + n] = True
        check_normwise(got[None, None, o:o + n], ref[None, None, o:o + n], what=f"block {k} {b.ncp[k]}")
    assert np.all(got[~inside] == 777.0)
