"""Decodes whose items are split along x, on grids that leave lanes without a
column: the same values bit for bit as unsplit items, and the oracle's."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import check_normwise, mixed_batch, models, oracle_blocks

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mask", [1, 2, 14, 15, 15 | 0x100])
@pytest.mark.parametrize("nblocks,res,ncp_hi", [
    (1, (64, 64, 64), 64),     # one block: segments of eight positions, slab in chunks
    (3, (17, 9, 65), 20),      # segments of unequal length, a second chunk of one column
    (2, (8, 3, 2), 9),         # one segment; fewer columns than lanes
    (5, (250, 7, 33), 30),
    (4096, (35, 9, 5), 6),     # a large batch of small grids: dense segments
], ids=str)
def test_split_matches_whole_items(mask, nblocks, res, ncp_hi):
    import paper_2409_00184_amd as fa
    b = mixed_batch(300 + nblocks, nblocks, ncp_hi=ncp_hi)
    m = models(b)

    def run(**kw):
        nch = bin(mask & 15).count("1")
        shape = (nblocks,) + res + (4,) if mask & 0x100 else (nblocks, nch) + res
        out = torch.full(shape, 777.0, device="cuda")
        return fa.decode(m, res, mask, out=out, **kw)

    got = run()
    whole = fa.FATune(8, 4, 1 << 20, 0, 0, 1)  # a given grid runs whole items
    assert torch.equal(got, run(tune=whole))
    assert torch.equal(got, run(plan=fa.Plan(m, res)))
    assert torch.equal(got, run(plan=fa.Plan(m, res, rows=3, waves=2, grid=7)))
    if mask == 15:
        assert torch.equal(got[:, :1], fa.decode(m, res, 1))
    take = np.unique(np.linspace(0, nblocks - 1, 5).astype(int))
    ob = oracle_blocks(b)
    sub = oracle.Blocks(b.ncp[take], b.deg[take], b.knot_off[take], b.ctrl_off[take], ob.knots, ob.ctrl)
    ref = oracle.decode_blocks(sub, res, mask & 15)
    out = got[torch.as_tensor(take).cuda()].cpu().numpy()
    check_normwise(np.moveaxis(out, -1, 1) if mask & 0x100 else out, ref, 1e-5, str((nblocks, res)))


@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("mask", [1, 14, 15, 15 | 0x100])
@pytest.mark.parametrize("nblocks,res,ncp_hi", [
    (1, (64, 64, 64), 32),
    (3, (17, 19, 66), 45),   # blocks that the tile does not take among them
    (6, (40, 33, 7), 64),
], ids=str)
def test_matrix_split_matches_whole_items(dtype, mask, nblocks, res, ncp_hi):
    import paper_2409_00184_amd as fa
    b = mixed_batch(400 + nblocks, nblocks, ncp_hi=ncp_hi)
    m = models(b)
    got = fa.decode(m, res, mask, dtype, tune=fa.FATune(0, 0, 0, 1, 0, 0))
    assert torch.equal(got, fa.decode(m, res, mask, dtype, tune=fa.FATune(0, 0, 1 << 20, 1, 0, 0)))
    assert torch.equal(got, fa.decode(m, res, mask, dtype, plan=fa.Plan(m, res, kernel=1)))
    # the 2-byte lattice on the vector ALUs: the matrix form rounds the z and
    # y bases and the z stage once more each (4 u S against u S); S of a value
    # is at most max |P| by convexity, of a derivative NCP p max |P| at most
    u = 2.0 ** -8 if dtype == "bf16" else 2.0 ** -11
    ref = fa.decode(m, res, mask, dtype)
    for k in range(nblocks):
        P = b.ctrl[int(b.ctrl_off[k]):int(b.ctrl_off[k]) + int(np.prod(b.ncp[k]))]
        S = np.abs(P).max() * (1.0 if mask == 1 else float((b.ncp[k] * b.deg[k]).max()) * 64.0)
        assert float((got[k] - ref[k]).abs().max()) <= 7.0 * u * S
