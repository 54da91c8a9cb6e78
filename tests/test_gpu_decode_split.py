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
