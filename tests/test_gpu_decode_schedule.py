"""The split of a large batch's items along x: items that are split and items
that run whole in one launch give the values of a launch of whole items, bit for
bit, and the default schedule is not slower than that launch."""
import numpy as np
import pytest
import torch

from gpu_util import say

pytestmark = pytest.mark.gpu


def _items(nblocks, res, rows=8):
    return nblocks * -(-res[1] // rows) * -(-res[2] // 64)


def _out(m, res, mask):
    tail = res + (4,) if mask & 0x100 else (bin(mask & 15).count("1"),) + res
    return torch.full((m.nblocks,) + tail, 777.0, device="cuda")


def _whole(fa, m, res, mask, dtype, out):
    grid = _items(m.nblocks, res) - 1  # fewer workgroups than items: whole items
    return fa.decode(m, res, mask, dtype, tune=fa.FATune(8, 8, grid, 0, 0, 0), out=out)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("mask", [15, 15 | 0x100])
@pytest.mark.parametrize("nblocks,res,segs", [
    (1024, (64, 64, 64), 4),
    (2048, (40, 32, 64), 2),   # segments of 20 positions
    (1100, (61, 60, 53), 3),   # unequal segments
], ids=str)
def test_split_and_whole_items_in_one_launch(nblocks, res, segs, mask, dtype):
    import paper_2409_00184_amd as fa
    r = np.random.default_rng(nblocks)
    deg = r.integers(1, 4, nblocks)
    ncp = r.integers(deg + 1, 33)
    assert _items(nblocks, res) >= 8192  # large enough that items may run whole
    cost = (ncp - deg + segs * (deg + 1)) * (deg + 1) ** 2
    limit = (10 if mask & 0x100 else 7) * res[0]
    assert (cost >= limit).any() and (cost < limit).any()
    m = fa.uniform_models(np.repeat(ncp[:, None], 3, 1), deg)
    m.set_ctrl(torch.randn(m.ctrl.numel(), generator=torch.Generator("cuda").manual_seed(1), device="cuda"))
    want = _whole(fa, m, res, mask, dtype, _out(m, res, mask))
    assert torch.equal(fa.decode(m, res, mask, dtype, out=_out(m, res, mask)), want)
    got = fa.decode(m, res, mask, dtype, plan=fa.Plan(m, res), out=_out(m, res, mask))
    assert torch.equal(got, want)


@pytest.mark.parametrize("plan", [False, True])
@pytest.mark.parametrize("nblocks,res,ncp,degree,mask", [
    (1024, (64, 64, 64), 32, 3, 14),
    (1024, (64, 64, 64), 32, 3, 15),
    (4096, (64, 64, 16), 8, 3, 15),
    (4096, (64, 64, 16), 16, 3, 15 | 0x100),
    (8192, (32, 32, 32), 16, 3, 15 | 0x100),
    (1024, (64, 64, 48), 16, 3, 15),
], ids=str)
def test_default_schedule_is_not_slower_than_whole_items(nblocks, res, ncp, degree, mask, plan):
    import paper_2409_00184_amd as fa
    m = fa.uniform_models(np.full((nblocks, 3), ncp), np.full(nblocks, degree))
    m.set_ctrl(torch.randn(m.ctrl.numel(), device="cuda"))
    out = _out(m, res, mask)
    p = fa.Plan(m, res) if plan else None
    # whole items in the order of the default: a plan's or the batch's
    wp = fa.Plan(m, res, 8, 8, _items(nblocks, res) - 1) if plan else None

    def best(fn, reps=12):
        ev = [(torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
              for _ in range(reps)]
        for a, b in ev:
            a.record()
            fn()
            b.record()
        torch.cuda.synchronize()
        return min(a.elapsed_time(b) for a, b in ev)

    # the sides in turn; launches of one side differ by about 5%
    w, d = [], []
    for _ in range(3):
        w.append(best(lambda: fa.decode(m, res, mask, plan=wp, out=out) if plan
                      else _whole(fa, m, res, mask, "f32", out)))
        d.append(best(lambda: fa.decode(m, res, mask, plan=p, out=out)))
    say("whole", min(w), "default", min(d))
    assert min(d) <= 1.1 * min(w)
