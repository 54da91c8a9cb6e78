"""Items split along x against the same items whole: grids below the item count,
which fa_decode_blocks never splits; the matrix-core decode with its vector form
against the oracle element by element; more items than workgroups."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from gpu_util import U32, mixed_batch, models, oracle_blocks

pytestmark = pytest.mark.gpu
ULP = {"bf16": 2.0 ** -8, "f16": 2.0 ** -11}


def _decode(fa, m, res, mask, dtype, **kw):
    nch = bin(mask & 15).count("1")
    shape = (m.nblocks,) + res + (4,) if mask & 0x100 else (m.nblocks, nch) + res
    return fa.decode(m, res, mask, dtype, out=torch.full(shape, 777.0, device="cuda"), **kw)


def _items(nblocks, res, rows):
    return nblocks * -(-res[1] // rows) * -(-res[2] // 64)


@pytest.mark.parametrize("mask", [1, 2, 14, 15, 15 | 0x100])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("nblocks,res,ncp_hi", [
    (1, (64, 64, 64), 64),     # segments of eight positions, slab in chunks
    (3, (17, 9, 65), 20),      # segments of unequal length, a column tile of one
    (5, (250, 9, 33), 30),
], ids=str)
def test_vector_segments_match_whole_items(dtype, mask, nblocks, res, ncp_hi):
    import paper_2409_00184_amd as fa
    m = models(mixed_batch(600 + nblocks, nblocks, ncp_hi=ncp_hi))
    items = _items(nblocks, res, 8)
    grid = items - 1
    assert 0 < grid < items and res[0] >= 16 and 2 * items <= 1024  # split by default
    want = _decode(fa, m, res, mask, dtype, tune=fa.FATune(8, 4, grid, 0, 0, 0))
    assert not (want == 777.0).any()
    for kw in (dict(), dict(plan=fa.Plan(m, res)), dict(tune=fa.FATune(8, 8, 0, 0, 4096, 1)),
               dict(plan=fa.Plan(m, res, rows=3, waves=2, grid=grid))):
        assert torch.equal(_decode(fa, m, res, mask, dtype, **kw), want)


@pytest.mark.parametrize("mask", [1, 2, 14, 15, 15 | 0x100])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("nblocks,res,ncp_hi", [
    (1, (64, 64, 64), 32),
    (3, (17, 19, 66), 45),   # blocks that the tile does not take among them
    (6, (40, 33, 7), 64),
], ids=str)
def test_matrix_segments_match_whole_items(dtype, mask, nblocks, res, ncp_hi):
    import paper_2409_00184_amd as fa
    m = models(mixed_batch(700 + nblocks, nblocks, ncp_hi=ncp_hi))
    items = _items(nblocks, res, 16)
    grid = items - 1
    assert 0 < grid < items and res[0] >= 16 and 2 * items <= 512  # split by default
    want = _decode(fa, m, res, mask, dtype, tune=fa.FATune(0, 0, grid, 1, 0, 0))
    assert not (want == 777.0).any()
    for kw in (dict(tune=fa.FATune(0, 0, 0, 1, 0, 0)), dict(plan=fa.Plan(m, res, kernel=1)),
               dict(plan=fa.Plan(m, res, kernel=1, grid=grid))):
        assert torch.equal(_decode(fa, m, res, mask, dtype, **kw), want)


@pytest.mark.parametrize("mask", [1, 2, 4, 8, 14, 15, 15 | 0x100])
@pytest.mark.parametrize("dtype", ["bf16", "f16"])
@pytest.mark.parametrize("nblocks,res,ncp_hi,seed", [(3, (17, 19, 66), 45, 823), (6, (24, 33, 7), 64, 806)],
                         ids=str)
def test_matrix_decode_and_its_vector_form_against_oracle(dtype, mask, nblocks, res, ncp_hi, seed):
    """Every element within (6 u + 64 u32) S, S the oracle's sum of absolute
    products: the lattice, the z and y bases and the z stage are rounded to the
    input type (items of the vector form round the lattice alone)."""
    import paper_2409_00184_amd as fa
    b = mixed_batch(seed, nblocks, ncp_hi=ncp_hi)
    assert (b.ncp[:, 2] > 32).any() and (b.ncp[:, 2] <= 32).any()  # both forms
    m = models(b)
    got = _decode(fa, m, res, mask, dtype, tune=fa.FATune(0, 0, 0, 1, 0, 0))
    got = (got if mask & 0x100 else got.permute(0, 2, 3, 4, 1)).cpu().numpy()
    idx = np.stack(np.meshgrid(*(np.arange(n) for n in (nblocks,) + res), indexing="ij"), -1)
    ref, S = oracle.decode_samples(oracle_blocks(b), res, idx.reshape(-1, 4).astype(np.int32), with_abs=True)
    chans = [c for c in range(4) if mask >> c & 1]
    err = np.abs(got.reshape(-1, len(chans)).astype(np.float64) - ref[:, chans])
    lim = (6.0 * ULP[dtype] + 64 * U32) * S[:, chans] + 1e-30
    assert (err <= lim).all(), float((err / lim).max())


@pytest.mark.parametrize("mask", [1, 15, 15 | 0x100])
@pytest.mark.parametrize("kernel", [0, 1])
def test_more_items_than_workgroups(kernel, mask):
    """2^20 + 5 items, where a workgroup takes several: the values of the same
    micro-models in two batches of fewer items than that."""
    import paper_2409_00184_amd as fa
    n, res = (1 << 20) + 5, (3, 2, 5)
    desc = fa.host_descriptors(np.full((n, 3), 2, np.int32), np.ones((n, 3), np.int32),
                               np.zeros(n, np.int64), 8 * np.arange(n, dtype=np.int64))
    d = torch.from_numpy(desc.view(np.uint8)).cuda()
    knots = torch.tensor([0.0, 0.0, 1.0, 1.0] * 3, device="cuda")
    ctrl = torch.randn(8 * n, generator=torch.Generator("cuda").manual_seed(7), device="cuda")
    if kernel:
        ctrl = ctrl.bfloat16()

    def run(lo, hi):
        nch = bin(mask & 15).count("1")
        out = torch.full((hi - lo, nch * 30), 777.0, device="cuda")
        t = fa.FATune(0, 0, 0, kernel, 0, 0)
        st = fa.lib.fa_decode_blocks(d.data_ptr() + 64 * lo, hi - lo, knots.data_ptr(), ctrl.data_ptr(),
                                     fa.FA_BF16 if kernel else fa.FA_F32, fa._i32x3(res), mask,
                                     ctypes.byref(t), None, None, 0, out.data_ptr(),
                                     torch.cuda.current_stream().cuda_stream)
        assert st == 0
        return out

    half = n // 2
    got = run(0, n)
    assert not (got == 777.0).any()
    assert torch.equal(got[:half], run(0, half)) and torch.equal(got[half:], run(half, n))
