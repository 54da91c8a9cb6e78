"""The fit's matrix-core kernels at the edges of their 16-wide tiles, and the
lattice-size search with the smallest workspace it takes."""
import ctypes

import numpy as np
import pytest
import torch

import fa_inputs as fi
from test_gpu_adaptive import U32, _oracle_fit, tol_from

pytestmark = pytest.mark.gpu

# grid, (NCP per axis, degree) of each block: tiles of 16 samples and 16
# functions just full, one more and one less; rows that are not whole 16-byte
# vectors; the smallest and the largest grid; one function per sample
CASES = [
    ((16, 16, 16), [((16, 16, 16), 3), ((4, 15, 9), 3), ((15, 4, 16), 1)]),
    ((17, 15, 18), [((17, 8, 16), 2), ((5, 15, 17), 3)]),
    ((33, 48, 31), [((16, 32, 17), 3), ((32, 17, 16), 2), ((8, 33, 24), 3)]),
    ((64, 64, 64), [((48, 33, 32), 3), ((31, 47, 49), 2)]),
    ((64, 32, 63), [((40, 16, 40), 3)]),
    ((2, 5, 3), [((2, 4, 3), 1), ((2, 2, 2), 1)]),
]


@pytest.mark.parametrize("R,blocks", CASES, ids=["x".join(map(str, c[0])) for c in CASES])
def test_fit_at_tile_edges(R, blocks):
    import paper_2409_00184_amd as fa
    g = fi.rng(sum(R))
    m = fa.uniform_models([b[0] for b in blocks], [b[1] for b in blocks])
    Y = g.normal(size=(len(blocks),) + R).astype(np.float32)
    before = m.ctrl.clone()
    fa.fit(m, R, torch.as_tensor(Y).cuda())
    got = m.ctrl.cpu().numpy().astype(np.float64)
    inside = np.zeros(got.size, bool)
    for b, (n, p, ks, P) in enumerate(_oracle_fit(m, Y)):
        o = int(m.host_desc["ctrl_off"][b])
        inside[o:o + P.size] = True
        err = np.abs(got[o:o + P.size].reshape(n) - P)
        assert np.all(err <= U32 * np.abs(P) + tol_from(P, n, p, R, c32=0.0)), (n, p)
    assert np.array_equal(got[~inside], before.cpu().numpy()[~inside])  # gaps between lattices


def test_search_with_the_least_workspace():
    """One candidate at a time (the smallest workspace that the call takes)
    and several at a time: the same error map, bit for bit."""
    import paper_2409_00184_amd as fa
    g = fi.rng(5)
    R, nb, p = (16, 18, 17), 3, 2
    y = torch.as_tensor(g.normal(size=(nb,) + R).astype(np.float32)).cuda()
    lo, hi = 4, 16
    ref = fa.ncp_search(y, p, lo, hi)
    res = (ctypes.c_int32 * 3)(*R)
    least = fa.lib.fa_ncp_search_workspace(nb, res, p, hi)
    wide = fa.lib.fa_ncp_search_workspace_wide(nb, res, p, hi)
    assert wide > least
    ws = torch.empty(wide, dtype=torch.uint8, device="cuda")
    for size in (least, wide - 1, wide):
        out = torch.full_like(ref, -1.0)
        assert fa.lib.fa_ncp_search(y.data_ptr(), nb, res, p, lo, hi, out.data_ptr(), ws.data_ptr(), size,
                                    torch.cuda.current_stream().cuda_stream) == fa.FA_OK
        assert torch.equal(out, ref), size
