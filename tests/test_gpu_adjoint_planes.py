"""The adjoint of derivative cotangents with x first: lattices of few planes
for their slices, or of more columns than two tiles, against the oracle, with
one, two and four row bands, with segments (few blocks) and without; and an
infinite and a NaN value, which reach their windows and nothing else.  The
last shapes are near the line between the two forms, on either side of it."""
import numpy as np
import pytest
import torch

import fa_inputs as fi
import oracle
from gpu_util import check_normwise, models, oracle_blocks

pytestmark = pytest.mark.gpu

SHAPES = [  # resolution, NCP, degree, blocks
    ((64, 64, 64), (40, 40, 40), 1, 1),     # eight segments
    ((40, 41, 43), (40, 40, 40), 2, 2),     # rows that are not whole vectors
    ((64, 33, 17), (3, 33, 17), 2, 130),    # no segments
    ((60, 12, 63), (2, 36, 50), 1, 2),      # one row band, more functions than rows
    ((30, 17, 33), (2, 17, 33), 1, 130),    # two row bands
    ((33, 64, 64), (3, 64, 64), 1, 1),      # fewer planes than segments
    ((100, 20, 30), (4, 16, 32), 3, 2),
    ((64, 64, 64), (16, 16, 16), 3, 2),
]


def _batch(ncp, p, nblocks):
    n = nblocks
    kl = [[fi.clamped_uniform_knots(a, p) if (b + i) % 3 else fi.jittered_knots(fi.rng(b), a, p)
           for i, a in enumerate(ncp)] for b in range(n)]
    return fi.pack([list(ncp)] * n, [[p] * 3] * n, kl, [np.zeros(ncp)] * n)


def _spans(t, n, R):
    u = np.arange(R, dtype=np.float32) / np.float32(R - 1)
    return np.minimum(np.searchsorted(t[:n + 1], u, side="right") - 1, n - 1)


@pytest.mark.parametrize("mask", [2, 6, 9, 14, 15])
@pytest.mark.parametrize("res,ncp,p,nblocks", SHAPES, ids=str)
def test_planes_against_oracle(res, ncp, p, nblocks, mask):
    import paper_2409_00184_amd as fa
    b = _batch(ncp, p, nblocks)
    m = models(b)
    nch = bin(mask).count("1")
    r = fi.rng(sum(res) + mask)
    g = r.normal(size=(nblocks, nch) + res).astype(np.float32)
    G = torch.full_like(m.ctrl, 777.0)
    got = fa.decode_backward(m, res, torch.as_tensor(g).cuda(), mask, grad_ctrl=G).cpu().numpy()
    again = fa.decode_backward(m, res, torch.as_tensor(g).cuda(), mask, grad_ctrl=G).cpu().numpy()
    assert np.array_equal(again, got)  # deterministic
    # one value of the first block not finite
    at = tuple(int(r.integers(0, n)) for n in res)
    g[(0, int(r.integers(0, nch))) + at] = np.nan if mask & 1 else np.inf
    bad = fa.decode_backward(m, res, torch.as_tensor(g).cuda(), mask).cpu().numpy()
    hit = np.zeros(ncp, bool)
    t, w = b.knots[int(b.knot_off[0]):], []
    for a in range(3):
        s = int(_spans(t, ncp[a], res[a])[at[a]])
        w.append(slice(s - p, s + 1))
        t = t[ncp[a] + p + 1:]
    hit[tuple(w)] = True
    h = hit.ravel()
    inside = np.zeros(got.size, bool)
    ref = oracle.decode_adjoint(oracle_blocks(b), res, np.where(np.isfinite(g), g, 0).astype(np.float64), mask)
    for k in range(nblocks):
        o, n = int(b.ctrl_off[k]), int(np.prod(ncp))
        inside[o:o + n] = True
        want = ref[o:o + n].copy()
        for v in (got[o:o + n].copy(), bad[o:o + n].copy()):
            if k == 0:  # away from the window of the value that is not finite
                v[h] = want[h]
            check_normwise(v[None, None], want[None, None], what=f"block {k}")
    o, n = int(b.ctrl_off[0]), int(np.prod(ncp))
    assert np.array_equal(np.isfinite(bad[o:o + n]), ~h)
    assert np.all(got[~inside] == 777.0)
