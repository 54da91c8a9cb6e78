"""The adjoint of more micro-models than one launch can hold threads for."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mask", [1, 2])
def test_adjoint_of_more_than_two_to_the_23_blocks(mask):
    import paper_2409_00184_amd as fa
    # trilinear micro-models of 2 x 2 x 2 control points at the grid points
    # themselves: the value adjoint is the cotangent, that of d/dx its
    # difference along x; the models share one knot vector
    n = (1 << 23) + 3
    desc = fa.host_descriptors(np.full((n, 3), 2, np.int32), np.ones((n, 3), np.int32),
                               np.zeros(n, np.int64), 8 * np.arange(n, dtype=np.int64))
    knots = torch.tensor([0.0, 0.0, 1.0, 1.0] * 3, device="cuda")
    d = torch.from_numpy(desc.view(np.uint8)).cuda()
    g = torch.randint(-8, 9, (n, 2, 2, 2), device="cuda", generator=torch.Generator("cuda").manual_seed(3))
    g = g.float()
    G = torch.full((n, 2, 2, 2), 777.0, device="cuda")
    st = fa.lib.fa_decode_backward(d.data_ptr(), n, knots.data_ptr(), fa._i32x3((2, 2, 2)), mask,
                                   g.data_ptr(), G.data_ptr(),
                                   torch.cuda.current_stream().cuda_stream)
    assert st == 0
    want = g if mask == 1 else torch.stack((-(g[:, 0] + g[:, 1]), g[:, 0] + g[:, 1]), 1)
    assert torch.equal(G, want)
