"""Convolutions on the row-marching kernel at its edges, by the rule that picks it
(the shapes of tests/test_nn_route_host.py: widths around its 16-pixel tiles and its
strips, one row, one column, bands that do not divide the height, both orders of the
reduction), and shapes of a few rows or columns that it leaves to the other kernels.
Each against the same call with an output that the row kernel cannot take (2 bytes
past an 8-byte boundary): the same bits, as every sum runs in the same order.  The
other kernels are held to a float64 reference in their own tests."""
import pytest

from paper_2506_20513_amd import nn
from tests.test_nn_route_host import EDGES

pytestmark = pytest.mark.gpu

OTHER = [(2048, 1, 16, 64, 32), (4096, 2, 2, 64, 32), (512, 2, 2, 128, 256), (11, 60, 19, 128, 128),
         (16, 100, 65, 32, 32), (2048, 1, 32, 32, 64)]


@pytest.mark.parametrize("N,H,W,Ci,Co", EDGES + OTHER)
def test_both_routes_give_the_same_bits(N, H, W, Ci, Co):
    import torch
    g = torch.Generator(device="cuda").manual_seed(N * 1000 + W)
    x = torch.randn(N * H * W * Ci, generator=g, device="cuda").bfloat16()
    w = (torch.randn(Co * 9 * Ci, generator=g, device="cuda") * 0.05).bfloat16()
    b = torch.randn(Co, generator=g, device="cuda")
    n = N * H * W * Co
    mask = torch.randn(n, generator=g, device="cuda").bfloat16()
    y = torch.full((2, n + 8), float("nan"), dtype=torch.bfloat16, device="cuda").view(-1)
    for masked in (False, True):
        out = []
        for shift in (0, 1):
            y.fill_(float("nan"))
            o = y[shift:shift + n]
            if masked:
                nn.conv3x3_masked(x, w, mask, o, N, H, W, Ci, Co)
            else:
                nn.conv3x3(x, w, b, o, N, H, W, Ci, Co, True)
            assert bool(torch.isnan(y[:shift]).all()) and bool(torch.isnan(y[shift + n:]).all())
            out.append(o.clone())
        assert bool(torch.isfinite(out[0]).all()) and bool(out[0].any())
        assert torch.equal(out[0], out[1]), masked
