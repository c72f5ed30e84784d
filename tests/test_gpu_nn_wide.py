"""The per-pixel kernels of the network's input and loss at channel counts far past
the network's own: around the line where a thread per value takes over, and where
the index of a pixel's last 16-byte piece outgrows the kernels' short division (the
smallest such count is 65776 for 64 pixels; see
test_short_division_of_wide_pixels).  Every value is one float32 operation rounded to
bfloat16, so results are exact."""
import pytest

from paper_2506_20513_amd import nn


def test_short_division_of_wide_pixels():
    """The piece index of 64 pixels of C channels, e < 8 C, over C / 8: exact by the
    high word of e m for every C that takes those kernels (up to 2048)."""
    def div(n, d):
        return n if d == 1 else (n * ((2 ** 32 - 1) // d + 1)) >> 32

    assert div(64 * 8222 - 1, 8222) == 64            # not 63: 65776 channels
    for nv in range(1, 2048 // 8 + 1):
        for px in range(64):
            assert div(px * nv, nv) == px and div(px * nv + nv - 1, nv) == px


@pytest.mark.gpu
@pytest.mark.parametrize("P,C", [(64, 65776), (3, 2056), (65, 2048), (5, 65536), (2, 66008)])
def test_pack4_of_wide_pixels(P, C):
    import torch
    planes, sc = torch.randn(1, 4, 1, P, device="cuda"), torch.rand(1, 4, device="cuda") + 0.5
    x = torch.full((P * C + 8,), 7.0, dtype=torch.bfloat16, device="cuda")
    nn.pack4(planes, sc, x[:P * C], 1, 1, P, C)
    ref = torch.zeros(P, C, device="cuda")
    ref[:, :4] = (planes[0, :, 0] * sc[0, :, None]).t()
    assert torch.equal(x[:P * C].view(P, C), ref.bfloat16())
    assert bool((x[P * C:] == 7).all())


@pytest.mark.gpu
@pytest.mark.parametrize("P,C,cout", [(64, 65776, 2), (65, 128, 2), (63, 136, 2), (70, 128, 3),
                                      (129, 128, 1), (524288 + 3, 32, 2), (131, 32, 8)])
def test_loss_of_wide_pixels(P, C, cout):
    """Each route of the loss: its gradient is one rounding of a float64 value to
    bfloat16 through float32, the loss a float64 sum in another order."""
    import torch
    g = torch.Generator().manual_seed(P)
    y, tgt = torch.randn(P, C, generator=g).bfloat16().cuda(), torch.randn(P, cout, generator=g).cuda()
    dy = torch.full((P * C + 8,), 7.0, dtype=torch.bfloat16, device="cuda")
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    part = torch.empty(nn.FWI_NN_MSE_BLOCKS, dtype=torch.float64, device="cuda")
    nn.mse(y.view(-1), tgt, dy[:P * C], loss, part, P, C, cout)
    d = y[:, :cout].double() - tgt.double()
    assert abs(float(loss) - float((d * d).mean())) <= 1e-12 * float((d * d).mean())
    got = dy[:P * C].view(P, C)
    grad = 2.0 / (P * cout) * d
    assert bool(((got[:, :cout].double() - grad).abs() <= 2.0 ** -8 * grad.abs()).all())
    assert not bool(got[:, cout:].any()) and bool((dy[P * C:] == 7).all())
