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
