"""The row-marching convolution (csrc/fwi_nn.hip, k_conv3x3_rows) at the sizes
where it can go wrong: widths around its 16-pixel tiles and its strips (128, 64
and 32 pixels for 32, 64 and 128 input channels), single rows and columns, bands
that do not divide the height, every split of the channels over its waves, both
orders of the reduction (large and small layers) and an output it cannot take
(not 8-byte aligned: another kernel).  Reference and tolerance are those of the
convolution's other tests: plain float64, 2^-8 |ref| + 1e-5 sum |terms|."""
import pytest

from tests.test_gpu_nn import _bf, _close_bf16, _conv_ref, _dev
from paper_2506_20513_amd import nn

pytestmark = pytest.mark.gpu

CASES = [
    # small layers, reduction over (ky, kx, ci)
    (1, 1, 1, 32, 32, 0), (2, 1, 15, 64, 32, 1), (1, 2, 16, 128, 64, 1), (3, 7, 17, 64, 128, 0),
    (1, 5, 33, 128, 32, 1), (2, 9, 65, 64, 64, 1), (1, 3, 129, 32, 96, 0), (1, 40, 1, 32, 64, 1),
    (1, 11, 31, 128, 192, 0),
    # layers the LDS tiling would fill the chip with, reduction over (ky, ci / 32, kx)
    (2, 130, 128, 32, 32, 1), (1, 131, 257, 32, 64, 0), (1, 300, 129, 64, 64, 1),
    (3, 101, 128, 64, 32, 0), (1, 257, 144, 64, 128, 1), (4, 67, 128, 128, 128, 0),
    (2, 190, 96, 128, 32, 1)]


@pytest.mark.parametrize("N,H,W,Ci,Co,relu", CASES)
def test_rows_convolution(N, H, W, Ci, Co, relu):
    import torch
    x, w = _bf((N, H, W, Ci), 1), _bf((Co, 3, 3, Ci), 2, 0.1)
    b = torch.randn(Co, dtype=torch.float64, generator=torch.Generator().manual_seed(3))
    b = b.float().double()
    ref, aref = _conv_ref(x, w, b, relu)
    n = N * H * W * Co
    for shift in (0, 1):                 # 1: y two bytes past an 8-byte boundary
        y = torch.full((n + 8,), float("nan"), dtype=torch.bfloat16, device="cuda")
        nn.conv3x3(_dev(x).view(-1), _dev(w).view(-1), _dev(b.float()), y[shift:shift + n], N, H, W,
                   Ci, Co, relu)
        torch.cuda.synchronize()
        _close_bf16(y[shift:shift + n].view(N, H, W, Co), ref, aref + b.abs(), f"shift {shift}")
        rest = torch.cat([y[:shift], y[shift + n:]])
        assert bool(torch.isnan(rest).all()), "written outside y"
