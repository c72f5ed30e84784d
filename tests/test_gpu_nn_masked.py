"""Kernels that apply the adjoint of a ReLU as they store: the same bits as the
plain kernel followed by relu_bwd, over every kernel the convolution chooses from
(row-marching in both orders, LDS tiles of both sizes, the smallest layers'), masks
off the vector alignment, and masks holding zeros of both signs, NaN and infinity."""
import pytest

from tests.test_gpu_nn import _bf, _dev
from paper_2506_20513_amd import nn

pytestmark = pytest.mark.gpu


def _mask(n, shift):
    import torch
    m = torch.randn(n, generator=torch.Generator().manual_seed(4)).bfloat16()
    for i, v in enumerate((0.0, -0.0, float("nan"), float("inf"), -float("inf"), 1e-40)):
        m[i::17 + i] = v
    buf = torch.zeros(n + 8, dtype=torch.bfloat16, device="cuda")
    buf[shift:shift + n] = m.cuda()
    return buf[shift:shift + n]


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("N,H,W,Ci,Co", [
    (1, 9, 33, 32, 64), (2, 130, 128, 32, 32), (1, 5, 33, 64, 128), (1, 300, 129, 64, 64),
    (1, 3, 40, 128, 32), (4, 67, 128, 128, 128),       # rows
    (1, 7, 33, 96, 32), (2, 90, 100, 96, 64), (2, 190, 200, 256, 64)])   # small, LDS 64, 128
def test_masked_convolution(N, H, W, Ci, Co, shift):
    import torch
    x, w = _dev(_bf((N, H, W, Ci), 1)).view(-1), _dev(_bf((Co, 3, 3, Ci), 2, 0.1)).view(-1)
    n = N * H * W * Co
    mask, new = _mask(n, shift), lambda: torch.full((n,), 7.0, dtype=torch.bfloat16, device="cuda")
    plain, ref, y = new(), new(), new()
    nn.conv3x3(x, w, None, plain, N, H, W, Ci, Co, False)
    nn.relu_bwd(mask, plain, ref, n)
    nn.conv3x3_masked(x, w, mask, y, N, H, W, Ci, Co)
    torch.cuda.synchronize()
    # (one row kernel sums in the order of the kernel it stands in for: with a
    # mask off its alignment that kernel runs, in the same order)
    assert torch.equal(y, ref)


@pytest.mark.parametrize("shift", [0, 1])
@pytest.mark.parametrize("C", [32, 4])
def test_masked_adjoints(C, shift):
    import torch
    N, H, W = 2, 6, 10
    n, new = N * H * W * C, lambda k: torch.full((k,), 7.0, dtype=torch.bfloat16, device="cuda")
    mask = _mask(n, shift)
    q, s, g = (_dev(_bf(sh, i)).view(-1) for i, sh in
               enumerate(((N, H // 2, W // 2, C), (N, H, W, C), (N, 2 * H, 2 * W, C))))
    for skip in (None, s):
        plain, ref, y = new(n), new(n), new(n)
        nn.pool2_bwd_add(q, skip, plain, N, H, W, C)
        nn.relu_bwd(mask, plain, ref, n)
        nn.pool2_bwd_masked(q, skip, mask, y, N, H, W, C)
        torch.cuda.synchronize()
        assert torch.equal(y, ref)
    plain, ref, y = new(n), new(n), new(n)
    nn.up2_bwd(g, plain, N, H, W, C)
    nn.relu_bwd(mask, plain, ref, n)
    nn.up2_bwd_masked(g, mask, y, N, H, W, C)
    torch.cuda.synchronize()
    assert torch.equal(y, ref)
