"""The network's element-wise kernels at sizes around their waves: pixel counts
that do not fill a wave or a block, channel counts of one to five 8-channel pieces
(the divisors of the index arithmetic), one-pixel coarse images, and the transposed
weights of channel counts off the 32 x 32 tiles.  References are the same float32
operations in torch, so every result is exact; the loss, a double sum in another
order, within 1e-13 of a float64 one, and its gradient, one rounding of a float64
value, within the rounding of bfloat16."""
import pytest

from tests.test_gpu_nn import _bf, _dev
from paper_2506_20513_amd import nn

pytestmark = pytest.mark.gpu


def _new(n, torch):
    return torch.full((n,), 7.0, dtype=torch.bfloat16, device="cuda")


@pytest.mark.parametrize("N,H,W,C", [(1, 2, 2, 8), (3, 6, 10, 24), (2, 14, 2, 40), (1, 2, 66, 32),
                                     (5, 34, 30, 256), (7, 128, 130, 16)])
def test_coarse_grid_kernels(N, H, W, C):
    import torch
    x, q, s = (_dev(_bf(sh, i)) for i, sh in
               enumerate(((N, H, W, C), (N, H // 2, W // 2, C), (N, H, W, C))))
    X = x.float().view(N, H // 2, 2, W // 2, 2, C)
    a, b, d, e = X[:, :, 0, :, 0], X[:, :, 0, :, 1], X[:, :, 1, :, 0], X[:, :, 1, :, 1]
    total = ((a + b) + d) + e
    up = q.float().repeat_interleave(2, 1).repeat_interleave(2, 2)
    nlo, nhi = q.numel(), x.numel()
    y = _new(nlo, torch)
    nn.pool2(x.view(-1), y, N, H, W, C)
    assert torch.equal(y, (0.25 * total).bfloat16().view(-1))
    nn.up2_bwd(x.view(-1), y, N, H // 2, W // 2, C)
    assert torch.equal(y, total.bfloat16().view(-1))
    z = _new(nhi, torch)
    nn.up2_add(q.view(-1), s.view(-1), z, N, H, W, C)
    assert torch.equal(z, (up + s.float()).bfloat16().view(-1))
    nn.up2_add(q.view(-1), None, z, N, H, W, C)
    assert torch.equal(z, up.bfloat16().view(-1))
    nn.pool2_bwd_add(q.view(-1), s.view(-1), z, N, H, W, C)
    assert torch.equal(z, (0.25 * up + s.float()).bfloat16().view(-1))


@pytest.mark.parametrize("N,H,W,C", [(1, 1, 1, 8), (3, 7, 13, 32), (2, 5, 64, 24), (4, 33, 31, 40)])
def test_pixel_kernels(N, H, W, C):
    import torch
    g = torch.Generator().manual_seed(5)
    P = N * H * W
    planes, sc = torch.randn(N, 4, H, W, generator=g).cuda(), torch.rand(N, 4, generator=g).cuda()
    x = _new(P * C + 8, torch)
    nn.pack4(planes, sc, x[:P * C], N, H, W, C)
    ref = torch.zeros(P, C, device="cuda")
    ref[:, :4] = (planes * sc[:, :, None, None]).permute(0, 2, 3, 1).reshape(P, 4)
    assert torch.equal(x[:P * C].view(P, C), ref.bfloat16())
    assert bool((x[P * C:] == 7).all())
    y, so = _dev(_bf((P, C), 6)), torch.rand(N, 2, generator=g).cuda()
    out = torch.empty(N * 2 * H * W, device="cuda")
    nn.unpack2(y.view(-1), so, out, N, H, W, C)
    r = (y[:, :2].float().view(N, H * W, 2) * so[:, None, :]).permute(0, 2, 1)
    assert torch.equal(out.view(N, 2, -1), r)
    for cout in {1, 2, min(C, 8), C}:
        tgt = torch.randn(P, cout, generator=g).cuda()
        dy = _new(P * C + 8, torch)
        loss = torch.zeros(1, dtype=torch.float64, device="cuda")
        part = torch.empty(nn.FWI_NN_MSE_BLOCKS, dtype=torch.float64, device="cuda")
        nn.mse(y.view(-1), tgt, dy[:P * C], loss, part, P, C, cout)
        d = y[:, :cout].double() - tgt.double()
        want = float((d * d).mean())
        assert abs(float(loss) - want) <= 1e-13 * want
        grad = torch.zeros(P, C, dtype=torch.float64, device="cuda")
        grad[:, :cout] = 2.0 / (P * cout) * d
        err = (dy[:P * C].view(P, C).double() - grad).abs()
        assert bool((err <= 2.0 ** -8 * grad.abs()).all())
        assert bool((dy[P * C:] == 7).all())


def test_flipped_layers_off_the_tiles():
    import torch
    cis, cos = [32, 1, 33, 7, 96], [64, 40, 31, 1, 32]
    offs, at = [], 5
    for a, b in zip(cis, cos):
        offs.append(at)
        at += 9 * a * b + 3
    w = _dev(_bf((at,), 1))
    wf, ref = _new(at, torch), _new(at, torch)
    nn.flip_layers(w, wf, offs, cis, cos)
    for o, a, b in zip(offs, cis, cos):
        v = w[o:o + 9 * a * b].view(b, 9, a)
        ref[o:o + 9 * a * b] = v.flip(1).permute(2, 1, 0).reshape(-1)
    torch.cuda.synchronize()
    assert torch.equal(wf, ref)
