"""The row-marching weight gradient (csrc/fwi_nn.hip, k_wgrad_rows) at the sizes
where it can go wrong: images around the 128 pixels it starts at, widths around
its 8-pixel groups and its strips (256 and 128 pixels for eight and four waves),
rows that do not divide a step, one record and many, blocks that cross strips and
images, several channel tiles, a scratch only 4-byte aligned.  Reference and
tolerance are those of the weight gradient's other test: plain float64,
1e-5 sum |terms|."""
import pytest

from tests.test_gpu_nn import _bf, _conv_ref, _dev
from paper_2506_20513_amd import nn

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,H,W,Ci,Co,nsplit", [
    # just below the line (flattened form) and on it
    (2, 1, 127, 32, 32, 3), (2, 1, 128, 32, 32, 3), (1, 128, 1, 32, 64, 9), (3, 13, 10, 64, 32, 2),
    # eight waves: strips of up to 256 pixels, several rows per step
    (2, 9, 255, 32, 32, 64), (1, 5, 257, 64, 64, 100), (2, 17, 40, 32, 96, 7),
    (3, 33, 7, 32, 32, 1000), (2, 11, 136, 96, 32, 5), (1, 31, 83, 64, 32, 1000),
    # four waves: more than 8 steps per block
    (2, 20, 200, 32, 32, 1), (1, 13, 1000, 32, 64, 3), (3, 77, 65, 64, 32, 2),
    (1, 150, 129, 32, 32, 4), (5, 160, 9, 32, 32, 1)])
def test_rows_weight_gradient(N, H, W, Ci, Co, nsplit):
    import torch
    x, g = _bf((N, H, W, Ci), 7), _bf((N, H, W, Co), 9)
    w = _bf((Co, 3, 3, Ci), 8, 0.1).double().requires_grad_(True)
    (_conv_ref(x, w, None, False)[0] * g.double()).sum().backward()
    wa = w.detach().abs().requires_grad_(True)
    (_conv_ref(x.abs(), wa, None, False)[0] * g.double().abs()).sum().backward()
    n = nn.wgrad_workspace(Ci, Co, nsplit) // 4
    for shift in (0, 1):                 # 1: the scratch 4 bytes past a 16-byte boundary
        ws = torch.full((n + 4,), float("nan"), device="cuda")
        dw = torch.full((Co * 9 * Ci,), float("nan"), device="cuda")
        db = torch.full((Co,), float("nan"), device="cuda")
        nn.wgrad(_dev(x), _dev(g), dw, db, N, H, W, Ci, Co, nsplit, ws[shift:shift + n])
        torch.cuda.synchronize()
        err = (dw.double().cpu().view(Co, 3, 3, Ci) - w.grad).abs()
        worst = float((err / (1e-5 * wa.grad + 1e-30)).max())
        print(f"shift {shift}: max err / bound", worst, flush=True)
        assert worst <= 1.0
        dbr = g.double().sum(dim=(0, 1, 2))
        assert float((db.double().cpu() - dbr).abs().max()) <= \
            1e-5 * float(g.double().abs().sum(dim=(0, 1, 2)).max())
        rest = torch.cat([ws[:shift], ws[shift + n:]])
        assert bool(torch.isnan(rest).all()), "written outside the scratch"
