"""fwi_tv_gradient with grad the same array as X: the tiles of the last launch read
X over their halos, so no tile may overwrite it before its neighbours have.  The
same bits as the call with a copy, for every tile shape, one iteration, and
iteration counts at and around a launch's; a field of zeros stays as it is.

The sizes give many more tiles than the chip holds at once, or a single launch of
iterations, so that a tile that wrote early would be seen by later ones."""
import pytest

from paper_2506_20513_amd import tv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nf,ny,nx,iters", [(1, 64, 96, 1), (2, 128, 128, 10), (2, 128, 128, 13),
                                            (2, 300, 500, 10), (1, 700, 701, 2),
                                            (2, 1500, 1600, 5), (2, 1500, 1600, 6)])
def test_in_place_is_the_call_on_a_copy(nf, ny, nx, iters):
    import torch
    g = torch.Generator(device="cuda").manual_seed(ny + iters)
    X = torch.rand(nf, ny, nx, generator=g, device="cuda") * 9 + 1
    X[:, ny // 3:, nx // 2:] *= 1.6
    if nf > 1:
        X[1] = 0
    op = tv.TV(nf, ny, nx, [6.0, 4.0][:nf], [2.0, 3.0][:nf], [-1.0, 0.5][:nf], iters)
    want = X.clone()
    op(X, want)
    op(X, X)
    torch.cuda.synchronize()
    assert torch.equal(X, want)
    assert nf == 1 or not bool(X[1].any())
