"""The TV iteration's tiles (csrc/fwi_tv.hip): each of the three tile shapes,
chosen by the number of cells, at field sides around whole tiles, sides
smaller than a tile (the halo wraps round several times) and iteration counts
around the launches' 10 and 5, against the FP64 oracle.

Tolerance: the gradient tolerance 1e-3 of the other TV tests on the added
term; float32 rounding of the iterates (6e-8 per operation, a contraction)
against a term of 1e-2 to 1e-1 of the model leaves about 1e-5."""
import numpy as np
import pytest

import oracle.tv_oracle as T
from paper_2506_20513_amd import tv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nf,ny,nx,iters", [
    (1, 12, 44, 10), (2, 13, 45, 11), (1, 11, 43, 21), (1, 2, 2, 25), (3, 3, 200, 9),
    (1, 361, 364, 10), (2, 421, 397, 12), (1, 400, 600, 3),
    (1, 1021, 541, 5), (1, 990, 702, 11), (4, 361, 433, 6)])
def test_tile_shapes_against_the_oracle(nf, ny, nx, iters):
    import torch
    rng = np.random.default_rng(ny * 3000 + nx)
    X = (rng.uniform(0.5, 9.0, (nf, 1, 1)) * (1 + 0.2 * rng.standard_normal((nf, ny, nx))))
    X[:, ny // 3:, nx // 2:] *= 1.6
    X = X.astype(np.float32)
    mu, lam, w = [6.0, 4.0, 1.0, 9.0][:nf], [2.0, 3.0, 0.7, 5.0][:nf], [0.5, 2.0, 1.0, 0.1][:nf]
    g0 = rng.standard_normal((nf, ny, nx)).astype(np.float32) * 0.1
    gd = torch.from_numpy(g0).cuda()
    tv.TV(nf, ny, nx, mu, lam, w, iters)(torch.from_numpy(X).cuda(), gd)
    got = gd.cpu().numpy().astype(np.float64) - g0
    for f in range(nf):
        ref = T.tv_gradient(X[f].astype(np.float64), mu[f], lam[f], iters, w[f])
        e = np.linalg.norm(got[f] - ref) / np.linalg.norm(ref)
        print(f"field {f} {ny}x{nx} iters {iters}: rel L2 {e:.2e}", flush=True)
        assert e <= 1e-3
