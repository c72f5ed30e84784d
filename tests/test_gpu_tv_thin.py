"""The TV iteration's tiles for large fields of a few rows (12 rows, 2 of them
owned) and for a single iteration (a halo of one cell), at the edges of their rules
and of their tiles, against the FP64 oracle; tolerance as in the other TV tests."""
import numpy as np
import pytest

import oracle.tv_oracle as T
from paper_2506_20513_amd import tv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nf,ny,nx,iters", [(1, 2, 65537, 7), (2, 3, 30001, 12), (1, 6, 22000, 5),
                                            (1, 7, 20003, 11), (1, 363, 363, 1), (2, 1025, 127, 1),
                                            (1, 2, 70000, 1)])
def test_thin_fields_and_single_iterations(nf, ny, nx, iters):
    import torch
    rng = np.random.default_rng(ny * 3000 + nx)
    X = (6.0 * (1 + 0.2 * rng.standard_normal((nf, ny, nx))))
    X[:, ny // 3:, nx // 2:] *= 1.6
    X = X.astype(np.float32)
    g = torch.zeros(nf, ny, nx, device="cuda")
    tv.TV(nf, ny, nx, 6.0, 2.0, 0.5, iters)(torch.from_numpy(X).cuda(), g)
    got = g.cpu().numpy().astype(np.float64)
    for f in range(nf):
        ref = T.tv_gradient(X[f].astype(np.float64), 6.0, 2.0, iters, 0.5)
        e = np.linalg.norm(got[f] - ref) / np.linalg.norm(ref)
        print(f"field {f} {ny}x{nx} iters {iters}: rel L2 {e:.2e}", flush=True)
        assert e <= 1e-3
