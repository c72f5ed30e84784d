"""The TV term for mu and lam at the ends of float32: mu + 8 lam or its reciprocal
overflows, or is a subnormal number, though the U update is a ratio of the two and
well defined.  Against the FP64 oracle, within 1e-5 of the field's largest value:
six iterations of about ten float32 roundings (6e-8 each) of values up to it, some
4e-6 (the term itself vanishes for a large lam, so there is no relative bound)."""
import numpy as np
import pytest

import oracle.tv_oracle as T
from paper_2506_20513_amd import tv

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mu,lam", [(2e-40, 3e-40), (1e-39, 1e-39), (8e-39, 2e-39), (1e-30, 1e-30),
                                    (1e30, 2e30), (1.2e38, 1e37), (1e38, 1e38), (3e38, 1e30)])
def test_mu_and_lam_at_the_ends_of_float32(mu, lam):
    import torch
    mu, lam, iters = float(np.float32(mu)), float(np.float32(lam)), 6
    rng = np.random.default_rng(17)
    X = (5 * (1 + 0.2 * rng.standard_normal((70, 90)))).astype(np.float32)
    X[30:, 50:] *= 1.6
    g = torch.zeros(1, 70, 90, device="cuda")
    tv.TV(1, 70, 90, mu, lam, 1.0, iters)(torch.from_numpy(X[None]).cuda(), g)
    got = g.cpu().numpy()[0].astype(np.float64)
    ref = T.tv_gradient(X.astype(np.float64), mu, lam, iters, 1.0)
    err = np.abs(got - ref).max() / np.abs(X).max()
    print(mu, lam, err, flush=True)
    assert err <= 1e-5
