"""Small problems run on the tile kernels (tiles of 64 columns and 32 or 64
rows, 8 of them halo on every side: 48 columns and 16 or 48 rows owned).
Their results against the FP64 oracle at the sizes where a tile can go wrong:
totals one below, at and one above whole tiles, grids smaller than a tile,
no CPML and CPML in the columns and rows next to a tile's edge, partial
passes, receivers on every kind of row, several in one cell, on the source
and in the halo of the neighbouring tile, the source in a tile's corner.

Tolerances are those of every parity test (relative L2 1e-4 on traces, 1e-3 on
gradients and the source adjoint): both sides follow the same recurrence, FP32
against FP64, over a few hundred steps."""
import numpy as np
import pytest

import oracle
from paper_2506_20513_amd import fwi
from paper_2506_20513_amd import inputs as I
from tests.gpu_util import Run, np_, rel_l2

pytestmark = pytest.mark.gpu

TR_TOL = 1e-4
GR_TOL = 1e-3

# (NX, NY, npml, nt, shots): NX around multiples of 48, NY around multiples of
# 16 and 48, nt around multiples of the 8 levels of a pass; the last ones have
# more than 192 tall tiles and so run on those
CASES = [(47, 15, 0, 90, 1), (48, 16, 2, 97, 2), (49, 17, 3, 95, 1), (96, 47, 8, 136, 2),
         (97, 49, 10, 121, 2), (143, 33, 7, 104, 1), (145, 97, 20, 150, 1), (11, 9, 0, 41, 1),
         (100, 50, 5, 61, 70), (97, 97, 9, 83, 25)]


def _geometry(NX, NY, npml, S, rng):
    lo, xi, yi = max(1, npml), min(NX - 2, NX - 1 - npml), min(NY - 2, NY - 1 - npml)
    src = np.stack([rng.integers(lo, xi + 1, S), rng.integers(lo, yi + 1, S)], 1).astype(np.int32)
    # the first source at the corner cell of an owned tile part, if it is inside
    src[0] = min(max(lo, 47), xi), min(max(lo, 15), yi)
    rec = np.stack([rng.integers(lo, xi + 1, (S, 24)), rng.integers(lo, yi + 1, (S, 24))], 2)
    rec[:, 0] = src                       # on the source
    rec[:, 3] = rec[:, 1]                 # three receivers in one cell
    rec[:, 7] = rec[:, 1]
    rec[:, 8, 0], rec[:, 9, 0] = lo, xi   # the first and last columns
    rec[:, 10, 1], rec[:, 11, 1] = lo, yi
    for k, i in enumerate((47, 48, 56)):  # around the first tile's right side, one row
        rec[:, 12 + k] = min(max(lo, i), xi), lo
    return src, np.ascontiguousarray(rec, dtype=np.int32)


@pytest.mark.parametrize("NX,NY,npml,nt,S", CASES)
def test_tile_edges_against_the_oracle(NX, NY, npml, nt, S):
    import torch
    rng = np.random.default_rng(NX * 1000 + NY)
    dx, dy = 0.02, 0.0146
    dt = 0.9 / (I.C0 * np.sqrt(1 / dx ** 2 + 1 / dy ** 2))
    eps = rng.uniform(1.0, 9.0, (NY, NX)).astype(np.float32)
    sig = rng.uniform(0.0, 0.02, (NY, NX)).astype(np.float32)
    sig[NY // 2, NX // 3] = 1e3           # a conductor cell
    src, rec = _geometry(NX, NY, npml, S, rng)
    w = np.stack([I.ricker(nt, dt, 400e6, amp=a) for a in rng.uniform(0.5, 2, S)])
    kw = dict(cpml_kappa_max=1.5, cpml_alpha_max=np.pi * 400e6 * I.EPS0)
    grid = fwi.make_grid(NX - 2 * npml, NY - 2 * npml, npml, nt, dx, dy, dt, **kw)
    P = oracle.Problem(eps, sig, npml, dx, dy, dt, **kw)
    obs, _ = P.forward(src, rec, w, nt)
    obs = (0.7 * obs).astype(np.float32)
    J, oge, ogs, otr = P.gradient(src, rec, w, obs, nt)
    r = Run(grid, src, rec, w, eps, sig)
    mis, ge, gs, tr = r.gradient(obs)
    errs = dict(traces=rel_l2(np_(tr), otr), misfit=abs(float(mis.item()) - J) / J,
                ge=rel_l2(np_(ge), oge), gs=rel_l2(np_(gs), ogs))
    print((NX, NY, npml, nt, S), errs, flush=True)
    assert errs["traces"] <= TR_TOL and errs["misfit"] <= 1e-4
    assert errs["ge"] <= GR_TOL and errs["gs"] <= GR_TOL
    # the stored-history and the checkpointed adjoint: the fused call's bits
    for mode in (fwi.FWI_SAVE_HISTORY, fwi.FWI_SAVE_CHECKPOINT):
        t2, ws = r.forward(mode)
        g2, s2, _ = r.adjoint(t2 - torch.from_numpy(obs).cuda(), mode, ws, want_src_adjoint=True)
        assert torch.equal(t2, tr) and torch.equal(g2, ge) and torch.equal(s2, gs), mode
