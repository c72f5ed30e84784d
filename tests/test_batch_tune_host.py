"""What the batch plan's autotuner times, on the CPU: kernels do not run, and the time
between two events is the most levels that an entry of the launch between them advances,
in milliseconds.  Every launch that the autotuner times is then as good as any other per
level, so each candidate costs three per time step (sweep, re-forward and adjoint) -
unless a launch of a few levels is timed and charged as a full pass."""
import ctypes

import numpy as np
import pytest

from paper_2506_20513_amd import fwi
from paper_2506_20513_amd import inputs as I
from tests.host_routes import build

CODE = """
#include <hip/hip_runtime.h>
#include "fwi_internal.h"
#include <algorithm>
static float g_ms = 0.f;
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { *ms = g_ms; return hipSuccess; }
namespace fwi {
hipError_t launch_fwd_table(const FwdStreamArgs *tab, const unsigned *, int nm, unsigned, int, bool,
                            int, hipStream_t) {
    g_ms = 0.f;
    for (int m = 0; m < nm; ++m) g_ms = std::max(g_ms, (float)tab[m].nlev);
    return hipSuccess;
}
hipError_t launch_adj_table(const AdjStreamArgs *tab, const unsigned *, int nm, unsigned, int, bool,
                            hipStream_t) {
    g_ms = 0.f;
    for (int m = 0; m < nm; ++m) g_ms = std::max(g_ms, (float)tab[m].nlev);
    return hipSuccess;
}
}  // namespace fwi
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("tune")
    return build(d, "tune", CODE, ["hipEventElapsedTime=stub_hipEventElapsedTime",
                                   "launch_fwd_table=stub_launch_fwd_table",
                                   "launch_adj_table=stub_launch_adj_table"])


def _buf(n, held):
    a = np.zeros(int(n) + 256, np.uint8)
    held.append(a)
    return a.ctypes.data + (-a.ctypes.data) % 256


# equal windows of one step over whole passes of 8, and of 5; uneven ones; less than a pass
@pytest.mark.parametrize("nts", [(57, 57, 57), (61, 61), (57, 41, 90), (64, 64), (5, 5), (12, 9)])
def test_every_candidate_costs_three_per_step(lib, nts):
    held, probs = [], (fwi.fwi_batch_problem * len(nts))()
    keep = []
    for k, nt in enumerate(nts):
        cfg = I.config_tiny().with_(nt=nt)
        src, rec = I.geometry(cfg)
        S, R = src.shape[0], rec.shape[1]
        geom = fwi.Geometry(src, rec, _buf(S * nt * 4, held))
        plane = cfg.NX * cfg.NY * 4
        p = fwi.BatchProblem(fwi.grid_from_config(cfg), geom, _buf(plane, held), _buf(plane, held),
                             _buf(S * nt * R * 4, held), _buf(8, held), _buf(plane, held),
                             _buf(plane, held))
        keep.append(p)
        probs[k] = p.c
    need = ctypes.c_size_t()
    assert lib.fwi_batch_workspace_bytes(len(nts), probs, ctypes.byref(need)) == 0
    ws, plan, info = _buf(need.value, held), ctypes.c_void_p(), fwi.fwi_batch_info()
    assert lib.fwi_batch_plan_create(len(nts), probs, ctypes.c_void_p(ws), need,
                                     fwi.FWI_TUNE_BANDS | fwi.FWI_TUNE_DEPTH, None,
                                     ctypes.byref(plan)) == 0
    assert lib.fwi_batch_plan_info(plan, ctypes.byref(info)) == 0
    cost = list(info.tune_ms)[:info.ntune]
    lib.fwi_batch_plan_destroy(plan)
    assert len(cost) >= 10 and np.allclose(cost, 3.0), cost
