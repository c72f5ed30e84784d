"""The line between the tile and the streaming kernels (use_tiles in csrc/fwi_host.cpp),
and the batches that stay on streams: calls on either side of it that were measured,
among them grids that fit the tiles badly, with many shots, and traces-only calls,
which a line drawn from one kind of call had sent to the slower kernels."""
import ctypes

import pytest

from tests.host_routes import build

CODE = """
#include "fwi_host.h"
using namespace fwi;
using namespace fwi::host;
extern "C" int route(int NX, int NY, int S, int mode, int *o) {
    Dims d{};
    d.NX = NX; d.NY = NY; d.npml = 10; d.nt = 96; d.S = S; d.R = 4;
    d.pitch = (NX + 63) / 64 * 64; d.W = d.Hs = 21;
    d.plane = (size_t)NY * d.pitch; d.xs = (size_t)NY * d.W; d.ys = (size_t)d.Hs * d.pitch;
    Layout L;
    const int rc = make_layout(d, mode, L);
    o[0] = L.tile; o[1] = L.pass; o[2] = L.depth;
    return rc;
}
"""
NONE, CHECKPOINT, HISTORY, GRADIENT = 0, 1, 2, -1


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    lib = build(tmp_path_factory.mktemp("routes"), "routes", CODE)

    def f(NX, NY, S, mode):
        o = (ctypes.c_int * 3)()
        assert lib.route(NX, NY, S, mode, o) == 0
        assert o[1] == (8 if o[0] else o[2])
        return o[0]
    return f


# (NX, NY, shots): the kernels of a gradient and of a traces-only call
@pytest.mark.parametrize("NX,NY,S,gradient,traces", [
    (148, 148, 1, 32, 32), (240, 140, 4, 32, 32), (552, 296, 24, 64, 64), (148, 148, 50, 64, 64),
    (100, 100, 100, 64, 64), (1000, 1000, 12, 64, 64), (2088, 1064, 4, 64, 64),
    (1160, 920, 8, 64, 64), (300, 4000, 12, 64, 64),
    # tiles of which little is grid, more of them than the chip holds: gradients up to
    # 2.6 times faster on streams, traces 2.3 times
    (56, 56, 600, 0, 0), (56, 56, 2000, 0, 0), (100, 100, 200, 0, 64), (100, 100, 600, 0, 0),
    (148, 148, 300, 0, 0), (52, 600, 200, 0, 0), (200, 200, 160, 0, 0),
    (552, 296, 48, 0, 0), (740, 540, 24, 64, 0),
    (2088, 1064, 6, 0, 0), (4000, 300, 12, 0, 0), (2088, 1064, 64, 0, 0)])
def test_measured_calls_take_the_faster_kernels(route, NX, NY, S, gradient, traces):
    assert route(NX, NY, S, GRADIENT) == gradient
    assert route(NX, NY, S, CHECKPOINT) == route(NX, NY, S, HISTORY) == gradient
    assert route(NX, NY, S, NONE) == traces


FAR_CODE = """
#include "fwi_host.h"
#include <cstring>
using namespace fwi;
using namespace fwi::host;
static char ws[1 << 20];
extern "C" int far_of(int NX, int NY, int S, int mode) {
    Dims d{};
    d.NX = NX; d.NY = NY; d.npml = 10; d.nt = 96; d.S = S; d.R = 4;
    d.pitch = (NX + 63) / 64 * 64; d.W = d.Hs = 21;
    d.plane = (size_t)NY * d.pitch; d.xs = (size_t)NY * d.W; d.ys = (size_t)d.Hs * d.pitch;
    Layout L;
    if (make_layout(d, mode, L) != FWI_OK) return -1;
    const FwdStreamArgs a = fwd_args(Ptrs{ws, &L});
    return a.tl.tile ? 2 : a.far;
}
"""


def test_only_large_sweeps_store_past_the_caches(tmp_path):
    """2: tiles; else whether the streaming sweep's stores pass the caches by, which
    costs it up to a fifth where the caches hold a part of its fields."""
    f = build(tmp_path, "far", FAR_CODE).far_of
    assert [f(740, 540, 24, NONE), f(552, 296, 48, NONE), f(2088, 1064, 8, NONE)] == [0, 0, 0]
    assert [f(2088, 1064, 64, m) for m in (NONE, GRADIENT)] == [1, 1]
    assert f(100, 100, 900, NONE) == f(552, 296, 150, NONE) == 1
    assert f(552, 296, 24, GRADIENT) == 2 and f(552, 296, 48, GRADIENT) == 0
