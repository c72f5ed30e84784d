"""Every shot group of one call takes the same kernels: tiles or streams, and the tile
height, go by the shots of the call, also where they do not divide by the groups."""
import ctypes

import pytest

from tests.host_routes import build

CODE = """
#include "fwi_host.h"
using namespace fwi;
using namespace fwi::host;
// tile heights of the groups of a call, and of one group for all its shots
extern "C" int group_tiles(int NX, int NY, int S, int nt, int G, int *tiles) {
    Dims d{};
    d.NX = NX; d.NY = NY; d.npml = 10; d.nt = nt; d.S = S; d.R = 4;
    d.pitch = (NX + 63) / 64 * 64; d.W = d.Hs = 21;
    d.plane = (size_t)NY * d.pitch; d.xs = (size_t)NY * d.W; d.ys = (size_t)d.Hs * d.pitch;
    Layout L;
    int rc = make_layout(d, -1, L);
    if (rc != FWI_OK) return rc;
    tiles[0] = L.tile;
    GroupLayout GL;
    rc = make_group_layout(d, G, GL);
    for (int g = 0; rc == FWI_OK && g < G; ++g) tiles[1 + g] = GL.grp[g].tile;
    return rc;
}
"""


@pytest.fixture(scope="module")
def group_tiles(tmp_path_factory):
    lib = build(tmp_path_factory.mktemp("groups"), "groups", CODE)

    def f(NX, NY, S, nt, G):
        o = (ctypes.c_int * 5)()
        assert lib.group_tiles(NX, NY, S, nt, G, o) == 0
        return list(o)[:1 + G]
    return f


def test_groups_of_a_call_take_the_same_kernels(group_tiles):
    seen = set()
    for NX, NY in ((270, 270), (148, 148), (552, 296), (740, 540), (1100, 1000), (2088, 1064), (60, 60)):
        for S in list(range(2, 130)) + [333, 1001]:
            for G in (2, 3, 4):
                if G > S:
                    continue
                t = group_tiles(NX, NY, S, 96, G)
                assert len(set(t)) == 1, (NX, NY, S, G, t)
                seen.add(t[0])
    assert seen == {0, 32, 64}
