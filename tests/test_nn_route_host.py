"""The rules that pick the kernel of a convolution and of its weight gradient
(csrc/fwi_nn_route.h), compiled by the host compiler: the row-marching kernel for the network's layers, not for images of a
few rows or columns (where it starts a block per image and was up to thirty times
slower), never with more threads than a launch holds, and with a split that covers
the image; the shapes that tests/test_gpu_nn_route.py runs take the kernel they are
there for."""
import ctypes
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2506_20513_amd", "csrc")
CODE = """
#include "fwi_nn_route.h"
extern "C" void route(int N, int H, int W, int Ci, int Co, int aligned, long long *o) {
    const fwi_nn::ConvRoute c = fwi_nn::conv_route(N, H, W, Ci, Co, aligned != 0);
    o[0] = c.kernel; o[1] = c.bn; o[2] = c.kxc; o[3] = c.rows.strip; o[4] = c.rows.nstrip;
    o[5] = c.rows.rows; o[6] = c.rows.nrow; o[7] = c.rows.nco; o[8] = c.rows.blocks;
    o[9] = c.rows.ct; o[10] = c.rows.cg; o[11] = c.rows.pg;
}
extern "C" void wgrad(int N, int H, int W, int Ci, int Co, int nsplit, long long *o) {
    const fwi_nn::WgradRoute r = fwi_nn::wgrad_route(N, H, W, Ci, Co, nsplit);
    o[0] = r.waves; o[1] = r.records; o[2] = r.plan.strip; o[3] = r.plan.nstrip;
    o[4] = r.plan.srow; o[5] = r.plan.steps;
}
"""
ROWS, LDS, DIRECT = 0, 1, 2

# edges of the row-marching kernel, large and small layers
EDGES = [(300, 20, 31, 32, 64), (8, 257, 128, 32, 32), (4, 500, 129, 32, 32), (4, 701, 127, 32, 32),
         (1, 300, 257, 32, 64), (2, 200, 128, 32, 96), (3, 400, 144, 32, 32), (1, 100, 65, 64, 32),
         (2, 45, 64, 64, 64), (2, 300, 15, 64, 64), (1, 300, 191, 64, 64), (1, 40, 129, 64, 128),
         (4, 100, 129, 64, 128), (1, 600, 127, 64, 32), (9, 100, 1, 128, 64), (3, 64, 33, 128, 64),
         (1, 31, 97, 128, 32), (4, 67, 128, 128, 128), (2, 190, 96, 128, 32), (1, 256, 161, 128, 256),
         (1, 11, 31, 128, 192), (1, 1, 2000, 128, 256), (5, 7, 33, 128, 64)]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("route")
    src, so = d / "route.cpp", d / "route.so"
    src.write_text(CODE)
    subprocess.run([cxx, "-std=c++17", "-O2", "-Wall", "-fPIC", "-shared", "-I", CSRC, str(src),
                    "-o", str(so)], check=True)
    return ctypes.CDLL(str(so))


@pytest.fixture(scope="module")
def route(lib):
    def f(N, H, W, Ci, Co, aligned=1):
        o = (ctypes.c_longlong * 12)()
        lib.route(N, H, W, Ci, Co, aligned, o)
        return list(o)
    return f


@pytest.mark.parametrize("shape", [
    (8192, 1, 16, 64, 32), (8192, 2, 16, 32, 32), (16384, 1, 1, 64, 32), (1024, 1, 1, 128, 256),
    (4096, 2, 2, 64, 32), (512, 2, 2, 128, 256), (2048, 1, 32, 64, 64), (256, 1, 512, 64, 32),
    (2048, 1, 128, 64, 32), (1, 2, 32768, 128, 256), (11, 234, 19, 128, 128), (300, 12, 16, 64, 64),
    (16, 100, 65, 32, 32)])
def test_images_of_few_rows_or_columns_keep_the_other_kernels(route, shape):
    assert route(*shape)[0] != ROWS


@pytest.mark.parametrize("shape", [
    (32, 128, 128, 32, 32), (32, 64, 64, 32, 64), (32, 64, 64, 64, 64), (32, 32, 32, 64, 128),
    (32, 32, 32, 128, 128), (32, 16, 16, 128, 256), (32, 32, 32, 128, 64), (32, 64, 64, 64, 32),
    (1, 1024, 2048, 32, 32), (1, 512, 1024, 64, 64), (1, 256, 512, 128, 128), (3, 45, 83, 128, 64)])
def test_layers_of_the_network_march_rows(route, shape):
    assert route(*shape)[0] == ROWS
    assert route(*shape, 0)[0] != ROWS            # 8-byte stores need their alignment
    assert route(*shape[:3], 256, 64)[0] != ROWS  # too many weights for the registers


def test_splits_cover_the_image_and_launches_hold_them(route):
    for N, H, W, Ci, Co in EDGES + [(1, h, w, ci, 64) for ci in (32, 64, 128)
                                    for h in (1, 7, 300, 4097, 32768) for w in (1, 17, 333, 32768)]:
        k, bn, kxc, strip, nstrip, rows, nrow, nco, blocks, ct, cg, pg = route(N, H, W, Ci, Co)
        assert bn in (32, 64) and Co % bn == 0
        if not blocks:
            assert k != ROWS
            continue
        assert strip <= 4096 // Ci and (nstrip - 1) * strip < W <= nstrip * strip
        assert (nrow - 1) * rows < H <= nrow * rows and cg * pg == 4
        assert nco * 16 * ct * cg == Co and blocks == N * nrow * nstrip * nco
    for N, H, W in ((1 << 24, 1, 16), (1 << 24, 2, 32), (1 << 25, 16, 1), (1 << 26, 8, 8)):
        assert route(N, H, W, 32, 32)[0] != ROWS and route(N, H, W, 64, 128)[0] != ROWS


def test_the_edge_shapes_take_the_row_kernel(route):
    got = {s: route(*s) for s in EDGES}
    assert [s for s in EDGES if got[s][0] != ROWS] == []
    assert {got[s][2] for s in EDGES} == {0, 1}   # both orders of the reduction


def _nsplit(N, H, W, Ci, Co):
    """as the network chooses it"""
    return max(1, min(-(-N * H * W // 32), -(-1024 // (Co // 32 * (Ci // 32))), 1024))


@pytest.fixture(scope="module")
def wgrad(lib):
    def f(N, H, W, Ci, Co, nsplit=None):
        o = (ctypes.c_longlong * 6)()
        lib.wgrad(N, H, W, Ci, Co, nsplit or _nsplit(N, H, W, Ci, Co), o)
        return list(o)
    return f


@pytest.mark.parametrize("shape,rows", [
    # one to three columns fill at most three eighths of a step
    ((1, 8192, 1, 256, 256), 0), ((1, 32768, 2, 128, 128), 0), ((512, 128, 2, 64, 64), 0),
    ((512, 128, 1, 128, 256), 0), ((64, 64, 2, 256, 256), 0), ((64, 130, 1, 32, 32), 0),
    ((64, 1, 130, 256, 256), 0), ((1000, 12, 11, 128, 64), 0), ((512, 8, 8, 128, 128), 0),
    # the network's layers, and narrow ones that gain all the same
    ((32, 128, 128, 32, 32), 1), ((32, 64, 64, 64, 64), 1), ((32, 32, 32, 128, 128), 1),
    ((32, 16, 16, 256, 256), 1), ((3, 45, 83, 64, 128), 1), ((1, 1024, 2048, 32, 32), 1),
    ((700, 13, 14, 256, 256), 1), ((64, 64, 4, 64, 64), 1), ((1, 8192, 8, 128, 128), 1)])
def test_weight_gradients_of_narrow_images_stay_flattened(wgrad, shape, rows):
    assert (wgrad(*shape)[0] > 0) == bool(rows)


def test_weight_gradient_splits_cover_the_image(wgrad):
    for N, H, W in [(n, h, w) for n in (1, 5) for h in (1, 2, 33, 500) for w in (1, 7, 130, 257, 3000)]:
        for ci, co, ns in ((32, 32, None), (128, 256, None), (32, 32, 1), (64, 64, 7), (1024, 1024, 3)):
            waves, records, strip, nstrip, srow, steps = wgrad(N, H, W, ci, co, ns)
            assert waves in (0, 4, 8) and 1 <= records <= (ns or _nsplit(N, H, W, ci, co))
            if waves:
                assert (nstrip - 1) * strip < W <= nstrip * strip and 1 <= srow <= H
                assert srow * (-(-strip // 8) * 8) <= 32 * waves
                assert records <= steps == N * nstrip * -(-H // srow)
