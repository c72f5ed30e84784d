// Which kernel a 3x3 convolution and its weight gradient take (fwi_nn.hip), and how
// the row-marching ones split their images.  Host code without a GPU type in it, so that the rule can be
// checked on the CPU.
#pragma once

#include <stdint.h>

#include <algorithm>
#include <cmath>

namespace fwi_nn {

// Bands of rows per image for `base` strips and channel groups: a block pays
// about 6 rows' time for its weights and first rows and reads 2 halo rows; with
// one block per CU nothing hides its latencies (weighed 1.3), two share a CU, and
// of a last, partial round beyond that half the idle time counts.  Fitted to
// sweeps of the block count over the network's layers: 32 images of 128 x 128,
// 32 channels, best at 512 blocks (18.6 us; 256: 22.4, 1024: 20.8), of 32 x 32,
// 64 to 128 channels, at 256 (13.2; 512: 14.8, 1024: 20.8).
inline int row_bands(long long base, int H) {
    int best = 1;
    double best_t = 1e300;
    // of the band counts with the same rows per band the smallest is the cheapest
    for (int nb = 1; nb <= H && (nb == 1 || base * nb <= 4096);) {
        const int rows = (H + nb - 1) / nb;
        const double r = (double)(base * nb) / 256.0, up = std::ceil(r);
        const double rounds = r <= 1.0 ? 1.3 : (r <= 2.0 ? up : r + 0.5 * (up - r));
        const double t = (rows + 2) * rounds + 6.0 * std::ceil(r / 2.0);
        if (t < best_t) {
            best_t = t;
            best = nb;
        }
        nb = rows > 1 ? (H - 1) / (rows - 1) + 1 : H + 1;
    }
    return best;
}

// The row-marching kernel's waves (CG groups of 16 CT channels x PG groups of
// 16-pixel tiles) and its split of N images: strips of columns, bands of rows.
struct RowsPlan {
    int ct, cg, pg;
    int strip, nstrip, rows, nrow, nco;
    long long blocks;
};

inline RowsPlan rows_strips(int W, int Ci, int Co) {
    RowsPlan p{};
    p.ct = Ci == 128 ? 1 : 2;
    p.cg = Co % 64 ? (Ci == 128 ? 2 : 1) : (Ci == 128 || (Ci == 64 && Co % 128 == 0)) ? 4 : 2;
    p.pg = 4 / p.cg;
    const int BW = 4096 / Ci;
    p.nstrip = (W + BW - 1) / BW;
    p.strip = (W + p.nstrip - 1) / p.nstrip;
    p.nco = Co / (16 * p.ct * p.cg);
    return p;
}

inline void rows_bands(RowsPlan &p, int N, int H) {
    const int bands = row_bands((long long)N * p.nstrip * p.nco, H);
    p.rows = (H + bands - 1) / bands;
    p.nrow = (H + p.rows - 1) / p.rows;
    p.blocks = (long long)N * p.nrow * p.nstrip * p.nco;
}

// Microseconds of a convolution, fitted to 160 shapes of 3 thousand to 700
// thousand pixels, images of 1 to 300 rows and columns and a few far beyond, each
// with the channel counts 32 -> 32, 64 up to 128 -> 256 (mostly within 10%).
// Row-marching kernel: a start, and per round of blocks (one per CU, then two side
// by side) a block's start and its rows, each of which costs as many 16-pixel tiles
// as the wave with the most has.
struct RowsFit {
    double start, block, row, tile, two, idle;
};
inline const RowsFit &rows_fit(int Ci, int Co) {
    static const RowsFit f32 = {5.75, 0.5, 0.34, 0.10, 1.13, 0.0}, f32w = {5.2, 0.2, 0.28, 0.19, 1.32, 0.06},
                         f64 = {3.3, 2.9, 0.20, 0.39, 1.68, 0.5}, f128 = {3.8, 1.2, 0.43, 0.42, 1.79, 0.45};
    return Ci == 128 ? f128 : Ci == 64 ? f64 : Co % 64 ? f32 : f32w;
}
// tiles per row of the wave with the most
inline int most_tiles(const RowsPlan &p, int Ci) {
    const int all = 4096 / Ci / 16;
    return std::min((all + p.pg - 1) / p.pg, (p.strip + 15) / 16);
}
inline double rows_time(const RowsPlan &p, int Ci, int Co) {
    const RowsFit &f = rows_fit(Ci, Co);
    const double r = (double)p.blocks / 256.0;
    const double rounds =
        r <= 1.0 ? 1.0 : r <= 2.0 ? f.two : f.two * (r / 2 + f.idle * (std::ceil(r / 2) - r / 2));
    return f.start + rounds * (f.block + (p.rows + 2) * (f.row + f.tile * most_tiles(p, Ci)));
}
// The other two: the LDS-tiled kernel, which is busy with any shape, and the direct
// one of small layers.
inline double lds_time(int64_t P, int Ci, int Co) {
    return 4.5 + Ci / 24.0 + 1e-7 * Ci * Co * (0.21 + 9.0 / Ci) * P;
}
inline double direct_time(int64_t P, int Ci, int Co) {
    return 5.0 + Ci / 24.0 + 1.03e-7 * Ci * Co * P;
}

// The kernel: the LDS-tiled one when it gives the chip enough blocks, with the
// narrower channel tile (bn) where only that one does, else the direct one; and in
// place of either the row-marching one where it is faster by 8% by the times above
// (below 8.3 us a call is bound by its launch).  Its order of the reduction is that of
// the kernel it stands for, so the choice does not change a bit.  Many rows of wide
// images suit it (32 images of 128 x 128, 32 channels: 39 -> 18 us; 128 -> 64
// channels, 3 of 45 x 83: 26.6 -> 9.5), images of a few rows or columns do not: a
// block starts for each (8192 images of 1 x 16, 64 -> 32 channels: 14 us, 135 by
// rows; 16384 of one pixel: 8.8, 264; 11 of 234 x 19, 128 channels: 27.7, 35.9).
struct ConvRoute {
    enum Kernel { Rows, Lds, Direct } kernel;
    int bn;                 // channel tile of the LDS-tiled kernel
    bool kxc;               // reduction over (ky, kx, ci) as the direct kernel has it
    RowsPlan rows;
};

inline ConvRoute conv_route(int N, int H, int W, int Ci, int Co, bool aligned8) {
    const int64_t P = (int64_t)N * H * W;
    ConvRoute c{};
    c.bn = Co % 64 == 0 ? 64 : 32;
    if (c.bn == 64 && (P + 127) / 128 * (Co / 64) < 256) c.bn = 32;
    c.kxc = (P + 127) / 128 * (Co / c.bn) < 256;
    c.kernel = c.kxc ? ConvRoute::Direct : ConvRoute::Lds;
    // 32 channels of a small layer are bound by the launch on any kernel
    if (!aligned8 || (Ci != 32 && Ci != 64 && Ci != 128) || (c.kxc && Ci == 32)) return c;
    const double other = c.kxc ? direct_time(P, Ci, Co) : lds_time(P, Ci, Co), launch = 8.3;
    const double most = 0.92 * std::max(launch, other);
    c.rows = rows_strips(W, Ci, Co);
    // no split does better than every CU busy with rows alone
    const RowsFit &f = rows_fit(Ci, Co);
    const double least = (double)N * H * c.rows.nstrip * c.rows.nco / 256 * std::min(1.0, f.two / 2) *
                         (f.row + f.tile * most_tiles(c.rows, Ci));
    if (launch >= most || f.start + least >= most) return c;
    rows_bands(c.rows, N, H);
    // (a launch holds fewer than 2^32 threads)
    if (c.rows.blocks < 1 << 24 && rows_time(c.rows, Ci, Co) < most) c.kernel = ConvRoute::Rows;
    return c;
}

// Strips and rows per step of k_wgrad_rows: the pair with the fewest steps (of
// at most BW pixels each), the widest strips among equals (least halo).
struct WgradPlan {
    int strip, nstrip, srow;
    long long steps;
};

inline WgradPlan wgrad_plan(int BW, int N, int H, int W) {
    WgradPlan best{};
    const int least = (W + BW - 1) / BW;
    for (int n = least; n <= least + 8; ++n) {
        const int strip = n == 1 ? W : ((W + n - 1) / n + 7) / 8 * 8;
        const int strip8 = (strip + 7) / 8 * 8;
        const int ns = (W + strip - 1) / strip, srow = std::min(BW / strip8, H);
        const long long steps = (long long)N * ns * ((H + srow - 1) / srow);
        if (best.steps == 0 || steps < best.steps) best = {strip, ns, srow, steps};
        if (strip8 <= 16) break;
    }
    return best;
}

// Rows: as many blocks as the chip holds at once, one of eight waves per CU or two
// of four (at most one per step and record).  Eight waves write half the records:
// with up to 8 steps per block (3 x 45 x 83, 64 -> 128: 17.9 us against 22.1 with
// four; 32 x 128 x 128, 32 channels: 30.3, 31.7).  Beyond, two blocks that wait for
// each other's loads (1024 x 2048, 32 channels: 83.7 against 79.0; 512 x 1024, 64:
// 76.2, 68.2).
struct WgradRoute {
    int waves;              // of the row-marching kernel, 0: the flattened one
    int records;            // partial sums written
    WgradPlan plan;
};

// Rows or the flattened kernel, by the time of each, in us: both write and read
// their records (37.7 MB of them: 16 us), the flattened one takes its chunks of 32
// pixels in any shape, the rows take steps of 256 (eight waves) or 128 pixels, of
// which a narrow image fills an eighth per column, and pay for each strip's start.
// Constants from 40 shapes x 7 channel counts, within 15% of nearly all.  Images of
// 32 x 16 x 16, 256 channels: rows 33.3, flattened 44.4; 700 of 13 x 14: 337, 437; but
// 8192 x 1, 256 channels: 103, 44; 512 of 128 x 2: 757, 449; 1000 of 12 x 11, 64
// channels: 43.3, 40.7.  Below 128 pixels an image leaves a step mostly padding (512 x
// 8 x 8, 128 channels: 47.2, 44.6; 1024 x 1 x 1, 64 channels: 64.1, 12.8).
inline WgradRoute wgrad_route(int N, int H, int W, int Ci, int Co, int nsplit) {
    const int tiles = (Co / 32) * (Ci / 32);
    WgradRoute flat{0, nsplit, {}};
    if (H * W < 128) return flat;
    auto blocks = [&](long long steps, int fill) {
        return (int)std::min<long long>({(long long)nsplit, steps, (long long)std::max(1, fill)});
    };
    const double work = (double)N * H * W * tiles;
    auto share = [&](int records) { return records * 36.0 * Ci * Co / 37.7e6; };
    const double f = share(nsplit), busy = std::max(1.0, 512.0 / ((double)nsplit * tiles));
    const double flat_time =
        std::max(std::max(11.5, 8 + 16 * f), 6 + 12 * f + 4.9e-5 * work * busy);
    WgradRoute r{8, 0, wgrad_plan(256, N, H, W)};
    r.records = blocks(r.plan.steps, 256 / tiles);
    double step = 1.7, start = 0.3, record = 16;
    if (r.plan.steps > 8LL * r.records) {
        r = {4, 0, wgrad_plan(128, N, H, W)};
        r.records = blocks(r.plan.steps, 512 / tiles);
        step = 1.35, start = 0.9, record = 8;
    }
    const int per = (H + r.plan.srow - 1) / r.plan.srow;
    const double each = std::ceil((double)r.plan.steps / r.records);
    // (more tiles than the chip holds blocks: rounds of them)
    const double rounds = std::max(1.0, (double)r.records * tiles / (r.waves == 8 ? 256 : 512));
    const double time = 10 + record * share(r.records) + rounds * each * (step + start / per);
    return time < 0.94 * flat_time ? r : flat;
}

}  // namespace fwi_nn
