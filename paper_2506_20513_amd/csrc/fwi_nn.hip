// Kernels of the learned gradient preconditioner: a small encoder-decoder
// CNN with 3x3 convolutions on BF16 activations and weights, FP32
// accumulation on the gfx950 matrix cores (v_mfma_f32_16x16x32_bf16).
//
// Layouts: activations NHWC [N][H][W][C] bf16 with C a multiple of 32;
// weights [Co][3][3][Ci] bf16 (FP32 masters held by the optimiser); all
// convolutions are 3x3, stride 1, zero padding 1.
//
// MFMA 16x16x32 operand layout (lane l of the wave): A holds row l%16,
// columns 8*(l/16) .. +7; B holds rows 8*(l/16) .. +7 of column l%16; the
// 16x16 result holds rows 4*(l/16) .. +3 of column l%16.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <type_traits>

#include "fwi_nn.h"
#include "fwi_nn_route.h"

namespace {

using bf16 = __bf16;
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// ---------------------------------------------------------------------------
// floor(n / d) for n d < 2^32 as the high word of n m with
// m = floor((2^32 - 1) / d) + 1 = 2^32 / d + e, 0 < e <= 1.  Then n m / 2^32 =
// n / d + n e / 2^32 with n e / 2^32 <= n / 2^32 < 1 / d, less than the
// distance from n / d up to the next integer, so the floor is exact.  d = 1
// (where m would overflow) is passed through.  Its users: the convolution and
// weight-gradient kernels with d = H or W <= 2^15 (checked by the host) and n < 2 d
// + 2^8; k_wgrad_rows with d <= 2^8 + 2 and n < 2^10; store_first_pieces with d
// <= 2^8 pieces of a pixel and n < 64 d.
struct SmallDiv {
    unsigned d, m;
    __device__ explicit SmallDiv(unsigned dd) : d(dd), m(dd > 1 ? 0xffffffffu / dd + 1u : 0u) {}
    __device__ __forceinline__ unsigned div(unsigned n) const { return d > 1 ? __umulhi(n, m) : n; }
    __device__ __forceinline__ unsigned mod(unsigned n) const { return n - d * div(n); }
};

// y = act(conv3x3(x, w) + bias) as an implicit GEMM: rows are output pixels
// in flattened (n, y, x) order, columns output channels, the reduction runs
// over (ky, kx, ci).  Tiling over flattened pixels keeps every lane busy on
// images narrower than a tile.  This form, with operands read straight from
// global memory, serves layers too small for the LDS-tiled kernel below: a
// block of four waves covers 64 * MT consecutive pixels; wave w owns MT
// tiles of 16 pixels times 16 * NT output channels.  A tap at
// (ky, kx) reads pixel p + (ky - 1) W + (kx - 1) when it lies in the image.
template <int NT, int MT, bool MASK>
__global__ __launch_bounds__(256) void k_conv3x3(const bf16 *__restrict__ x,
                                                 const bf16 *__restrict__ w,
                                                 const float *__restrict__ bias,
                                                 const bf16 *__restrict__ mask,
                                                 bf16 *__restrict__ y, int N, int H, int W,
                                                 int Ci, int Co, int relu) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t P = (int64_t)N * H * W;
    const int64_t base = ((int64_t)blockIdx.x * 4 + wave) * (16 * MT);
    const int co0 = blockIdx.y * (16 * NT);
    const int kq = (lane >> 4) * 8;
    int py[MT], px[MT];
    int64_t pp[MT];
    bool pv[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
        const int64_t p = base + m * 16 + (lane & 15);
        pv[m] = p < P;
        pp[m] = pv[m] ? p : 0;
        px[m] = (int)(pp[m] % W);
        py[m] = (int)((pp[m] / W) % H);
    }
    f32x4 acc[MT][NT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bf16x8 zero{};
    for (int ky = 0; ky < 3; ++ky) {
        for (int kx = 0; kx < 3; ++kx) {
            const int64_t shift = (int64_t)(ky - 1) * W + (kx - 1);
            const bf16 *xp[MT];
            bool ok[MT];
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                const int yy = py[m] + ky - 1, xx = px[m] + kx - 1;
                ok[m] = pv[m] && yy >= 0 && yy < H && xx >= 0 && xx < W;
                // out-of-image taps read a valid address and are zeroed
                xp[m] = x + (ok[m] ? (pp[m] + shift) * Ci : 0) + kq;
            }
            const bf16 *wp = w + ((size_t)(co0 + (lane & 15)) * 9 + ky * 3 + kx) * Ci + kq;
            for (int c0 = 0; c0 < Ci; c0 += 32) {
                bf16x8 a[MT];
#pragma unroll
                for (int m = 0; m < MT; ++m) {
                    a[m] = *reinterpret_cast<const bf16x8 *>(xp[m] + c0);
                    if (!ok[m]) a[m] = zero;
                }
#pragma unroll
                for (int j = 0; j < NT; ++j) {
                    const bf16x8 bv =
                        *reinterpret_cast<const bf16x8 *>(wp + (size_t)j * 16 * 9 * Ci + c0);
#pragma unroll
                    for (int m = 0; m < MT; ++m) acc[m][j] = mfma(a[m], bv, acc[m][j]);
                }
            }
        }
    }
#pragma unroll
    for (int j = 0; j < NT; ++j) {
        const int co = co0 + 16 * j + (lane & 15);
        const float bb = bias ? bias[co] : 0.f;
#pragma unroll
        for (int m = 0; m < MT; ++m) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t po = base + m * 16 + 4 * (lane >> 4) + r;
                if (po < P) {
                    float v = acc[m][j][r] + bb;
                    if (relu) v = fmaxf(v, 0.f);
                    if (MASK && !((float)mask[po * Co + co] > 0.f)) v = 0.f;
                    y[po * Co + co] = (bf16)v;
                }
            }
        }
    }
}

// The same convolution with both operand tiles staged in LDS: a block
// computes BM (128 or 64) consecutive (flattened) pixels x BN output
// channels.  A reduction step covers one kernel row ky and 32 input channels
// for all three kx taps: it stages the input rows of pixels base - 1 ..
// base + BM shifted by ky - 1 image rows (BM + 2 rows, zero where that row
// leaves the image) and the three BN x 32 weight tiles of (ky, kx = 0, 1, 2).
// Tap kx of output pixel p reads staged row p - base + kx, so the three taps
// share the staged rows; a tap that would wrap across a row edge (kx = 0 at
// column 0, kx = 2 at column W-1) gets a zero fragment.  Two LDS buffers, one
// barrier per step; the global loads of step k+1 are in flight while step k
// issues its 3 x (BM / 64) x BN/16 MFMAs per wave.  The 64-pixel tile
// doubles the blocks of layers with few pixels, where one block per CU
// leaves every global-load latency exposed.
constexpr int kTP = 40;      // LDS row pitch in bf16: 32 channels + 8 padding (80 bytes)

template <int BN, int BM, bool MASK>
__global__ __launch_bounds__(256) void k_conv3x3_lds(const bf16 *__restrict__ x,
                                                     const bf16 *__restrict__ w,
                                                     const float *__restrict__ bias,
                                                     const bf16 *__restrict__ mask,
                                                     bf16 *__restrict__ y, int N, int H, int W,
                                                     int Ci, int Co, int relu) {
    static_assert(BM == 64 || BM == 128, "64 or 128 pixels per block");
    constexpr int AR = BM + 2, NTL = BN / 16, MW = BM / 64;   // MW: 16-pixel tiles per wave
    constexpr int APieces = AR * 4, BPieces = 3 * BN * 4;     // 16-byte pieces per step
    constexpr int AU = (APieces + 255) / 256, BU = (BPieces + 255) / 256;
    __shared__ __attribute__((aligned(16))) bf16 As[2][AR * kTP];
    __shared__ __attribute__((aligned(16))) bf16 Bs[2][3 * BN * kTP];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int64_t P = (int64_t)N * H * W;
    const int64_t base = (int64_t)blockIdx.x * BM;
    const int co0 = blockIdx.y * BN;
    const int col0 = (int)(base % W), row0 = (int)((base / W) % H);
    const int nck = Ci / 32, K = 3 * nck;
    const SmallDiv dW((unsigned)W), dH((unsigned)H);
    // this lane's output pixels (offsets in the block) and their columns
    int pofs[MW], pcol[MW];
#pragma unroll
    for (int m = 0; m < MW; ++m) {
        pofs[m] = wave * 16 * MW + m * 16 + (lane & 15);
        pcol[m] = (int)dW.mod((unsigned)(col0 + pofs[m]));
    }
    uint4 ra[AU], rb[BU];
    auto fetch = [&](int k) {
        const int ky = k / nck, c0 = (k - ky * nck) * 32;
#pragma unroll
        for (int u = 0; u < AU; ++u) {
            const int idx = t + 256 * u;
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (idx < APieces) {
                const int j = idx >> 2, c = (idx & 3) * 8;
                const int64_t q = base - 1 + j;
                if (q >= 0 && q < P) {
                    const int d = col0 - 1 + j;                 // >= -1
                    const int row = row0 + (d >= 0 ? (int)dW.div((unsigned)d) : -1);
                    const int yy = (int)dH.mod((unsigned)(row + H)) + ky - 1;
                    if (yy >= 0 && yy < H)
                        v = *reinterpret_cast<const uint4 *>(
                            x + (q + (int64_t)(ky - 1) * W) * Ci + c0 + c);
                }
            }
            ra[u] = v;
        }
#pragma unroll
        for (int u = 0; u < BU; ++u) {
            const int idx = t + 256 * u;
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (idx < BPieces) {
                const int kx = idx / (BN * 4), r = idx - kx * (BN * 4);
                const int n = r >> 2, c = (r & 3) * 8;
                v = *reinterpret_cast<const uint4 *>(
                    w + ((size_t)(co0 + n) * 9 + ky * 3 + kx) * Ci + c0 + c);
            }
            rb[u] = v;
        }
    };
    auto stash = [&](int buf) {
#pragma unroll
        for (int u = 0; u < AU; ++u) {
            const int idx = t + 256 * u;
            if (idx < APieces)
                *reinterpret_cast<uint4 *>(&As[buf][(idx >> 2) * kTP + (idx & 3) * 8]) = ra[u];
        }
#pragma unroll
        for (int u = 0; u < BU; ++u) {
            const int idx = t + 256 * u;
            if (idx < BPieces)
                *reinterpret_cast<uint4 *>(&Bs[buf][(idx >> 2) * kTP + (idx & 3) * 8]) = rb[u];
        }
    };
    f32x4 acc[MW][NTL];
#pragma unroll
    for (int m = 0; m < MW; ++m)
#pragma unroll
        for (int n = 0; n < NTL; ++n) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
    const bf16x8 zero{};
    fetch(0);
    stash(0);
    __syncthreads();
    for (int k = 0; k < K; ++k) {
        const int buf = k & 1;
        if (k + 1 < K) fetch(k + 1);
#pragma unroll
        for (int kx = 0; kx < 3; ++kx) {
            bf16x8 a[MW];
#pragma unroll
            for (int m = 0; m < MW; ++m) {
                a[m] = *reinterpret_cast<const bf16x8 *>(
                    &As[buf][(pofs[m] + kx) * kTP + 8 * (lane >> 4)]);
                if ((kx == 0 && pcol[m] == 0) || (kx == 2 && pcol[m] == W - 1)) a[m] = zero;
            }
#pragma unroll
            for (int n = 0; n < NTL; ++n) {
                const bf16x8 bv = *reinterpret_cast<const bf16x8 *>(
                    &Bs[buf][(kx * BN + n * 16 + (lane & 15)) * kTP + 8 * (lane >> 4)]);
#pragma unroll
                for (int m = 0; m < MW; ++m) acc[m][n] = mfma(a[m], bv, acc[m][n]);
            }
        }
        if (k + 1 < K) stash(buf ^ 1);
        __syncthreads();
    }
#pragma unroll
    for (int n = 0; n < NTL; ++n) {
        const int co = co0 + n * 16 + (lane & 15);
        const float bb = bias ? bias[co] : 0.f;
#pragma unroll
        for (int m = 0; m < MW; ++m) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int64_t po = base + wave * 16 * MW + m * 16 + 4 * (lane >> 4) + r;
                if (po < P) {
                    float v = acc[m][n][r] + bb;
                    if (relu) v = fmaxf(v, 0.f);
                    if (MASK && !((float)mask[po * Co + co] > 0.f)) v = 0.f;
                    y[po * Co + co] = (bf16)v;
                }
            }
        }
    }
}

// The same convolution for 32, 64 and 128 input channels, marching down the rows
// of a strip of at most 4096 / CI pixels of one image.  Each wave keeps the weights of its 16
// CT output channels for all nine taps and all input channels in registers
// (9 CI / 32 CT fragments); the input rows pass once through a ring of four
// rows in LDS, one pixel of halo on both sides and zeros outside the image, so
// a fragment needs no mask.  Per output row one row is loaded (in flight while
// the row before it is computed) and one barrier passed.  The four waves are CG
// groups of channels x PG groups of 16-pixel tiles.  The weights are the row
// operand of the products, so a lane holds four neighbouring channels of one
// pixel and stores them as 8 bytes.  KXC: the reduction runs over (ky, kx, ci)
// instead of (ky, ci / 32, kx): the order of the kernel that serves the same
// layer otherwise, so every sum is the same bit for bit.
//
// 32 channels are bound by memory (1024 x 2048 pixels: 120 -> 50 us, 5.4 TB/s;
// 32 images of 128 x 128: 39 -> 18 us), 64 and 128 channels by the fragment reads
// from LDS, one kilobyte for CT products (512 x 1024 pixels, 64 channels: 81 -> 43
// us, 0.9 PFLOP/s; 256 x 512, 128 channels: 71 -> 50 us); the network's training
// layers of 64 and 128 channels by the start of a block, about 11 us (32 images
// of 64 x 64, 64 channels: 28.6 -> 20.7 us).  256 channels would need 288
// registers of weights per lane: one wave per SIMD, slower (70 -> 91 us).
template <int CI, int CT, int CG, int PG, bool KXC, bool MASK>
__global__ __launch_bounds__(256) void k_conv3x3_rows(const bf16 *__restrict__ x,
                                                      const bf16 *__restrict__ w,
                                                      const float *__restrict__ bias,
                                                      const bf16 *__restrict__ mask,
                                                      bf16 *__restrict__ y, int H, int W, int Co,
                                                      int relu, int strip, int nstrip, int rows,
                                                      int nrow) {
    static_assert(CG * PG == 4, "four waves");
    constexpr int NC = CI / 32, PITCH = CI + 8, BW = 4096 / CI, PT = (BW / 16 + PG - 1) / PG;
    constexpr int RowPieces = (BW + 2) * CI / 8, U = (RowPieces + 255) / 256;
    __shared__ __attribute__((aligned(16))) bf16 ring[4][(BW + 2) * PITCH];
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int cg = wave % CG, pg = wave / CG, kq = 8 * (lane >> 4);
    // block -> (image, band of rows, strip); strips fastest
    const int sx = blockIdx.x % nstrip, by = blockIdx.x / nstrip;
    const int n = by / nrow, y0 = by % nrow * rows, y1 = min(H, y0 + rows);
    const int xs = sx * strip, sw = min(strip, W - xs);
    const int co0 = (blockIdx.y * CG + cg) * 16 * CT;
    const bf16 *xi = x + (size_t)n * H * W * CI;

    uint4 pre[U];
    const int pieces = (sw + 2) * (CI / 8);
    auto fetch = [&](int yy, uint4 *pre) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int idx = t + 256 * u, j = idx / (CI / 8), c = idx % (CI / 8) * 8;
            const int xx = xs - 1 + j;
            pre[u] = make_uint4(0u, 0u, 0u, 0u);
            if (idx < pieces && yy >= 0 && yy < H && xx >= 0 && xx < W)
                pre[u] = *reinterpret_cast<const uint4 *>(xi + ((size_t)yy * W + xx) * CI + c);
        }
    };
    auto stash = [&](int slot, const uint4 *pre) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int idx = t + 256 * u, j = idx / (CI / 8), c = idx % (CI / 8) * 8;
            if (idx < pieces) *reinterpret_cast<uint4 *>(&ring[slot][j * PITCH + c]) = pre[u];
        }
    };
    uint4 first[3][U];
#pragma unroll
    for (int k = 0; k < 3; ++k) fetch(y0 - 1 + k, first[k]);
    bf16x8 wf[3][NC][3][CT];
#pragma unroll
    for (int ky = 0; ky < 3; ++ky)
#pragma unroll
        for (int c = 0; c < NC; ++c)
#pragma unroll
            for (int kx = 0; kx < 3; ++kx)
#pragma unroll
                for (int ct = 0; ct < CT; ++ct)
                    wf[ky][c][kx][ct] = *reinterpret_cast<const bf16x8 *>(
                        w + ((size_t)(co0 + 16 * ct + (lane & 15)) * 9 + ky * 3 + kx) * CI +
                        32 * c + kq);
    float bb[CT][4];
#pragma unroll
    for (int ct = 0; ct < CT; ++ct)
#pragma unroll
        for (int r = 0; r < 4; ++r)
            bb[ct][r] = bias ? bias[co0 + 16 * ct + 4 * (lane >> 4) + r] : 0.f;
#pragma unroll
    for (int k = 0; k < 3; ++k) stash(k, first[k]);

    for (int yo = y0; yo < y1; ++yo) {
        const int k0 = yo - y0;
        __syncthreads();
        if (yo + 1 < y1) fetch(yo + 2, pre);
        // NP tiles of 16 pixels from tile pt0 on, together
        auto tiles = [&](auto np, int pt0) {
            constexpr int NP = decltype(np)::value;
            f32x4 acc[NP][CT];
#pragma unroll
            for (int i = 0; i < NP; ++i)
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) acc[i][ct] = f32x4{0.f, 0.f, 0.f, 0.f};
            const int p0 = (pg * PT + pt0) * 16 + (lane & 15);
            const size_t o0 = (((size_t)n * H + yo) * W + xs + p0) * Co + co0 + 4 * (lane >> 4);
            bf16x4 mk[NP][CT];                               // in flight during the products
            if (MASK)
#pragma unroll
                for (int i = 0; i < NP; ++i)
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct)
                        if (p0 + 16 * i < sw)
                            mk[i][ct] = *reinterpret_cast<const bf16x4 *>(
                                mask + o0 + (size_t)16 * i * Co + 16 * ct);
#pragma unroll
            for (int ky = 0; ky < 3; ++ky) {
                const bf16 *row = &ring[(k0 + ky) & 3][p0 * PITCH + kq];
                auto tap = [&](int c, int kx) {
#pragma unroll
                    for (int i = 0; i < NP; ++i) {
                        const bf16x8 a = *reinterpret_cast<const bf16x8 *>(
                            row + (16 * i + kx) * PITCH + 32 * c);
#pragma unroll
                        for (int ct = 0; ct < CT; ++ct)
                            acc[i][ct] = mfma(wf[ky][c][kx][ct], a, acc[i][ct]);
                    }
                };
                if (KXC) {
#pragma unroll
                    for (int kx = 0; kx < 3; ++kx)
#pragma unroll
                        for (int c = 0; c < NC; ++c) tap(c, kx);
                } else {
#pragma unroll
                    for (int c = 0; c < NC; ++c)
#pragma unroll
                        for (int kx = 0; kx < 3; ++kx) tap(c, kx);
                }
            }
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                if (p0 + 16 * i >= sw) continue;
                bf16 *out = y + o0 + (size_t)16 * i * Co;
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    bf16x4 v;
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        float f = acc[i][ct][r] + bb[ct][r];
                        if (relu) f = fmaxf(f, 0.f);
                        if (MASK && !((float)mk[i][ct][r] > 0.f)) f = 0.f;
                        v[r] = (bf16)f;
                    }
                    *reinterpret_cast<bf16x4 *>(out + 16 * ct) = v;
                }
            }
        };
        // this wave's tiles, two at a time
        const int nt = min(PT, (sw - pg * PT * 16 + 15) / 16);
        int pt = 0;
        if (PT > 1)
            for (; pt + 1 < nt; pt += 2) tiles(std::integral_constant<int, (PT > 1 ? 2 : 1)>(), pt);
        if (pt < nt) tiles(std::integral_constant<int, 1>(), pt);
        if (yo + 1 < y1) stash((k0 + 3) & 3, pre);
    }
}

template <int CI, int CT, int CG, int PG>
hipError_t launch_rows(const bf16 *x, const bf16 *w, const float *bias, const bf16 *mask, bf16 *y,
                       int N, int H, int W, int Co, int relu, const fwi_nn::ConvRoute &route,
                       hipStream_t st) {
    const fwi_nn::RowsPlan &p = route.rows;
    if (p.ct != CT || p.cg != CG || p.pg != PG) return hipErrorInvalidValue;
    const dim3 grid((unsigned)(N * p.nrow * p.nstrip), (unsigned)p.nco);
    // 32 channels: one order
    constexpr bool two = CI > 32;
    auto kernel = route.kxc && two ? (mask ? k_conv3x3_rows<CI, CT, CG, PG, two, true>
                                           : k_conv3x3_rows<CI, CT, CG, PG, two, false>)
                                   : (mask ? k_conv3x3_rows<CI, CT, CG, PG, false, true>
                                           : k_conv3x3_rows<CI, CT, CG, PG, false, false>);
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, x, w, bias, mask, y, H, W, Co, relu, p.strip,
                       p.nstrip, p.rows, p.nrow);
    return hipGetLastError();
}

// wf[ci][ky][kx][co] = w[co][2-ky][2-kx][ci]: the weights of the transposed
// convolution (input gradient = conv3x3(output gradient, wf)).
__global__ void k_flip(const bf16 *__restrict__ w, bf16 *__restrict__ wf, int Ci, int Co) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= Co * 9 * Ci) return;
    const int ci = t % Ci, k = (t / Ci) % 9, co = t / (9 * Ci);
    const int ky = k / 3, kx = k % 3;
    wf[((size_t)ci * 9 + (2 - ky) * 3 + (2 - kx)) * Co + co] = w[t];
}

// Several layers at once (one launch for the whole network): a block transposes
// 32 x 32 channels of one tap through LDS, reads and writes coalesced.  (A
// thread per element of wf, reading w Ci elements apart: 17 us for the
// preconditioner's 1.8 M weights; 7 us now.)
constexpr int kFlipMax = 32;
struct FlipTable {
    int n;
    int64_t off[kFlipMax], tile0[kFlipMax + 1];   // first element; first tile, and all
    int32_t ci[kFlipMax], co[kFlipMax];
};

__global__ __launch_bounds__(256) void k_flip_layers(const bf16 *__restrict__ w,
                                                     bf16 *__restrict__ wf, FlipTable tb) {
    __shared__ bf16 tile[32][34];
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    for (int64_t b = blockIdx.x; b < tb.tile0[tb.n]; b += gridDim.x) {
        int l = 0;
        while (b >= tb.tile0[l + 1]) ++l;
        const int Ci = tb.ci[l], Co = tb.co[l], nci = (Ci + 31) / 32;
        const int i = (int)(b - tb.tile0[l]), k = i % 9;
        const int ci0 = i / 9 % nci * 32, co0 = i / 9 / nci * 32;
        const bf16 *src = w + tb.off[l];
        bf16 *dst = wf + tb.off[l];
        for (int j = ty; j < 32; j += 8)
            if (co0 + j < Co && ci0 + tx < Ci)
                tile[j][tx] = src[((int64_t)(co0 + j) * 9 + (8 - k)) * Ci + ci0 + tx];
        __syncthreads();
        for (int j = ty; j < 32; j += 8)
            if (ci0 + j < Ci && co0 + tx < Co)
                dst[((int64_t)(ci0 + j) * 9 + k) * Co + co0 + tx] = tile[tx][j];
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// Weight and bias gradients: dw[co][ky][kx][ci] = sum_q dz[q][co] x[q + (ky-1, kx-1)][ci],
// db[co] = sum_q dz[q][co].  A GEMM whose reduction runs over output pixels
// q: a block owns a 32 (co) x 32 (ci) tile for all nine taps, loops over
// every gridDim.x-th chunk of CH pixels and writes its partial sums to
// record blockIdx.x of part (Co 9 Ci weight sums, then Co bias sums).
//
// Per chunk q0 .. q0+CH-1 the block stages, in natural (pixel-major) layout:
//   Z[j][c]      = dz[q0 + j][co tile]                          (CH rows)
//   X[ky][j][c]  = x[q0 - 1 + j + (ky-1) W][ci tile]             (CH + 2 rows)
// and each wave runs nine MFMAs per 32 pixels of the chunk.  Chunks of 64
// pixels (half the barriers and staging rounds per MFMA) made the training
// step 4% slower than chunks of 32 (2.32 against 2.22 ms at about 1024
// blocks per layer; 2.30 and 2.36 ms at 512 and 2048 blocks).
// X rows are zero where the row of q = q0 - 1 + j plus ky - 1 leaves the
// image (or q is outside 0 .. P-1).  A tap (ky, kx) reads X[ky] from row kx
// on, so the three kx taps share one staged tile; the taps that would wrap
// across a row edge (kx = 0 at column 0, kx = 2 at column W-1) are removed
// by zeroing those pixels in the dz fragment, in registers.
//
// The matrix fragments need 8 consecutive pixels of one channel per lane, a
// column of the pixel-major tiles: each comes from two transposing LDS
// reads (ds_read_b64_tr_b16).  Within a group of 16 lanes, lane i receives
// element i % 4 of the 8-byte chunks read by lanes i/4, i/4+4, i/4+8 and
// i/4+12; so with lane s of the group reading row base + s/4 at channel
// 4 (s % 4), lane i gets channel i at rows base .. base + 3.
constexpr int kWP = 40;     // LDS row pitch in bf16: 32 channels + 8 padding
constexpr int kWgradChunk = 32;   // pixels staged per step of k_wgrad

typedef __attribute__((address_space(3))) bf16x4 *lds_bf16x4_ptr;

// channels [16 h, 16 h + 16) of rows base .. base + 7 of a pixel-major LDS
// tile, as this lane's 8-pixel fragment
__device__ __forceinline__ bf16x8 tr_fragment(const bf16 *tile, int base, int h, int lane) {
    const int s = lane & 15;
    const bf16 *p0 = tile + (base + (s >> 2)) * kWP + 16 * h + 4 * (s & 3);
    const bf16 *p1 = p0 + 4 * kWP;
    const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(p0));
    const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4_ptr)(p1));
    return bf16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
}

template <int CH>
__global__ __launch_bounds__(256) void k_wgrad(const bf16 *__restrict__ x,
                                               const bf16 *__restrict__ dz,
                                               float *__restrict__ part, int N, int H, int W,
                                               int Ci, int Co) {
    static_assert(CH % 32 == 0, "chunks of whole 32-pixel fragments");
    constexpr int NH = CH / 32;                   // 32-pixel halves per chunk
    constexpr int XR = CH + 2;                    // staged X rows per ky
    __shared__ __attribute__((aligned(16))) bf16 Z[CH * kWP];
    __shared__ __attribute__((aligned(16))) bf16 X[3][XR * kWP];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, t = threadIdx.x;
    const int nci = Ci / 32;
    const int cit = blockIdx.y % nci, cot = blockIdx.y / nci;
    const int64_t P = (int64_t)N * H * W;
    const int64_t nchunk = (P + CH - 1) / CH;
    const int mt = wave >> 1, nt = wave & 1;      // this wave's 16 x 16 sub-tile
    const int g = lane >> 4;                      // pixel group: rows 8 g .. 8 g + 7
    f32x4 acc[9];
#pragma unroll
    for (int k = 0; k < 9; ++k) acc[k] = f32x4{0.f, 0.f, 0.f, 0.f};
    float bsum = 0.f;                               // bias partial (ci tile 0)
    const bool do_bias = cit == 0;
    const bf16 zero = (bf16)0.f;
    // staging: CH x 4 pieces of Z, then 3 x (CH + 2) x 4 pieces of X (16
    // bytes each), kPer per thread; the pieces of the next chunk are loaded
    // into registers while the current chunk computes.  Column and image row
    // of the chunk's first pixel advance incrementally from chunk to chunk,
    // and the few divisions left are high multiplies, so the index
    // arithmetic stays small against the MFMAs.
    constexpr int kZ = CH * 4;
    constexpr int kPieces = kZ + 3 * XR * 4;
    constexpr int kPer = (kPieces + 255) / 256;
    const SmallDiv dW((unsigned)W), dH((unsigned)H);
    const int64_t step = (int64_t)gridDim.x * CH;          // pixels between a block's chunks
    const int dcol = (int)(step % W);
    const int drow = (int)((step / W) % H);
    int col0 = (int)(((int64_t)blockIdx.x * CH) % W);
    int row0 = (int)(((int64_t)blockIdx.x * CH / W) % H);
    uint4 pre[kPer];
    auto fetch = [&](int64_t q0, int c0, int r0, uint4 *out) {
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int idx = t + 256 * u;
            uint4 v = make_uint4(0u, 0u, 0u, 0u);
            if (idx < kZ) {
                const int j = idx >> 2, c = (idx & 3) * 8;
                const int64_t q = q0 + j;
                if (q < P) v = *reinterpret_cast<const uint4 *>(dz + q * Co + cot * 32 + c);
            } else if (idx < kPieces) {
                const int r = idx - kZ;
                const int ky = r / (XR * 4), j = (r >> 2) % XR, c = (r & 3) * 8;
                const int64_t q = q0 - 1 + j;
                if (q >= 0 && q < P) {
                    const int d = c0 - 1 + j;                    // >= -1
                    const int row = r0 + (d >= 0 ? (int)dW.div((unsigned)d) : -1);
                    const int yy = (int)dH.mod((unsigned)(row + H)) + ky - 1;
                    if (yy >= 0 && yy < H)
                        v = *reinterpret_cast<const uint4 *>(
                            x + (q + (int64_t)(ky - 1) * W) * Ci + cit * 32 + c);
                }
            }
            out[u] = v;
        }
    };
    if ((int64_t)blockIdx.x < nchunk) fetch((int64_t)blockIdx.x * CH, col0, row0, pre);
    for (int64_t ch = blockIdx.x; ch < nchunk; ch += gridDim.x) {
        __syncthreads();   // previous chunk's reads done
#pragma unroll
        for (int u = 0; u < kPer; ++u) {
            const int idx = t + 256 * u;
            if (idx < kZ) {
                *reinterpret_cast<uint4 *>(&Z[(idx >> 2) * kWP + (idx & 3) * 8]) = pre[u];
            } else if (idx < kPieces) {
                const int r = idx - kZ;
                *reinterpret_cast<uint4 *>(&X[r / (XR * 4)][((r >> 2) % XR) * kWP + (r & 3) * 8]) =
                    pre[u];
            }
        }
        __syncthreads();
        // column and row of the next chunk's first pixel
        int ncol = col0 + dcol, nrow = row0 + drow;
        if (ncol >= W) {
            ncol -= W;
            ++nrow;
        }
        if (nrow >= H) nrow -= H;
        if (ch + gridDim.x < nchunk) fetch((ch + gridDim.x) * CH, ncol, nrow, pre);
#pragma unroll
        for (int hf = 0; hf < NH; ++hf) {
            // dz fragment (channels 16 mt .. +15, pixels 32 hf + 8 g .. +7)
            // and its two edge-masked copies
            const int pb = 32 * hf + 8 * g;
            const bf16x8 a1 = tr_fragment(Z, pb, mt, lane);
            bf16x8 a0 = a1, a2 = a1;
            int col = (int)dW.mod((unsigned)(col0 + pb));
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                if (col == 0) a0[e] = zero;
                if (col == W - 1) a2[e] = zero;
                col = col + 1 == W ? 0 : col + 1;
            }
#pragma unroll
            for (int ky = 0; ky < 3; ++ky) {
#pragma unroll
                for (int kx = 0; kx < 3; ++kx) {
                    const bf16x8 bv = tr_fragment(X[ky], pb + kx, nt, lane);
                    const bf16x8 a = kx == 0 ? a0 : (kx == 1 ? a1 : a2);
                    acc[ky * 3 + kx] = mfma(a, bv, acc[ky * 3 + kx]);
                }
            }
        }
        if (do_bias && t < 32) {
#pragma unroll 8
            for (int j = 0; j < CH; ++j) bsum += (float)Z[j * kWP + t];
        }
        col0 = ncol;
        row0 = nrow;
    }
    // this block's partial sums: record blockIdx.x of Co 9 Ci weight sums
    // followed by Co bias sums
    const size_t tile = (size_t)Co * 9 * Ci;
    float *o = part + blockIdx.x * (tile + Co);
#pragma unroll
    for (int k = 0; k < 9; ++k)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int co = cot * 32 + 16 * mt + 4 * (lane >> 4) + r;
            const int ci = cit * 32 + 16 * nt + (lane & 15);
            o[((size_t)co * 9 + k) * Ci + ci] = acc[k][r];
        }
    if (do_bias && t < 32) o[tile + cot * 32 + t] = bsum;
}

// The same gradients where images fill its steps (fwi_nn_route.h), marching down the
// rows of strips of at most BW pixels as the row convolution does: input rows pass
// once through a ring in LDS (one pixel of halo, zeros outside the image),
// output-gradient rows through another.  A block owns 32 x 32 channels for all nine
// taps; each of its NW waves keeps all of them (36 sums of 16 x 16 in registers), so a
// fragment read from LDS serves several products, and the waves take turns at the
// pixels.  The reduction index of a product is 32 pixels: four groups of 8
// neighbouring pixels of a row, which may lie in different rows, so the matrix cores
// work on images of eight columns as on wide ones (rows are padded to 8 pixels with
// zero gradients).  A lane reads 12 pixels of one channel by three transposing reads
// and shifts the fragments of the three kx taps out of them.  Block b takes the steps
// (strips of the images, srow rows at a time) [b T / G, (b + 1) T / G) and writes one
// record of sums.  The accumulators leave two waves per SIMD and take the registers to
// their end (256, with 4 values of the staging spilled, 20 bytes of scratch per lane),
// so a step's loads (issued one step ahead) are what it waits for, about 1.8 us for
// 0.6 us of products and LDS reads; loads two steps ahead (62 spilled), or half the
// sums per wave and four waves, are slower (41 and 54 us against 31 for 32 x 128 x 128
// pixels, 32 -> 32 channels).
typedef float f32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));   // records: 4-byte aligned
constexpr int kWRP = 40;    // pitch of a pixel in LDS: 32 channels + 8 padding

template <int NW>
__global__ __launch_bounds__(64 * NW, 2) void k_wgrad_rows(
    const bf16 *__restrict__ x, const bf16 *__restrict__ dz, float *__restrict__ part, int N,
    int H, int W, int Ci, int Co, int strip, int nstrip, int srow) {
    constexpr int BW = 32 * NW, NT = 64 * NW, P = kWRP;
    // 16-byte pieces per thread of srow rows: at most BW pixels of Z; of X two
    // pixels of halo more per row, of at most BW / 8 rows
    constexpr int UX = (BW * 5 + NT - 1) / NT, UZ = BW * 4 / NT;
    // X ring: 2 srow + 2 rows of strip8 + 4 pixels, at most 4 (BW + 4) pixels as
    // srow strip8 <= BW and strip8 >= 8; Z: 2 srow rows of strip8 pixels; pixels
    // of zeros behind each
    constexpr int XAll = 4 * (BW + 4) + 12, ZAll = 2 * BW + 8;
    __shared__ __attribute__((aligned(16))) bf16 Xs[XAll * P];
    __shared__ __attribute__((aligned(16))) bf16 Zs[ZAll * P];
    const int t = threadIdx.x, lane = t & 63, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    const int nci = Ci / 32, cit = blockIdx.y % nci * 32, cot = blockIdx.y / nci * 32;
    const int strip8 = (strip + 7) / 8 * 8, G8 = strip8 / 8, xrow = strip8 + 4;
    const int nx = 2 * srow + 2, nz = 2 * srow;              // ring sizes in rows
    const int xzero = nx * xrow, zzero = nz * strip8;        // pixel index of the zeros behind
    // this thread's pieces of srow rows: row and pixel
    const SmallDiv dX((unsigned)(strip + 2)), dZ((unsigned)strip), dG((unsigned)G8);
    int xr[UX], xj[UX], zr[UZ], zj[UZ];
#pragma unroll
    for (int u = 0; u < UX; ++u) {
        const unsigned q = (unsigned)(t + NT * u) >> 2;
        xr[u] = (int)dX.div(q);
        xj[u] = (int)dX.mod(q);
    }
#pragma unroll
    for (int u = 0; u < UZ; ++u) {
        const unsigned q = (unsigned)(t + NT * u) >> 2;
        zr[u] = (int)dZ.div(q);
        zj[u] = (int)dZ.mod(q);
    }
    const int c8 = (t & 3) * 8;
    const int per = (H + srow - 1) / srow;                   // steps of a strip
    const long long T = (long long)N * nstrip * per;
    const long long s0 = T * blockIdx.x / gridDim.x, s1 = T * (blockIdx.x + 1) / gridDim.x;

    int sw = 0, xs = 0;                                      // the strip's width and first column
    const bf16 *xi = x, *zi = dz;
    // nr rows of X from row yy on; srow rows of Z
    auto fetch_x = [&](uint4 (&px)[UX], int yy, int nr) {
#pragma unroll
        for (int u = 0; u < UX; ++u) {
            px[u] = make_uint4(0u, 0u, 0u, 0u);
            const int y = yy + xr[u], xx = xs - 1 + xj[u];
            if (xr[u] < nr && y >= 0 && y < H && xx >= 0 && xx < W && xj[u] < sw + 2)
                px[u] = *reinterpret_cast<const uint4 *>(xi + ((size_t)y * W + xx) * Ci + cit + c8);
        }
    };
    auto fetch_z = [&](uint4 (&pz)[UZ], int yy) {
#pragma unroll
        for (int u = 0; u < UZ; ++u) {
            pz[u] = make_uint4(0u, 0u, 0u, 0u);
            const int y = yy + zr[u];
            if (zr[u] < srow && y < H && zj[u] < sw)
                pz[u] = *reinterpret_cast<const uint4 *>(zi + ((size_t)y * W + xs + zj[u]) * Co +
                                                         cot + c8);
        }
    };
    auto stash_x = [&](const uint4 (&px)[UX], int slot, int nr) {   // slot of the first row
#pragma unroll
        for (int u = 0; u < UX; ++u) {
            int r = slot + xr[u];
            if (r >= nx) r -= nx;
            if (xr[u] < nr) *reinterpret_cast<uint4 *>(&Xs[(r * xrow + xj[u]) * P + c8]) = px[u];
        }
    };
    auto stash_z = [&](const uint4 (&pz)[UZ], int slot) {
#pragma unroll
        for (int u = 0; u < UZ; ++u)
            if (zr[u] < srow)
                *reinterpret_cast<uint4 *>(&Zs[((slot + zr[u]) * strip8 + zj[u]) * P + c8]) = pz[u];
    };
    f32x4 acc[2][2][9], bacc[2];
#pragma unroll
    for (int o = 0; o < 2; ++o) {
        bacc[o] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int k = 0; k < 9; ++k) acc[o][i][k] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    bf16x8 ones;
#pragma unroll
    for (int e = 0; e < 8; ++e) ones[e] = (bf16)1.f;
    const bool do_bias = cit == 0;
    // transposing read of pixels p .. p + 3, channels ch .. ch + 15
    const int lo = ((lane & 15) >> 2) * P + 4 * (lane & 3);
    auto tr = [&](const bf16 *tile, int p, int ch) {
        return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
                                             (lds_bf16x4_ptr)(tile + p * P + ch + lo)));
    };

    int xb = 0, zb = 0;                                      // slots of row y - 1 of X, y of Z
    int y = 0;
    const int chunks = (srow * G8 + 3) / 4;
    for (long long st = s0; st < s1; ++st) {
        if (st == s0 || y >= H) {                            // a new strip
            const long long col = st / per;
            y = (int)(st - col * per) * srow;
            const long long n = col / nstrip;
            xs = (int)(col - n * nstrip) * strip;
            sw = min(strip, W - xs);
            xi = x + n * H * W * Ci;
            zi = dz + n * H * W * Co;
            xb = zb = 0;
            // rows y - 1 .. y + srow of X, all in flight together
            uint4 p0[UX], p1[UX], p2[UX], pz[UZ];
            const int more = min(srow, 2);
            fetch_x(p0, y - 1, srow);
            fetch_x(p1, y - 1 + srow, more);
            if (more == 1) fetch_x(p2, y + srow, 1);
            fetch_z(pz, y);
            if (st == s0) {
                // the padding pixels stay zero from here on
                for (int i = t; i < XAll * P / 8; i += NT)
                    reinterpret_cast<uint4 *>(Xs)[i] = make_uint4(0u, 0u, 0u, 0u);
                for (int i = t; i < ZAll * P / 8; i += NT)
                    reinterpret_cast<uint4 *>(Zs)[i] = make_uint4(0u, 0u, 0u, 0u);
            }
            __syncthreads();
            stash_x(p0, 0, srow);
            stash_x(p1, srow, more);
            if (more == 1) stash_x(p2, 2, 1);
            stash_z(pz, 0);
        }
        __syncthreads();
        const bool next = st + 1 < s1 && y + srow < H;
        uint4 px[UX], pz[UZ];
        if (next) {
            fetch_x(px, y + srow + 1, srow);
            fetch_z(pz, y + srow);
        }
        for (int c = wave; c < chunks; c += NW) {
            const int gi = 4 * c + g;
            const int r = (int)dG.div((unsigned)gi), p8 = 8 * (gi - r * G8);
            const bool in = r < srow && y + r < H;
            const int zp = in ? (zb + r) * strip8 + p8 : zzero;
            bf16x8 a[2];
#pragma unroll
            for (int o = 0; o < 2; ++o) {
                const uint2 d0 = tr(Zs, zp, 16 * o), d1 = tr(Zs, zp + 4, 16 * o);
                a[o] = __builtin_bit_cast(bf16x8, make_uint4(d0.x, d0.y, d1.x, d1.y));
                if (do_bias) bacc[o] = mfma(a[o], ones, bacc[o]);
            }
#pragma unroll
            for (int ky = 0; ky < 3; ++ky) {
                int q = xb + r + ky;
                if (q >= nx) q -= nx;
                const int xp = in ? q * xrow + p8 : xzero;
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    const uint2 d0 = tr(Xs, xp, 16 * i), d1 = tr(Xs, xp + 4, 16 * i),
                                d2 = tr(Xs, xp + 8, 16 * i);
                    const bf16x8 b0 =
                        __builtin_bit_cast(bf16x8, make_uint4(d0.x, d0.y, d1.x, d1.y));
                    const bf16x8 b1 = __builtin_bit_cast(
                        bf16x8, make_uint4(__builtin_amdgcn_alignbit(d0.y, d0.x, 16),
                                           __builtin_amdgcn_alignbit(d1.x, d0.y, 16),
                                           __builtin_amdgcn_alignbit(d1.y, d1.x, 16),
                                           __builtin_amdgcn_alignbit(d2.x, d1.y, 16)));
                    const bf16x8 b2 =
                        __builtin_bit_cast(bf16x8, make_uint4(d0.y, d1.x, d1.y, d2.x));
#pragma unroll
                    for (int o = 0; o < 2; ++o) {
                        acc[o][i][3 * ky] = mfma(b0, a[o], acc[o][i][3 * ky]);
                        acc[o][i][3 * ky + 1] = mfma(b1, a[o], acc[o][i][3 * ky + 1]);
                        acc[o][i][3 * ky + 2] = mfma(b2, a[o], acc[o][i][3 * ky + 2]);
                    }
                }
            }
        }
        if (next) {
            int xn = xb + srow + 2;                          // slot of row y + srow + 1
            if (xn >= nx) xn -= nx;
            zb = zb ? 0 : srow;
            stash_x(px, xn, srow);
            stash_z(pz, zb);
            xb += srow;
            if (xb >= nx) xb -= nx;
        }
        y += srow;
    }
    // the waves' sums in wave order: the waves take the 16 x 16 tiles of two taps
    // in turns.  A lane holds four input channels of one output channel and
    // stores them at once.
    const size_t tile = (size_t)Co * 9 * Ci;
    float *out = part + blockIdx.x * (tile + Co);
    float *red = reinterpret_cast<float *>(Xs);              // [wave][tap][tile][256]
    static_assert(sizeof(Xs) >= NW * 8 * 256 * sizeof(float), "two taps' tiles fit");
#pragma unroll
    for (int k0 = 0; k0 < 9; k0 += 2) {
        const int nk = k0 + 2 <= 9 ? 2 : 1;
        __syncthreads();
#pragma unroll
        for (int k = 0; k < nk; ++k)
#pragma unroll
            for (int m = 0; m < 4; ++m)
                *reinterpret_cast<f32x4 *>(&red[((wave * 2 + k) * 4 + m) * 256 + 4 * lane]) =
                    acc[m >> 1][m & 1][k0 + k];
        __syncthreads();
#pragma unroll
        for (int q = wave; q < nk * 4; q += NW) {
            f32x4 v = *reinterpret_cast<const f32x4 *>(&red[q * 256 + 4 * lane]);
#pragma unroll
            for (int w2 = 1; w2 < NW; ++w2)
                v += *reinterpret_cast<const f32x4 *>(&red[(w2 * 8 + q) * 256 + 4 * lane]);
            const int co = cot + 16 * (q >> 1 & 1) + (lane & 15);
            const int ci = cit + 16 * (q & 1) + 4 * g;
            *reinterpret_cast<f32x4_a4 *>(&out[((size_t)co * 9 + k0 + (q >> 2)) * Ci + ci]) = v;
        }
    }
    if (!do_bias) return;
    __syncthreads();
#pragma unroll
    for (int o = 0; o < 2; ++o)
        if ((lane & 15) == 0)
            *reinterpret_cast<f32x4 *>(&red[wave * 32 + 16 * o + 4 * g]) = bacc[o];
    __syncthreads();
    if (t < 32) {
        float v = red[t];
#pragma unroll
        for (int w2 = 1; w2 < NW; ++w2) v += red[w2 * 32 + t];
        out[tile + cot + t] = v;
    }
}

// sum_k part[k][i] over the nsplit records of n = n1 + n2 floats, written
// to out1[i] for i < n1 and to out2[i - n1] after: 64 outputs per block, GR
// groups of waves summing the splits k = g (mod GR) with four loads in
// flight each, combined in a fixed order (deterministic).  GR = 16 gives
// small layers (few outputs, many splits) more loads in flight per output.
template <int GR>
__global__ __launch_bounds__(64 * GR) void k_reduce(const float *__restrict__ part,
                                                    float *__restrict__ out1,
                                                    float *__restrict__ out2, size_t n1, size_t n,
                                                    int nsplit) {
    __shared__ float red[GR][64];
    const int lane = threadIdx.x & 63, g = threadIdx.x >> 6;
    const size_t i = (size_t)blockIdx.x * 64 + lane;
    float s0 = 0.f, s1 = 0.f, s2 = 0.f, s3 = 0.f;
    if (i < n) {
        int k = g;
        for (; k + 3 * GR < nsplit; k += 4 * GR) {
            s0 += part[(size_t)k * n + i];
            s1 += part[(size_t)(k + GR) * n + i];
            s2 += part[(size_t)(k + 2 * GR) * n + i];
            s3 += part[(size_t)(k + 3 * GR) * n + i];
        }
        if (k < nsplit) s0 += part[(size_t)k * n + i];
        if (k + GR < nsplit) s1 += part[(size_t)(k + GR) * n + i];
        if (k + 2 * GR < nsplit) s2 += part[(size_t)(k + 2 * GR) * n + i];
    }
    red[g][lane] = (s0 + s1) + (s2 + s3);
    __syncthreads();
    if (g != 0 || i >= n) return;
    float tot = red[0][lane];
#pragma unroll
    for (int v = 1; v < GR; ++v) tot += red[v][lane];
    if (i < n1)
        out1[i] = tot;
    else
        out2[i - n1] = tot;
}

// ---------------------------------------------------------------------------
// Element-wise pieces.
__global__ void k_relu_bwd(const bf16 *__restrict__ y, const bf16 *__restrict__ dy,
                           bf16 *__restrict__ dz, size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dz[i] = (float)y[i] > 0.f ? dy[i] : (bf16)0.f;
}

// 2x2 average pooling (H, W even) and its adjoint
__global__ void k_pool(const bf16 *__restrict__ x, bf16 *__restrict__ y, int N, int H, int W,
                       int C) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int Ho = H / 2, Wo = W / 2;
    if (i >= (size_t)N * Ho * Wo * C) return;
    const int c = (int)(i % C);
    size_t r = i / C;
    const int xo = (int)(r % Wo), yo = (int)((r / Wo) % Ho);
    const size_t n = r / ((size_t)Wo * Ho);
    const bf16 *p = x + ((n * H + 2 * yo) * W + 2 * xo) * C + c;
    const float s = (float)p[0] + (float)p[C] + (float)p[(size_t)W * C] + (float)p[(size_t)W * C + C];
    y[i] = (bf16)(0.25f * s);
}
__global__ void k_pool_bwd(const bf16 *__restrict__ dy, const bf16 *__restrict__ s,
                           const bf16 *__restrict__ mask, bf16 *__restrict__ dx, int N, int H, int W, int C) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)N * H * W * C) return;
    const int c = (int)(i % C);
    size_t r = i / C;
    const int xx = (int)(r % W), yy = (int)((r / W) % H);
    const size_t n = r / ((size_t)W * H);
    float v = 0.25f * (float)dy[((n * (H / 2) + yy / 2) * (W / 2) + xx / 2) * C + c];
    if (s) v += (float)s[i];
    if (mask && !((float)mask[i] > 0.f)) v = 0.f;
    dx[i] = (bf16)v;
}

// nearest 2x upsampling plus a skip: y = up(x) + s (s may be null), and the
// adjoint of the upsampling (sum of each 2x2 block)
__global__ void k_up_add(const bf16 *__restrict__ x, const bf16 *__restrict__ s,
                         bf16 *__restrict__ y, int N, int Ho, int Wo, int C) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)N * Ho * Wo * C) return;
    const int c = (int)(i % C);
    size_t r = i / C;
    const int xx = (int)(r % Wo), yy = (int)((r / Wo) % Ho);
    const size_t n = r / ((size_t)Wo * Ho);
    float v = (float)x[((n * (Ho / 2) + yy / 2) * (Wo / 2) + xx / 2) * C + c];
    if (s) v += (float)s[i];
    y[i] = (bf16)v;
}
__global__ void k_up_bwd(const bf16 *__restrict__ dy, const bf16 *__restrict__ mask,
                         bf16 *__restrict__ dx, int N, int Hi, int Wi, int C) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (size_t)N * Hi * Wi * C) return;
    const int c = (int)(i % C);
    size_t r = i / C;
    const int xx = (int)(r % Wi), yy = (int)((r / Wi) % Hi);
    const size_t n = r / ((size_t)Wi * Hi);
    const int W2 = 2 * Wi;
    const bf16 *p = dy + ((n * 2 * Hi + 2 * yy) * W2 + 2 * xx) * C + c;
    float v = (float)p[0] + (float)p[C] + (float)p[(size_t)W2 * C] + (float)p[(size_t)W2 * C + C];
    if (mask && !((float)mask[i] > 0.f)) v = 0.f;
    dx[i] = (bf16)v;
}

__global__ void k_add(const bf16 *a, const bf16 *b,
                      bf16 *y, size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) y[i] = (bf16)((float)a[i] + (float)b[i]);
}

// The same element-wise kernels on 8 channels (16 bytes) per thread, used
// when the channel count is a multiple of 8 and every operand is 16-byte
// aligned; each value is computed exactly as in the one-channel kernels.
__device__ __forceinline__ bf16x8 ld8(const bf16 *p) { return *reinterpret_cast<const bf16x8 *>(p); }
__device__ __forceinline__ void st8(bf16 *p, bf16x8 v) { *reinterpret_cast<bf16x8 *>(p) = v; }

__global__ void k_relu_bwd8(const bf16 *__restrict__ y, const bf16 *__restrict__ dy,
                            bf16 *__restrict__ dz, size_t n8) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n8) return;
    const bf16x8 a = ld8(y + 8 * i), g = ld8(dy + 8 * i);
    bf16x8 o;
#pragma unroll
    for (int k = 0; k < 8; ++k) o[k] = (float)a[k] > 0.f ? g[k] : (bf16)0.f;
    st8(dz + 8 * i, o);
}

__global__ void k_add8(const bf16 *a, const bf16 *b, bf16 *y, size_t n8) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n8) return;
    const bf16x8 u = ld8(a + 8 * i), v = ld8(b + 8 * i);
    bf16x8 o;
#pragma unroll
    for (int k = 0; k < 8; ++k) o[k] = (bf16)((float)u[k] + (float)v[k]);
    st8(y + 8 * i, o);
}

// floor(n / d) for n < 2^31 with m = floor(2^(31+s) / d) + 1, 2^(s-1) < d <= 2^s:
// m d = 2^(31+s) + e with 0 < e <= d <= 2^s, so n e < 2^(31+s) and the quotient is
// exact; m < 2^32.  From 2^31 on the plain 64-bit division.
struct Div31 {
    typedef unsigned T;
    unsigned d, m, s;
    explicit Div31(unsigned dd) : d(dd), m(0), s(0) {
        while ((1u << s) < d) ++s;
        if (s) m = (unsigned)(((uint64_t)1 << (31 + s)) / d + 1);
    }
    __device__ __forceinline__ unsigned div(unsigned n) const {
        return s ? __umulhi(n, m) >> (s - 1) : n;
    }
};
struct Div64 {
    typedef size_t T;
    unsigned d;
    explicit Div64(unsigned dd) : d(dd) {}
    __device__ __forceinline__ size_t div(size_t n) const { return n / d; }
};

// The 2 x 2 kernels below take one 8-channel piece of the coarse grid per thread:
// piece i is channel 8 c, column xo, row R of all images' rows, whose four fine
// pixels lie in the rows 2 R and 2 R + 1 of all images' rows.  All are bound by
// memory (up_add to 1024 x 2048 x 32 channels 49 us, 6.2 TB/s); four loads in
// flight and two short divisions instead of one load and five 64-bit ones matter
// where there is most to read: masked pool_bwd to 32 x 128 x 128 x 32 21.1 -> 18.6
// us, pool from there 8.2 -> 7.1.
template <class D>
struct Coarse {
    D dc, dw;
    int C8, Wo, C;
    size_t n8;
    Coarse(size_t rows, int wo, int c)
        : dc((unsigned)(c / 8)), dw((unsigned)wo), C8(c / 8), Wo(wo), C(c), n8(rows * wo * (c / 8)) {}
    // offset of the piece in the coarse tensor, and of its first fine pixel
    __device__ __forceinline__ bool at(size_t &coarse, size_t &fine) const {
        const size_t ii = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
        if (ii >= n8) return false;
        const typename D::T i = (typename D::T)ii, r = dc.div(i), R = dw.div(r);
        const int c = 8 * (int)(i - r * C8), xo = (int)(r - R * Wo);
        coarse = 8 * ii;
        fine = ((size_t)R * 4 * Wo + 2 * xo) * C + c;
        return true;
    }
    __device__ __forceinline__ size_t row() const { return (size_t)2 * Wo * C; }   // of the fine
};

template <class D>
__global__ void k_pool8(const bf16 *__restrict__ x, bf16 *__restrict__ y, Coarse<D> q) {
    size_t o, f;
    if (!q.at(o, f)) return;
    const bf16 *p = x + f, *p1 = p + q.row();
    const bf16x8 a = ld8(p), b = ld8(p + q.C), d = ld8(p1), e = ld8(p1 + q.C);
    bf16x8 v;
#pragma unroll
    for (int k = 0; k < 8; ++k)
        v[k] = (bf16)(0.25f * ((float)a[k] + (float)b[k] + (float)d[k] + (float)e[k]));
    st8(y + o, v);
}

template <class D>
__global__ void k_pool_bwd8(const bf16 *__restrict__ dy, const bf16 *__restrict__ s,
                            const bf16 *__restrict__ mask, bf16 *__restrict__ dx, Coarse<D> q) {
    size_t o, f;
    if (!q.at(o, f)) return;
    const size_t at[4] = {f, f + q.C, f + q.row(), f + q.row() + q.C};
    bf16x8 sv[4], mv[4];
    if (s)
#pragma unroll
        for (int j = 0; j < 4; ++j) sv[j] = ld8(s + at[j]);
    if (mask)
#pragma unroll
        for (int j = 0; j < 4; ++j) mv[j] = ld8(mask + at[j]);
    const bf16x8 g = ld8(dy + o);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        bf16x8 v;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            float w = 0.25f * (float)g[k];
            if (s) w += (float)sv[j][k];
            if (mask && !((float)mv[j][k] > 0.f)) w = 0.f;
            v[k] = (bf16)w;
        }
        st8(dx + at[j], v);
    }
}

template <class D>
__global__ void k_up_add8(const bf16 *__restrict__ x, const bf16 *__restrict__ s,
                          bf16 *__restrict__ y, Coarse<D> q) {
    size_t o, f;
    if (!q.at(o, f)) return;
    const size_t at[4] = {f, f + q.C, f + q.row(), f + q.row() + q.C};
    bf16x8 sv[4];
    if (s)
#pragma unroll
        for (int j = 0; j < 4; ++j) sv[j] = ld8(s + at[j]);
    const bf16x8 u = ld8(x + o);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        bf16x8 v = u;
        if (s)
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = (bf16)((float)u[k] + (float)sv[j][k]);
        st8(y + at[j], v);
    }
}

template <class D>
__global__ void k_up_bwd8(const bf16 *__restrict__ dy, const bf16 *__restrict__ mask,
                          bf16 *__restrict__ dx, Coarse<D> q) {
    size_t o, f;
    if (!q.at(o, f)) return;
    const bf16 *p = dy + f, *p1 = p + q.row();
    const bf16x8 a = ld8(p), b = ld8(p + q.C), d = ld8(p1), e = ld8(p1 + q.C);
    bf16x8 m;
    if (mask) m = ld8(mask + o);
    bf16x8 v;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        float w = (float)a[k] + (float)b[k] + (float)d[k] + (float)e[k];
        if (mask && !((float)m[k] > 0.f)) w = 0.f;
        v[k] = (bf16)w;
    }
    st8(dx + o, v);
}

// Mean squared error over the first `cout` channels of y [P][C] against
// target [P][cout] (FP32): per-block partial sums (double) and the gradient
// dy = 2 (y - t) / (P cout) (zero in the other channels).
__global__ __launch_bounds__(256) void k_mse(const bf16 *__restrict__ y,
                                             const float *__restrict__ tgt,
                                             bf16 *__restrict__ dy, double *__restrict__ partial,
                                             size_t P, int C, int cout) {
    __shared__ double red[256];
    double acc = 0.0;
    const double scale = 2.0 / ((double)P * cout);
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < P * C;
         i += (size_t)gridDim.x * blockDim.x) {
        const int c = (int)(i % C);
        const size_t p = i / C;
        float g = 0.f;
        if (c < cout) {
            const double d = (double)(float)y[i] - (double)tgt[p * cout + c];
            acc += d * d;
            g = (float)(scale * d);
        }
        if (dy) dy[i] = (bf16)g;
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// Stores the pixels w0 .. w0 + 63 (below P) of a wave, nv 16-byte pieces each:
// the first piece of pixel w0 + l is lane l's `first`, the others are zero.
// Neighbouring lanes store neighbouring pieces.
__device__ __forceinline__ void store_first_pieces(bf16 *x, int nv, size_t w0, size_t P, int lane,
                                                   uint4 first) {
    uint4 *out = reinterpret_cast<uint4 *>(x) + w0 * nv;
    const SmallDiv dv((unsigned)nv);
    for (int s = 0; s < nv; ++s) {
        const unsigned e = 64 * s + lane, px = dv.div(e);
        uint4 v;
        v.x = __shfl(first.x, px);
        v.y = __shfl(first.y, px);
        v.z = __shfl(first.z, px);
        v.w = __shfl(first.w, px);
        if (e != px * nv) v = make_uint4(0u, 0u, 0u, 0u);
        if (w0 + px < P) out[e] = v;
    }
}

// The same loss per pixel, for C a multiple of 8 and 16-byte aligned rows:
// a thread reads the cout channels of a pixel it needs and writes the whole
// dy row as 16-byte pieces (zero past cout), with no per-element division.
__global__ __launch_bounds__(256) void k_mse_px(const bf16 *__restrict__ y,
                                                const float *__restrict__ tgt,
                                                bf16 *__restrict__ dy,
                                                double *__restrict__ partial, size_t P, int C,
                                                int cout) {
    __shared__ double red[256];
    double acc = 0.0;
    const double scale = 2.0 / ((double)P * cout);
    const int nv = C / 8;
    for (size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x; p < P;
         p += (size_t)gridDim.x * blockDim.x) {
        for (int v = 0; v < nv; ++v) {
            uint4 out = make_uint4(0u, 0u, 0u, 0u);
            if (8 * v < cout) {
                unsigned short h[8];
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const int c = 8 * v + e;
                    float g = 0.f;
                    if (c < cout) {
                        const double d = (double)(float)y[p * C + c] - (double)tgt[p * cout + c];
                        acc += d * d;
                        g = (float)(scale * d);
                    }
                    const bf16 b = (bf16)g;
                    h[e] = __builtin_bit_cast(unsigned short, b);
                }
                out = make_uint4(h[0] | (unsigned)h[1] << 16, h[2] | (unsigned)h[3] << 16,
                                 h[4] | (unsigned)h[5] << 16, h[6] | (unsigned)h[7] << 16);
            }
            if (dy) *reinterpret_cast<uint4 *>(dy + p * C + 8 * v) = out;
        }
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// The same for one or two channels of few: the lanes of a wave store the pieces of
// its 64 pixels in turns (1024 x 2048 pixels, 2 of 32 channels: 77 -> 62 us).
__global__ __launch_bounds__(1024) void k_mse_first(const bf16 *__restrict__ y,
                                                    const float *__restrict__ tgt,
                                                    bf16 *__restrict__ dy,
                                                    double *__restrict__ partial, size_t P, int C,
                                                    int cout) {
    __shared__ double red[1024];
    double acc = 0.0;
    const double scale = 2.0 / ((double)P * cout);
    const int nv = C / 8, lane = threadIdx.x & 63;
    // whole waves of 64 pixels
    for (size_t p = (size_t)blockIdx.x * 1024 + threadIdx.x; p - lane < P;
         p += (size_t)gridDim.x * 1024) {
        unsigned short h[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            float g = 0.f;
            if (p < P && c < cout) {
                const double d = (double)(float)y[p * C + c] - (double)tgt[p * cout + c];
                acc += d * d;
                g = (float)(scale * d);
            }
            const bf16 b = (bf16)g;
            h[c] = __builtin_bit_cast(unsigned short, b);
        }
        if (dy)
            store_first_pieces(dy, nv, p - lane, P, lane,
                               make_uint4(h[0] | (unsigned)h[1] << 16, 0u, 0u, 0u));
    }
    red[threadIdx.x] = acc;
    __syncthreads();
    for (int s = 512; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) partial[blockIdx.x] = red[0];
}

// *out = scale * sum of the partials: 64 strided sums, then a fixed-order
// tree (deterministic)
__global__ __launch_bounds__(64) void k_sum(const double *__restrict__ partial, int n,
                                            double scale, double *__restrict__ out) {
    __shared__ double red[64];
    double a = 0.0;
    for (int i = threadIdx.x; i < n; i += 64) a += partial[i];
    red[threadIdx.x] = a;
    __syncthreads();
    for (int s = 32; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] += red[threadIdx.x + s];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = red[0] * scale;
}

// Adam on FP32 masters with a BF16 copy for the kernels (bf16 may be null).
__global__ void k_adam(float *__restrict__ w, const float *__restrict__ g, float *__restrict__ m,
                       float *__restrict__ v, bf16 *__restrict__ wb, size_t n, float lr,
                       float b1, float b2, float eps, float c1, float c2) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.f - b1) * gi;
    const float vi = b2 * v[i] + (1.f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float wi = w[i] - lr * (mi / c1) / (sqrtf(vi / c2) + eps);
    w[i] = wi;
    if (wb) wb[i] = (bf16)wi;
}

__global__ void k_to_bf16(const float *__restrict__ a, bf16 *__restrict__ b, size_t n) {
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) b[i] = (bf16)a[i];
}

// Network input / output conversion between float32 planes and NHWC bf16.
__global__ void k_pack4(const float *__restrict__ planes, const float *__restrict__ scale,
                        bf16 *__restrict__ x, int N, int H, int W, int C) {
    const size_t hw = (size_t)H * W, all = N * hw * C;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < all;
         i += (size_t)gridDim.x * blockDim.x) {
        const int c = (int)(i % C);
        const size_t p = i / C;               // pixel index n*H*W + y*W + x
        const size_t n = p / hw, q = p % hw;
        x[i] = c < 4 ? (bf16)(planes[(n * 4 + c) * hw + q] * scale[n * 4 + c]) : (bf16)0.f;
    }
}
// The same packing per pixel for C a multiple of 8 and x 16-byte aligned:
// four scaled plane values and zero padding.  Bound by the zeros it writes
// (1024 x 2048 x 32 channels: 49 us with the pixels' pieces stored by their own
// lanes, 64 bytes apart; 30 us, 5.5 TB/s, now).
__global__ __launch_bounds__(256) void k_pack4_px(const float *__restrict__ planes,
                                                  const float *__restrict__ scale,
                                                  bf16 *__restrict__ x, int N, int H, int W,
                                                  int C) {
    const int lane = threadIdx.x & 63;
    const size_t p = (size_t)blockIdx.x * 256 + threadIdx.x, w0 = p - lane;
    const size_t hw = (size_t)H * W, P = N * hw;
    uint2 v = make_uint2(0u, 0u);
    if (p < P) {
        const size_t n = P >> 32 ? p / hw : (unsigned)p / (unsigned)hw, q = p - n * hw;
        unsigned short h[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const bf16 b = (bf16)(planes[(n * 4 + c) * hw + q] * scale[n * 4 + c]);
            h[c] = __builtin_bit_cast(unsigned short, b);
        }
        v = make_uint2(h[0] | (unsigned)h[1] << 16, h[2] | (unsigned)h[3] << 16);
    }
    store_first_pieces(x, C / 8, w0, P, lane, make_uint4(v.x, v.y, 0u, 0u));
}
// One thread per pixel: a pixel's line is read once for both planes (1024 x 2048
// pixels of 32 channels: 42 us with a thread per value, 23 us now, 6.7 TB/s).
__global__ void k_unpack2(const bf16 *__restrict__ y, const float *__restrict__ scale,
                          float *__restrict__ out, int N, int H, int W, int C) {
    const size_t p = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    const size_t hw = (size_t)H * W, P = N * hw;
    if (p >= P) return;
    const size_t n = P >> 32 ? p / hw : (unsigned)p / (unsigned)hw, q = p - n * hw;
    const float a = (float)y[p * C], b = (float)y[p * C + 1];
    out[n * 2 * hw + q] = a * scale[n * 2];
    out[(n * 2 + 1) * hw + q] = b * scale[n * 2 + 1];
}

unsigned blocks_for(size_t n) { return (unsigned)((n + 255) / 256); }

int status(hipError_t e) { return e == hipSuccess ? FWI_NN_OK : FWI_NN_EHIP; }

bool al16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; }

template <class F>
void launch2x2(size_t rows, int wo, int C, F launch) {
    if (rows * wo * (C / 8) < (size_t)1 << 31)
        launch(Coarse<Div31>(rows, wo, C));
    else
        launch(Coarse<Div64>(rows, wo, C));
}

// the convolution, and with a mask zero where that is not positive
int conv3x3(const void *x, const void *w, const float *bias, const void *mask, void *y, int32_t N,
            int32_t H, int32_t W, int32_t Ci, int32_t Co, int32_t relu, void *stream) {
    if (!x || !w || !y || N < 1 || H < 1 || W < 1 || H > 32768 || W > 32768 || Ci < 32 ||
        Co < 32 || Ci % 32 || Co % 32 || !al16(x) || !al16(w))
        return FWI_NN_EINVAL;
    if ((int64_t)N * H * W >= (int64_t)1 << 36) return FWI_NN_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int64_t P = (int64_t)N * H * W;
    const bf16 *xb = static_cast<const bf16 *>(x);
    const bf16 *wb = static_cast<const bf16 *>(w);
    const bf16 *mb = static_cast<const bf16 *>(mask);
    bf16 *yb = static_cast<bf16 *>(y);
    const bool aligned8 =
        ((reinterpret_cast<uintptr_t>(y) | reinterpret_cast<uintptr_t>(mask)) & 7) == 0;
    const fwi_nn::ConvRoute route = fwi_nn::conv_route(N, H, W, Ci, Co, aligned8);
    if (route.kernel == fwi_nn::ConvRoute::Rows) {
        auto run = [&](auto f) { return f(xb, wb, bias, mb, yb, N, H, W, Co, relu, route, st); };
        const bool co64 = Co % 64 == 0;
        if (Ci == 32) return status(run(co64 ? launch_rows<32, 2, 2, 2> : launch_rows<32, 2, 1, 4>));
        if (Ci == 128)
            return status(run(co64 ? launch_rows<128, 1, 4, 1> : launch_rows<128, 1, 2, 2>));
        if (Co % 128 == 0) return status(run(launch_rows<64, 2, 4, 1>));
        return status(run(co64 ? launch_rows<64, 2, 2, 2> : launch_rows<64, 2, 1, 4>));
    }
    if (route.kernel == fwi_nn::ConvRoute::Lds) {
        // 64-pixel blocks where 128-pixel blocks would leave fewer than two blocks
        // per CU (below 1024 blocks of 128 they made the network's 32 x 32-pixel
        // layers slower)
        const int bn = route.bn;
        const int64_t lds_blocks = (P + 127) / 128 * (Co / bn);
        const int bm = lds_blocks < 512 ? 64 : 128;
        const dim3 grid((unsigned)((P + bm - 1) / bm), (unsigned)(Co / bn));
        // (the mask's test at run time cost the calls without one 3 to 5%)
        auto kernel = bn == 64 ? (bm == 128 ? (mb ? k_conv3x3_lds<64, 128, true>
                                                  : k_conv3x3_lds<64, 128, false>)
                                            : (mb ? k_conv3x3_lds<64, 64, true>
                                                  : k_conv3x3_lds<64, 64, false>))
                               : (bm == 128 ? (mb ? k_conv3x3_lds<32, 128, true>
                                                  : k_conv3x3_lds<32, 128, false>)
                                            : (mb ? k_conv3x3_lds<32, 64, true>
                                                  : k_conv3x3_lds<32, 64, false>));
        hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, xb, wb, bias, mb, yb, N, H, W, Ci, Co,
                           relu);
        return status(hipGetLastError());
    }
    // small layers: 64-pixel blocks of 32-channel tiles (four times the
    // blocks of the LDS tiling)
    const dim3 grid((unsigned)((P + 63) / 64), (unsigned)(Co / 32));
    auto kernel = mb ? k_conv3x3<2, 1, true> : k_conv3x3<2, 1, false>;
    hipLaunchKernelGGL(kernel, grid, dim3(256), 0, st, xb, wb, bias, mb, yb, N, H, W, Ci, Co, relu);
    return status(hipGetLastError());
}

int pool2_bwd(const void *dy, const void *skip, const void *mask, void *dx, int32_t N, int32_t H,
              int32_t W, int32_t C, void *stream) {
    if (!dy || !dx || N < 1 || H < 2 || W < 2 || H % 2 || W % 2 || C < 1) return FWI_NN_EINVAL;
    const size_t n = (size_t)N * H * W * C;
    const bf16 *sb = static_cast<const bf16 *>(skip), *mb = static_cast<const bf16 *>(mask);
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (C % 8 == 0 && al16(dy) && al16(dx) && (!skip || al16(skip)) && (!mask || al16(mask)))
        launch2x2((size_t)N * (H / 2), W / 2, C, [&](auto q) {
            hipLaunchKernelGGL(k_pool_bwd8<decltype(q.dc)>, dim3(blocks_for(q.n8)), dim3(256), 0, st,
                               static_cast<const bf16 *>(dy), sb, mb, static_cast<bf16 *>(dx), q);
        });
    else
        hipLaunchKernelGGL(k_pool_bwd, dim3(blocks_for(n)), dim3(256), 0,
                           st, static_cast<const bf16 *>(dy), sb, mb,
                           static_cast<bf16 *>(dx), N, H, W, C);
    return status(hipGetLastError());
}

int up2_bwd(const void *dy, const void *mask, void *dx, int32_t N, int32_t Hi, int32_t Wi,
            int32_t C, void *stream) {
    if (!dy || !dx || N < 1 || Hi < 1 || Wi < 1 || C < 1) return FWI_NN_EINVAL;
    const size_t n = (size_t)N * Hi * Wi * C;
    const bf16 *mb = static_cast<const bf16 *>(mask);
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (C % 8 == 0 && al16(dy) && al16(dx) && (!mask || al16(mask)))
        launch2x2((size_t)N * Hi, Wi, C, [&](auto q) {
            hipLaunchKernelGGL(k_up_bwd8<decltype(q.dc)>, dim3(blocks_for(q.n8)), dim3(256), 0, st,
                               static_cast<const bf16 *>(dy), mb, static_cast<bf16 *>(dx), q);
        });
    else
        hipLaunchKernelGGL(k_up_bwd, dim3(blocks_for(n)), dim3(256), 0,
                           st, static_cast<const bf16 *>(dy), mb,
                           static_cast<bf16 *>(dx), N, Hi, Wi, C);
    return status(hipGetLastError());
}

}  // namespace

extern "C" {

int fwi_nn_conv3x3(const void *x, const void *w, const float *bias, void *y, int32_t N,
                   int32_t H, int32_t W, int32_t Ci, int32_t Co, int32_t relu, void *stream) {
    return conv3x3(x, w, bias, nullptr, y, N, H, W, Ci, Co, relu, stream);
}

int fwi_nn_conv3x3_masked(const void *x, const void *w, const void *mask, void *y, int32_t N,
                          int32_t H, int32_t W, int32_t Ci, int32_t Co, void *stream) {
    if (!mask) return FWI_NN_EINVAL;
    return conv3x3(x, w, nullptr, mask, y, N, H, W, Ci, Co, 0, stream);
}

int fwi_nn_flip(const void *w, void *wf, int32_t Ci, int32_t Co, void *stream) {
    if (!w || !wf || Ci < 1 || Co < 1) return FWI_NN_EINVAL;
    const size_t n = (size_t)Co * 9 * Ci;
    hipLaunchKernelGGL(k_flip, dim3(blocks_for(n)), dim3(256), 0, static_cast<hipStream_t>(stream),
                       static_cast<const bf16 *>(w), static_cast<bf16 *>(wf), Ci, Co);
    return status(hipGetLastError());
}

int fwi_nn_flip_layers(const void *w, void *wf, int32_t nlayers, const int64_t *off,
                       const int32_t *ci, const int32_t *co, void *stream) {
    if (!w || !wf || !off || !ci || !co || nlayers < 1 || nlayers > kFlipMax)
        return FWI_NN_EINVAL;
    FlipTable tb{};
    tb.n = nlayers;
    int64_t end = 0, tiles = 0;
    for (int l = 0; l < nlayers; ++l) {
        if (off[l] < end || ci[l] < 1 || co[l] < 1 || (int64_t)9 * ci[l] * co[l] >= (1ll << 31))
            return FWI_NN_EINVAL;
        tb.off[l] = off[l];
        tb.ci[l] = ci[l];
        tb.co[l] = co[l];
        end = off[l] + (int64_t)9 * ci[l] * co[l];
        tb.tile0[l + 1] = tiles += (int64_t)9 * ((ci[l] + 31) / 32) * ((co[l] + 31) / 32);
    }
    hipLaunchKernelGGL(k_flip_layers, dim3((unsigned)std::min<int64_t>(tiles, 1 << 16)), dim3(256), 0,
                       static_cast<hipStream_t>(stream), static_cast<const bf16 *>(w),
                       static_cast<bf16 *>(wf), tb);
    return status(hipGetLastError());
}

size_t fwi_nn_wgrad_workspace(int32_t Ci, int32_t Co, int32_t nsplit) {
    return ((size_t)nsplit * Co * 9 * Ci + (size_t)nsplit * Co) * sizeof(float);
}

int fwi_nn_wgrad(const void *x, const void *dz, float *dw, float *db, int32_t N, int32_t H,
                 int32_t W, int32_t Ci, int32_t Co, int32_t nsplit, void *ws, size_t ws_bytes,
                 void *stream) {
    if (!x || !dz || !dw || !db || !ws || N < 1 || H < 1 || W < 1 || H > 32768 || W > 32768 ||
        Ci < 32 || Co < 32 ||
        Ci % 32 || Co % 32 || nsplit < 1 || nsplit > 65535 || !al16(x) || !al16(dz) ||
        (int64_t)N * H * W >= (int64_t)1 << 36 ||
        ws_bytes < fwi_nn_wgrad_workspace(Ci, Co, nsplit))
        return FWI_NN_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    float *part = static_cast<float *>(ws);
    const int tiles = (Co / 32) * (Ci / 32);
    const fwi_nn::WgradRoute r = fwi_nn::wgrad_route(N, H, W, Ci, Co, nsplit);
    nsplit = r.records;
    if (r.waves == 0)
        hipLaunchKernelGGL(k_wgrad<kWgradChunk>, dim3(nsplit, tiles), dim3(256), 0, st,
                           static_cast<const bf16 *>(x), static_cast<const bf16 *>(dz), part, N, H,
                           W, Ci, Co);
    else if (r.waves == 8)
        hipLaunchKernelGGL(k_wgrad_rows<8>, dim3(nsplit, tiles), dim3(512), 0, st,
                           static_cast<const bf16 *>(x), static_cast<const bf16 *>(dz), part, N, H,
                           W, Ci, Co, r.plan.strip, r.plan.nstrip, r.plan.srow);
    else
        hipLaunchKernelGGL(k_wgrad_rows<4>, dim3(nsplit, tiles), dim3(256), 0, st,
                           static_cast<const bf16 *>(x), static_cast<const bf16 *>(dz), part, N, H,
                           W, Ci, Co, r.plan.strip, r.plan.nstrip, r.plan.srow);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return FWI_NN_EHIP;
    const size_t nw = (size_t)Co * 9 * Ci, n = nw + Co;
    const unsigned nb = (unsigned)((n + 63) / 64);
    // sixteen wave groups where the outputs give fewer than 1024 blocks
    if (nb < 1024)
        hipLaunchKernelGGL(k_reduce<16>, dim3(nb), dim3(1024), 0, st, part, dw, db, nw, n, nsplit);
    else
        hipLaunchKernelGGL(k_reduce<4>, dim3(nb), dim3(256), 0, st, part, dw, db, nw, n, nsplit);
    return status(hipGetLastError());
}

int fwi_nn_relu_bwd(const void *y, const void *dy, void *dz, size_t n, void *stream) {
    if (!y || !dy || !dz) return FWI_NN_EINVAL;
    if (n == 0) return FWI_NN_OK;
    if (n % 8 == 0 && al16(y) && al16(dy) && al16(dz))
        hipLaunchKernelGGL(k_relu_bwd8, dim3(blocks_for(n / 8)), dim3(256), 0,
                           static_cast<hipStream_t>(stream), static_cast<const bf16 *>(y),
                           static_cast<const bf16 *>(dy), static_cast<bf16 *>(dz), n / 8);
    else
        hipLaunchKernelGGL(k_relu_bwd, dim3(blocks_for(n)), dim3(256), 0,
                           static_cast<hipStream_t>(stream), static_cast<const bf16 *>(y),
                           static_cast<const bf16 *>(dy), static_cast<bf16 *>(dz), n);
    return status(hipGetLastError());
}

int fwi_nn_pool2(const void *x, void *y, int32_t N, int32_t H, int32_t W, int32_t C, void *stream) {
    if (!x || !y || N < 1 || H < 2 || W < 2 || H % 2 || W % 2 || C < 1) return FWI_NN_EINVAL;
    const size_t n = (size_t)N * (H / 2) * (W / 2) * C;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (C % 8 == 0 && al16(x) && al16(y))
        launch2x2((size_t)N * (H / 2), W / 2, C, [&](auto q) {
            hipLaunchKernelGGL(k_pool8<decltype(q.dc)>, dim3(blocks_for(q.n8)), dim3(256), 0, st,
                               static_cast<const bf16 *>(x), static_cast<bf16 *>(y), q);
        });
    else
        hipLaunchKernelGGL(k_pool, dim3(blocks_for(n)), dim3(256), 0,
                           st, static_cast<const bf16 *>(x),
                           static_cast<bf16 *>(y), N, H, W, C);
    return status(hipGetLastError());
}

int fwi_nn_pool2_bwd_add(const void *dy, const void *skip, void *dx, int32_t N, int32_t H,
                         int32_t W, int32_t C, void *stream) {
    return pool2_bwd(dy, skip, nullptr, dx, N, H, W, C, stream);
}

int fwi_nn_pool2_bwd_masked(const void *dy, const void *skip, const void *mask, void *dx,
                            int32_t N, int32_t H, int32_t W, int32_t C, void *stream) {
    if (!mask) return FWI_NN_EINVAL;
    return pool2_bwd(dy, skip, mask, dx, N, H, W, C, stream);
}

int fwi_nn_pool2_bwd(const void *dy, void *dx, int32_t N, int32_t H, int32_t W, int32_t C,
                     void *stream) {
    return fwi_nn_pool2_bwd_add(dy, nullptr, dx, N, H, W, C, stream);
}

int fwi_nn_up2_add(const void *x, const void *skip, void *y, int32_t N, int32_t Ho, int32_t Wo,
                   int32_t C, void *stream) {
    if (!x || !y || N < 1 || Ho < 2 || Wo < 2 || Ho % 2 || Wo % 2 || C < 1) return FWI_NN_EINVAL;
    const size_t n = (size_t)N * Ho * Wo * C;
    hipStream_t st = static_cast<hipStream_t>(stream);
    if (C % 8 == 0 && al16(x) && al16(y) && (!skip || al16(skip)))
        launch2x2((size_t)N * (Ho / 2), Wo / 2, C, [&](auto q) {
            hipLaunchKernelGGL(k_up_add8<decltype(q.dc)>, dim3(blocks_for(q.n8)), dim3(256), 0, st,
                               static_cast<const bf16 *>(x),
                               static_cast<const bf16 *>(skip), static_cast<bf16 *>(y), q);
        });
    else
        hipLaunchKernelGGL(k_up_add, dim3(blocks_for(n)), dim3(256), 0,
                           st, static_cast<const bf16 *>(x),
                           static_cast<const bf16 *>(skip), static_cast<bf16 *>(y), N, Ho, Wo, C);
    return status(hipGetLastError());
}

int fwi_nn_up2_bwd(const void *dy, void *dx, int32_t N, int32_t Hi, int32_t Wi, int32_t C,
                   void *stream) {
    return up2_bwd(dy, nullptr, dx, N, Hi, Wi, C, stream);
}

int fwi_nn_up2_bwd_masked(const void *dy, const void *mask, void *dx, int32_t N, int32_t Hi,
                          int32_t Wi, int32_t C, void *stream) {
    if (!mask) return FWI_NN_EINVAL;
    return up2_bwd(dy, mask, dx, N, Hi, Wi, C, stream);
}

int fwi_nn_add(const void *a, const void *b, void *y, size_t n, void *stream) {
    if (!a || !b || !y) return FWI_NN_EINVAL;
    if (n == 0) return FWI_NN_OK;
    if (n % 8 == 0 && al16(a) && al16(b) && al16(y))
        hipLaunchKernelGGL(k_add8, dim3(blocks_for(n / 8)), dim3(256), 0,
                           static_cast<hipStream_t>(stream), static_cast<const bf16 *>(a),
                           static_cast<const bf16 *>(b), static_cast<bf16 *>(y), n / 8);
    else
        hipLaunchKernelGGL(k_add, dim3(blocks_for(n)), dim3(256), 0,
                           static_cast<hipStream_t>(stream), static_cast<const bf16 *>(a),
                           static_cast<const bf16 *>(b), static_cast<bf16 *>(y), n);
    return status(hipGetLastError());
}

int fwi_nn_mse(const void *y, const float *target, void *dy, double *loss, double *partials,
               size_t P, int32_t C, int32_t cout, void *stream) {
    if (!y || !target || !loss || !partials || P == 0 || C < 1 || cout < 1 || cout > C)
        return FWI_NN_EINVAL;
    hipStream_t st = static_cast<hipStream_t>(stream);
    // (of more channels, or more of them in the loss, the pieces' own thread is
    // faster: 8 of 32, 32 x 128 x 128 pixels: 48.8 and 30.4 us; 2 of 256, 7 x 34 x
    // 30: 13.4 and 11.4; 2 of 128, 32 x 32 x 32: 11.6 and 11.8)
    if (C % 8 == 0 && C <= 128 && cout <= 2 && (!dy || al16(dy)))
        hipLaunchKernelGGL(k_mse_first, dim3(FWI_NN_MSE_BLOCKS), dim3(1024), 0, st,
                           static_cast<const bf16 *>(y), target, static_cast<bf16 *>(dy), partials,
                           P, C, cout);
    else if (C % 8 == 0 && (!dy || al16(dy)))
        hipLaunchKernelGGL(k_mse_px, dim3(FWI_NN_MSE_BLOCKS), dim3(256), 0, st,
                           static_cast<const bf16 *>(y), target, static_cast<bf16 *>(dy), partials,
                           P, C, cout);
    else
        hipLaunchKernelGGL(k_mse, dim3(FWI_NN_MSE_BLOCKS), dim3(256), 0, st,
                           static_cast<const bf16 *>(y), target, static_cast<bf16 *>(dy), partials,
                           P, C, cout);
    hipLaunchKernelGGL(k_sum, dim3(1), dim3(64), 0, st, partials, FWI_NN_MSE_BLOCKS,
                       1.0 / ((double)P * cout), loss);
    return status(hipGetLastError());
}

int fwi_nn_adam(float *w, const float *g, float *m, float *v, void *wb, size_t n, float lr,
                float beta1, float beta2, float eps, int32_t step, void *stream) {
    if (!w || !g || !m || !v || step < 1) return FWI_NN_EINVAL;
    if (n == 0) return FWI_NN_OK;
    const float c1 = 1.f - powf(beta1, (float)step), c2 = 1.f - powf(beta2, (float)step);
    hipLaunchKernelGGL(k_adam, dim3(blocks_for(n)), dim3(256), 0, static_cast<hipStream_t>(stream),
                       w, g, m, v, static_cast<bf16 *>(wb), n, lr, beta1, beta2, eps, c1, c2);
    return status(hipGetLastError());
}

int fwi_nn_to_bf16(const float *a, void *b, size_t n, void *stream) {
    if (!a || !b) return FWI_NN_EINVAL;
    if (n == 0) return FWI_NN_OK;
    hipLaunchKernelGGL(k_to_bf16, dim3(blocks_for(n)), dim3(256), 0,
                       static_cast<hipStream_t>(stream), a, static_cast<bf16 *>(b), n);
    return status(hipGetLastError());
}

int fwi_nn_pack4(const float *planes, const float *scale, void *x, int32_t N, int32_t H,
                 int32_t W, int32_t C, void *stream) {
    if (!planes || !scale || !x || N < 1 || H < 1 || W < 1 || C < 4) return FWI_NN_EINVAL;
    const size_t n = (size_t)N * H * W * C;
    // past 2048 channels a thread per value: a wave would store its pixels' pieces
    // one after another (2 x 2 pixels of 65536 channels: 554 and 7.5 us), and its
    // piece indices outgrow the short division
    if (C % 8 == 0 && C <= 2048 && al16(x))
        hipLaunchKernelGGL(k_pack4_px, dim3(blocks_for((size_t)N * H * W)), dim3(256), 0,
                           static_cast<hipStream_t>(stream), planes, scale,
                           static_cast<bf16 *>(x), N, H, W, C);
    else
        hipLaunchKernelGGL(k_pack4, dim3(std::min(blocks_for(n), 1u << 22)), dim3(256), 0,
                           static_cast<hipStream_t>(stream), planes, scale,
                           static_cast<bf16 *>(x), N, H, W, C);
    return status(hipGetLastError());
}

int fwi_nn_unpack2(const void *y, const float *scale, float *out, int32_t N, int32_t H,
                   int32_t W, int32_t C, void *stream) {
    if (!y || !scale || !out || N < 1 || H < 1 || W < 1 || C < 2) return FWI_NN_EINVAL;
    const size_t n = (size_t)N * H * W;
    hipLaunchKernelGGL(k_unpack2, dim3(blocks_for(n)), dim3(256), 0,
                       static_cast<hipStream_t>(stream), static_cast<const bf16 *>(y), scale, out,
                       N, H, W, C);
    return status(hipGetLastError());
}

}  // extern "C"
