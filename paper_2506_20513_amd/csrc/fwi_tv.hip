// Total-variation regularisation term (Sec. 3.4, Algorithm 3): a
// split-Bregman iteration of TV denoising per field, its result turned into
// the gradient term weight * (X - s U).  The operation is documented in
// include/fwi_tv.h.
//
// Iteration t takes U_t and the multipliers B_{t-1} to B_t and U_{t+1}: with
// W = D U_t + B_{t-1},
//   Z_t = shrink(W, 1/lam),  B_t = W - Z_t,  P = Z_t - B_t = 2 Z_t - W,
//   U_{t+1} = (mu Xn + lam D^T P + lam (4 U_t + neighbours)) / (mu + 8 lam),
// so Z is never stored.  Arrays are row-major [nfield][ny][nx].
//
// Several iterations per launch on tiles: a workgroup holds a tile of 64
// columns (lane = column) x NW R rows of one field with a halo of D cells on
// every side in registers, R consecutive rows per wave, runs up to D
// iterations and writes the inner part.  Per iteration the waves exchange
// their first and last rows of U through LDS, with one barrier; the multipliers
// of the row above a wave's rows are carried along by it too.  The fields are
// periodic, so a tile reads its halo at wrapped indices and needs no other
// boundary case.  With one thread per cell and one launch per iteration the
// shrink of a cell was evaluated three times (for itself and for its right and
// lower neighbour) and 28 bytes per cell moved every iteration: 50 iterations on
// two 1064 x 2088 fields took 1.48 ms, 20 on two 128 x 128 fields 92 us.  Now
// 0.54 ms, bound by the vector instructions (about 45 per cell and iteration,
// 1.6 times for the halo: 0.40 ms at the full rate), and 27 us, bound by three
// launches and the serial iterations of a tile.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>

#include "fwi_tv.h"

namespace {

constexpr int kMaxBlocks = 1024;   // partial maxima per field
constexpr size_t kAlign = 256;

struct TvParams {
    float mu[FWI_TV_MAX_FIELDS];      // both times a power of two (see fwi_tv_gradient)
    float lam[FWI_TV_MAX_FIELDS];
    float t[FWI_TV_MAX_FIELDS];       // 1 / lam of the caller
    float weight[FWI_TV_MAX_FIELDS];
};

size_t up(size_t n) { return (n + kAlign - 1) / kAlign * kAlign; }

struct Layout {
    size_t u[2], bx[2], by[2], part, scale, total;
};

Layout layout(int nfield, int ny, int nx) {
    const size_t field = up((size_t)nfield * ny * nx * sizeof(float));
    Layout L;
    size_t o = 0;
    for (int k = 0; k < 2; ++k) { L.u[k] = o; o += field; }
    for (int k = 0; k < 2; ++k) { L.bx[k] = o; o += field; }
    for (int k = 0; k < 2; ++k) { L.by[k] = o; o += field; }
    L.part = o;
    o += up((size_t)nfield * kMaxBlocks * sizeof(float));
    L.scale = o;
    o += up((size_t)nfield * sizeof(float));
    L.total = o;
    return L;
}

__global__ __launch_bounds__(256) void k_absmax(const float *__restrict__ X,
                                                float *__restrict__ part, size_t n) {
    __shared__ float red[256];
    const float *x = X + (size_t)blockIdx.y * n;
    float m = 0.f;
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256)
        m = fmaxf(m, fabsf(x[i]));
    red[threadIdx.x] = m;
    __syncthreads();
    for (int s = 128; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + s]);
        __syncthreads();
    }
    if (threadIdx.x == 0) part[(size_t)blockIdx.y * kMaxBlocks + blockIdx.x] = red[0];
}

// The largest of a field's nb partial maxima (all threads of the workgroup).
template <int NT>
__device__ __forceinline__ float largest(const float *__restrict__ part, int nb, float *red) {
    static_assert((NT & (NT - 1)) == 0, "the tree halves the threads");
    float m = 0.f;
    for (int i = threadIdx.x; i < nb; i += NT) m = fmaxf(m, part[i]);
    red[threadIdx.x] = m;
    __syncthreads();
    for (int s = NT / 2; s > 0; s >>= 1) {
        if ((int)threadIdx.x < s) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + s]);
        __syncthreads();
    }
    return red[0];
}

// i modulo n, for any i
__device__ __forceinline__ int wrap(int i, int n) {
    i %= n;
    return i < 0 ? i + n : i;
}

// lane i receives the value of lane i + 1 / i - 1 (the last / first lane 0)
__device__ __forceinline__ float from_right(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, false));
}
__device__ __forceinline__ float from_left(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, false));
}

// n / d given rd = 1 / d rounded to nearest: one correction of n rd by the
// residual of the quotient, which gives the correctly rounded quotient (up to
// its last bit for the one significand of d with all bits set) in three
// operations instead of the ten of a division.
__device__ __forceinline__ float div_by(float n, float d, float rd) {
    const float q = n * rd;
    return fmaf(fmaf(-q, d, n), rd, q);
}

// 2 shrink(w, t) - w for both components (t = 1/lam), and B = w - shrink(w, t).
// The magnitude and the quotient (mag - t) / mag both start from one reciprocal
// square root and are corrected by their residuals, to within half a unit in
// the last place and a little (the library's sqrt and division together take
// three times the operations).  The smallest normal number in place of a
// smaller square keeps the reciprocal finite: such a w, below 1.1e-19 of the
// field's largest value, is below every t of a lam up to 9e18.
__device__ __forceinline__ void bregman(float wx, float wy, float t, float &px, float &py,
                                        float &bx, float &by) {
    const float m2 = fmaxf(fmaf(wx, wx, wy * wy), 1.17549435e-38f);
    const float r = __builtin_amdgcn_rsqf(m2);
    const float m0 = m2 * r;
    const float mag = fmaf(fmaf(-m0, m0, m2), 0.5f * r, m0);
    const float d = mag - t;
    const float q = d * r;
    const float f = mag > t ? fmaf(fmaf(-q, mag, d), r, q) : 0.f;
    const float zx = wx * f, zy = wy * f;
    bx = wx - zx;
    by = wy - zy;
    px = zx - bx;
    py = zy - by;
}

__device__ __forceinline__ float add_term(float g, float x, float s, float u, float weight) {
    return g + weight * (x - s * u);
}

// nit <= D iterations.  `first`: from U_0 = X / s and B = 0, with s from the
// partial maxima (stored for the later launches); `last`: the term goes to grad
// in place of U and B.
template <int D, int R, int NW>
__global__ __launch_bounds__(64 * NW) void k_tv_tile(
    const float *__restrict__ X, const float *__restrict__ part, int nb,
    float *__restrict__ scale, const float *__restrict__ U, const float *__restrict__ Bx,
    const float *__restrict__ By, float *__restrict__ Uo, float *__restrict__ Bxo,
    float *__restrict__ Byo, float *__restrict__ grad, int ny, int nx, TvParams p, int nit,
    int first, int last) {
    constexpr int OX = 64 - 2 * D, OY = NW * R - 2 * D;
    __shared__ float xch[2][NW][2][64];
    __shared__ float red[64 * NW];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int f = blockIdx.z;
    float s;
    if (first) {
        s = largest<64 * NW>(part + (size_t)f * kMaxBlocks, nb, red);
        if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) scale[f] = s;
    } else {
        s = scale[f];
    }
    if (s == 0.f) return;                // all-zero field: its term is zero
    const float inv = 1.f / s, mu = p.mu[f], lam = p.lam[f], t = p.t[f];
    const float den = mu + 8.f * lam, rden = 1.f / den;
    const size_t off = (size_t)f * ny * nx;
    const int x0 = (int)blockIdx.x * OX - D, y0 = (int)blockIdx.y * OY - D;
    const int j0 = y0 + wave * R;        // the wave's rows
    const int col = wrap(x0 + lane, nx);
    float u[R], bx[R], by[R], x[R];       // x: X / s
    float bxu = 0.f, byu = 0.f;          // multipliers of the row above
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const size_t c = off + (size_t)wrap(j0 + r, ny) * nx + col;
        x[r] = X[c] * inv;
        bx[r] = by[r] = 0.f;
        if (!first) {
            u[r] = U[c];
            bx[r] = Bx[c];
            by[r] = By[c];
        }
    }
    if (!first) {
        const size_t c = off + (size_t)wrap(j0 - 1, ny) * nx + col;
        bxu = Bx[c];
        byu = By[c];
    }
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (first) u[r] = x[r];
    for (int k = 0; k < nit; ++k) {
        const int b = k & 1;
        xch[b][wave][0][lane] = u[0];
        xch[b][wave][1][lane] = u[R - 1];
        __syncthreads();
        const float uup = wave > 0 ? xch[b][wave - 1][1][lane] : 0.f;
        const float udn = wave < NW - 1 ? xch[b][wave + 1][0][lane] : 0.f;
        const bool start = first && k == 0;          // Z = B = 0
        float pyu = 0.f;                             // P_y of the row above
        if (!start) {
            float px;
            bregman(from_right(uup) - uup + bxu, u[0] - uup + byu, t, px, pyu, bxu, byu);
        }
        float up = uup;                              // U_t of the row above
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float uc = u[r], ud = r + 1 < R ? u[r + 1 < R ? r + 1 : r] : udn;
            const float ur = from_right(uc), ul = from_left(uc);
            float px = 0.f, py = 0.f;
            if (!start) bregman(ur - uc + bx[r], ud - uc + by[r], t, px, py, bx[r], by[r]);
            const float dtp = -((px - from_left(px)) + (py - pyu));        // D^T P
            u[r] = div_by(mu * x[r] + lam * dtp + lam * (4.f * uc + ul + ur + up + ud), den, rden);
            up = uc;
            pyu = py;
        }
    }
    const bool own = lane >= D && lane < 64 - D && x0 + lane < nx;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int tr = wave * R + r, j = j0 + r;
        if (tr < D || tr >= D + OY || j >= ny || !own) continue;
        const size_t c = off + (size_t)j * nx + x0 + lane;
        if (last) {
            grad[c] = add_term(grad[c], X[c], s, u[r], p.weight[f]);
        } else {
            Uo[c] = u[r];
            Bxo[c] = bx[r];
            Byo[c] = by[r];
        }
    }
}

// The term for a grad that shares memory with X: the last tile launch reads X
// over its tiles' halos, which neighbouring tiles must not have overwritten, so it
// stores U instead and this one reads and writes each cell once (no __restrict__).
__global__ __launch_bounds__(256) void k_tv_term(const float *X, const float *scale,
                                                 const float *U, float *grad, size_t n,
                                                 TvParams p) {
    const int f = blockIdx.y;
    const float s = scale[f];
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (s == 0.f || i >= n) return;      // all-zero field: its term is zero
    const size_t c = f * n + i;
    grad[c] = add_term(grad[c], X[c], s, U[c], p.weight[f]);
}

template <int D, int R, int NW>
void run_tiles(const float *X, float *grad, int nfield, int ny, int nx, const TvParams &p,
               int iters, const Layout &L, char *w, int nb, hipStream_t st) {
    constexpr int OX = 64 - 2 * D, OY = NW * R - 2 * D;
    auto F = [&](size_t o) { return reinterpret_cast<float *>(w + o); };
    const dim3 grid((nx + OX - 1) / OX, (ny + OY - 1) / OY, nfield);
    const size_t n = (size_t)ny * nx;
    const uintptr_t a = reinterpret_cast<uintptr_t>(X), b = reinterpret_cast<uintptr_t>(grad);
    const bool shared = (a < b ? b - a : a - b) < nfield * n * sizeof(float);
    int k = 0;
    for (int t = 0; t < iters; t += D, k ^= 1) {
        const int nit = std::min(D, iters - t);
        hipLaunchKernelGGL((k_tv_tile<D, R, NW>), grid, dim3(64 * NW), 0, st, X, F(L.part), nb,
                           F(L.scale), F(L.u[k]), F(L.bx[k]), F(L.by[k]), F(L.u[k ^ 1]),
                           F(L.bx[k ^ 1]), F(L.by[k ^ 1]), grad, ny, nx, p, nit, t == 0,
                           t + nit == iters && !shared);
    }
    if (shared)
        hipLaunchKernelGGL(k_tv_term, dim3((unsigned)((n + 255) / 256), nfield), dim3(256), 0, st,
                           X, F(L.scale), F(L.u[k]), grad, n, p);
}

}  // namespace

extern "C" {

size_t fwi_tv_workspace_bytes(int32_t nfield, int32_t ny, int32_t nx) {
    if (nfield < 1 || nfield > FWI_TV_MAX_FIELDS || ny < 2 || nx < 2 ||
        (int64_t)ny * nx >= ((int64_t)1 << 31))
        return 0;
    return layout(nfield, ny, nx).total;
}

int fwi_tv_gradient(const float *X, float *grad, int32_t nfield, int32_t ny, int32_t nx,
                    const float *mu, const float *lam, const float *weight, int32_t iters,
                    void *ws, size_t ws_bytes, void *stream) {
    if (!X || !grad || !mu || !lam || !weight || nfield < 1 || nfield > FWI_TV_MAX_FIELDS ||
        ny < 2 || nx < 2 || (int64_t)ny * nx >= ((int64_t)1 << 31) || iters < 1)
        return -1;
    TvParams p{};
    for (int f = 0; f < nfield; ++f) {
        if (!(mu[f] > 0.f) || !(lam[f] > 0.f)) return -1;
        // The U update is a ratio, homogeneous in mu and lam.  Where mu + 8 lam or
        // its reciprocal could leave the normal numbers, both are scaled into them.
        const float m = std::max(mu[f], lam[f]);
        const int e = !std::isfinite(m) ? 0 : m > 0x1p100f ? -100 : m < 0x1p-100f ? 100 : 0;
        p.mu[f] = std::ldexp(mu[f], e);
        p.lam[f] = std::ldexp(lam[f], e);
        p.t[f] = 1.f / lam[f];
        p.weight[f] = weight[f];
    }
    const Layout L = layout(nfield, ny, nx);
    if (!ws || (reinterpret_cast<uintptr_t>(ws) % kAlign) != 0 || ws_bytes < L.total) return -4;
    char *w = static_cast<char *>(ws);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const size_t n = (size_t)ny * nx;
    const int nb = (int)std::min<size_t>(kMaxBlocks, (n + 255) / 256);
    hipLaunchKernelGGL(k_absmax, dim3(nb, nfield), dim3(256), 0, st, X,
                       reinterpret_cast<float *>(w + L.part), n);
    // Few cells: a deep halo, for fewer launches; many: a thin one, for less
    // recomputation (10 iterations on 32 and 48 rows, 5 on 40).  Measured, us
    // per call of 20 to 50 iterations, in that order: 2 x 128 x 128: 28, 35, 33;
    // 81 x 1258: 42, 51, 45; 2 x 256 x 512: 56, 41, 51; 2 x 500 x 700: 104, 122,
    // 100; and for the last kind against 4
    // iterations on 64 rows 2 x 1064 x 2088: 535 against 651.
    const size_t cells = (size_t)nfield * n;
    // Of many cells, one iteration alone takes a halo of one cell (2 x 1064 x
    // 2088: 28.5 -> 23.6 us; a thread per cell 26.3), and fields of a few rows the
    // lowest tile, which wastes the fewest (20 iterations on 2 x 100000: 183 -> 57,
    // a thread per cell 96; on two of 3 x 400000 that is still 546 against 382).
    const bool many = cells > (size_t)1 << 17;
    if (many && ny <= 6)
        run_tiles<5, 3, 4>(X, grad, nfield, ny, nx, p, iters, L, w, nb, st);
    else if (many && iters == 1)
        run_tiles<1, 5, 8>(X, grad, nfield, ny, nx, p, iters, L, w, nb, st);
    else if (!many)
        run_tiles<10, 4, 8>(X, grad, nfield, ny, nx, p, iters, L, w, nb, st);
    else if (cells <= (size_t)1 << 19)
        run_tiles<10, 3, 16>(X, grad, nfield, ny, nx, p, iters, L, w, nb, st);
    else
        run_tiles<5, 5, 8>(X, grad, nfield, ny, nx, p, iters, L, w, nb, st);
    return hipGetLastError() == hipSuccess ? 0 : -5;
}

}  // extern "C"
