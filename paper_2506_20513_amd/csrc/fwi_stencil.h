// Device helpers shared by the stencil kernels (fwi_stream.hip,
// fwi_tile.hip): memory access, lane shifts, CPML rows and columns, receiver
// ranges, block renumbering and the problem tables of the batched launches.
#pragma once

#include "fwi_internal.h"

namespace fwi {
namespace {

// Memory access helpers.  Per-lane accesses go through the global address
// space with a uniform base and a 32-bit offset (SGPR base + VGPR offset
// addressing); read-only tables indexed by uniform values go through the
// constant address space (scalar loads).  Offsets stay below 2^32 bytes by
// the grid-size check on the host.
#define FWI_AS_GLOBAL __attribute__((address_space(1)))
#define FWI_AS_CONST __attribute__((address_space(4)))
template <class T>
__device__ __forceinline__ T ldg(const T *base, unsigned idx) {
    return *(const FWI_AS_GLOBAL T *)((const FWI_AS_GLOBAL char *)base +
                                      (size_t)(idx * (unsigned)sizeof(T)));
}
template <class T>
__device__ __forceinline__ void stg(T *base, unsigned idx, T v) {
    *(FWI_AS_GLOBAL T *)((FWI_AS_GLOBAL char *)base + (size_t)(idx * (unsigned)sizeof(T))) = v;
}
// a store that is not read again before the caches have turned over
template <class T>
__device__ __forceinline__ void stg_nt(T *base, unsigned idx, T v) {
    __builtin_nontemporal_store(v, (FWI_AS_GLOBAL T *)((FWI_AS_GLOBAL char *)base +
                                                       (size_t)(idx * (unsigned)sizeof(T))));
}
template <class T>
__device__ __forceinline__ T ldc(const T *base, unsigned idx) {
    return ((const FWI_AS_CONST T *)base)[idx];
}
// The per-call cold arguments, read with scalar loads.
using ColdRef = const FWI_AS_CONST StreamCold *;

// lane i receives lane i-1's value (lane 0 receives 0)
__device__ __forceinline__ float from_left(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xf, 0xf, false));
}
// lane i receives lane i+1's value (lane 63 receives 0)
__device__ __forceinline__ float from_right(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xf, 0xf, false));
}

// Column of the x-direction CPML strip store holding column i, or -1.
__device__ __forceinline__ int xcol(int i, int NX, int npml) {
    if (i < npml) return i;
    if (i >= NX - 1 - npml) return i - (NX - 1 - npml) + npml;
    return -1;
}
// Row of the y-direction CPML strip store holding row j, or -1 (also for
// rows outside the grid).
__device__ __forceinline__ int yrow(int j, int NY, int npml) {
    if (j < 0 || j >= NY) return -1;
    if (j < npml) return j;
    if (j >= NY - 1 - npml) return j - (NY - 1 - npml) + npml;
    return -1;
}

// Blocks are dealt round-robin to the 8 XCDs; renumber them so that each XCD
// works on a contiguous range of the (band, strip, shot) order, with shots
// fastest: the waves co-resident on one XCD then share coefficient rows and
// strip halos through that XCD's L2.
__device__ __forceinline__ int xcd_logical(int b, int nb) {
    const int per = nb / 8, rem = nb % 8;
    const int x = b % 8, k = b / 8;
    return x < rem ? x * (per + 1) + k : rem * (per + 1) + (x - rem) * per + k;
}

// Receivers of shot s on row j whose column lies in [c0, c1): index range
// into the shot's (row, column)-sorted receiver list.
__device__ __forceinline__ void rec_range(const int *rrow, const int *rcol, int s, int NY,
                                          int R, int j, int c0, int c1, int &lo, int &hi) {
    const int *rr = rrow + (size_t)s * (NY + 1);
    lo = ldc(rr, j);
    hi = ldc(rr, j + 1);
    if (lo == hi) return;
    const int *rc = rcol + (size_t)s * R;
    int a = lo, b = hi;
    while (a < b) {
        const int m = (a + b) >> 1;
        if (ldc(rc, m) < c0) a = m + 1; else b = m;
    }
    int e = a, f = hi;
    while (e < f) {
        const int m = (e + f) >> 1;
        if (ldc(rc, m) < c1) e = m + 1; else f = m;
    }
    lo = a;
    hi = e;
}

// CPML constants of one row (y direction), scaled by 1/dy where the update
// multiplies by it.  Outside the y strips kappa = 1 and a = 0.
struct RowPml {
    float chy, cyE, bHy, aHy, bEy, aEy;
};
__device__ __forceinline__ RowPml row_pml(ColdRef cold, int j, float ch, float rdy) {
    RowPml r;
    r.chy = ch * rdy * ldc<float>(cold->p.kHy, j);
    r.cyE = rdy * ldc<float>(cold->p.kEy, j);
    r.bHy = ldc<float>(cold->p.bHy, j);
    r.aHy = ldc<float>(cold->p.aHy, j) * rdy;
    r.bEy = ldc<float>(cold->p.bEy, j);
    r.aEy = ldc<float>(cold->p.aEy, j) * rdy;
    return r;
}

// Lane (column) constants: kappa, b and a of the x direction, scaled by 1/dx.
struct ColPml {
    float chx, cxE, bHx, aHx, bEx, aEx;
};
__device__ __forceinline__ ColPml col_pml(ColdRef cold, int i, bool inx, float ch, float rdx) {
    ColPml c{0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    if (inx) {
        c.chx = ch * rdx * ldg<float>(cold->p.kHx, i);
        c.cxE = rdx * ldg<float>(cold->p.kEx, i);
        c.bHx = ldg<float>(cold->p.bHx, i);
        c.aHx = ldg<float>(cold->p.aHx, i) * rdx;
        c.bEx = ldg<float>(cold->p.bEx, i);
        c.aEx = ldg<float>(cold->p.aEx, i) * rdx;
    }
    return c;
}

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63u); }
// Index of the calling wave in its workgroup (wave-uniform).
__device__ __forceinline__ int wave_in_block() {
    return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
}

// A struct read from the constant address space dword by dword (scalar
// loads; unused fields are never loaded).
template <class T>
__device__ __forceinline__ T load_const(const T *p, int m) {
    static_assert(sizeof(T) % 4 == 0, "dword-sized struct");
    T v;
    const FWI_AS_CONST unsigned *src = (const FWI_AS_CONST unsigned *)(p + m);
    unsigned *dst = reinterpret_cast<unsigned *>(&v);
#pragma unroll
    for (int k = 0; k < (int)(sizeof(T) / 4); ++k) dst[k] = src[k];
    return v;
}

// The same pass for several independent problems in one launch: problem m
// owns blocks [boff[m], boff[m+1]) of the XCD-renumbered block order and
// reads its arguments from tab[m].
__device__ __forceinline__ int table_entry(const unsigned *boff, int nm, unsigned lb) {
    int lo = 0, hi = nm;                      // boff[lo] <= lb < boff[hi]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (ldc(boff, mid) <= lb) lo = mid; else hi = mid;
    }
    return lo;
}

// CPML memories of a state in their padded layout (see Ptrs::state): phx,
// phy, pex, pey behind one another from `p` on.
struct PsiPtr {
    const float *p;
    size_t y, x;         // padded sizes of a y-strip and an x-strip array
    __device__ __forceinline__ float *phx(int s, size_t ys) const {
        return const_cast<float *>(p) + (size_t)s * ys;
    }
    __device__ __forceinline__ float *phy(int s, size_t xs) const {
        return const_cast<float *>(p) + y + (size_t)s * xs;
    }
    __device__ __forceinline__ float *pex(int s, size_t xs) const {
        return const_cast<float *>(p) + y + x + (size_t)s * xs;
    }
    __device__ __forceinline__ float *pey(int s, size_t ys) const {
        return const_cast<float *>(p) + y + 2 * x + (size_t)s * ys;
    }
};

}  // namespace
}  // namespace fwi
