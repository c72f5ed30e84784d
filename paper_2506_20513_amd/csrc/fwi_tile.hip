// Tile kernels for the forward step (Algorithm 1) and its exact transpose
// with gradient imaging (Algorithm 2), gfx950, for fields that the
// last-level cache holds.  Paper: arXiv 2506.20513, Sec. 2.1 Eqs. (3)-(13),
// Sec. 3.2, Sec. 3.3.
//
// One workgroup of NW waves owns one shot and one tile of 64 columns x
// NW R rows, halo included: lane = column, every wave holds R consecutive
// rows of all fields in registers.  The whole tile is loaded at once, up to D
// time levels are advanced in registers, and the inner part, D cells away
// from every side, is written back: what the levels leave valid.  Per level
// the waves exchange only the first and the last row of Ez (adjoint: of
// lambda_E) through LDS, with one barrier; each wave carries the H row above
// its own rows along (the same operations the wave above does), so the E
// update needs no second exchange.  x neighbours come from the neighbouring
// lanes through DPP shifts.
//
// The streaming kernels (fwi_stream.hip) read every row once, with a load
// latency per row of the march (29.5 us per 4-step launch on 148 x 148 cells,
// one shot); here all loads of a tile are in flight together and the levels
// run without touching memory, at the price of a halo on all four sides.  A
// pass of 8 steps on that grid takes 9.7 us: about 4 us launch, loads and stores,
// then 0.7 us per level, bound by the vector instructions of a tile on its CU.
// On 552 x 296 cells x 24 shots a sweep of 8 steps takes 82 us; a SIMD issues
// vector instructions in two thirds of its cycles (half of them arithmetic), the
// rest is latency that one workgroup of 16 waves per CU does not hide.  Every cell
// sees the operations of the streaming kernels in their order (the fused
// multiply-adds are written out and nothing else is fused), so the results are the
// same bit for bit.
#include "fwi_stencil.h"

#include <type_traits>

#pragma clang fp contract(off)

namespace fwi {
namespace {

// Tile of a workgroup: its shot, first column and row (halo included), the
// rows [y0, y1) it owns, and the calling wave's place in it.
struct TileGeom {
    int s, x0, r0, y0, y1;
    int wave, j0;        // wave index, first row of the wave
    int i, cx;           // column of the lane, its x-direction CPML column or -1
    bool inx, own;
    bool xt, yt;         // x-direction CPML columns in the tile, y-direction CPML
                         // rows among the wave's rows and the rows next to them
};

template <int D, int R, int NW>
__device__ __forceinline__ TileGeom tile_geom(const Tiling &tl, int S, int NX, int NY, int npml,
                                              int blk) {
    constexpr int OX = 64 - 2 * D, OY = R * NW - 2 * D;
    TileGeom g;
    g.s = blk % S;
    const int t = blk / S;
    g.x0 = (t % tl.nstrip) * OX - D;
    g.y0 = (t / tl.nstrip) * OY;
    g.y1 = min(NY, g.y0 + OY);
    g.r0 = g.y0 - D;
    g.wave = wave_in_block();
    g.j0 = g.r0 + g.wave * R;
    g.i = g.x0 + lane_id();
    g.inx = g.i >= 0 && g.i < NX;
    g.cx = g.inx ? xcol(g.i, NX, npml) : -1;
    g.own = lane_id() >= D && lane_id() < 64 - D && g.i < NX;
    g.xt = g.x0 < npml || g.x0 + 63 >= NX - 1 - npml;
    g.yt = g.j0 - 1 < npml || g.j0 + R >= NY - 1 - npml;
    return g;
}

// v as a value of its own: what is computed from it after the levels is not
// kept in registers across them
__device__ __forceinline__ int anew(int v) {
    asm volatile("" : "+v"(v));
    return v;
}

// a[r] for a wave-uniform r, by selects (the empty asm keeps the compiler from
// selecting an address instead, which would put the array into memory)
template <int R>
__device__ __forceinline__ float pick(const float (&a)[R], int r) {
    float v = 0.f;
#pragma unroll
    for (int k = 0; k < R; ++k) {
        float x = a[k];
        asm volatile("" : "+v"(x));
        v = r == k ? x : v;
    }
    return v;
}

// The workgroup's barrier of a level.  The waves of a workgroup pass it in bodies of
// their own (by_kind): the language's barrier asks for one that all threads reach, so
// this one is written as what the hardware has, where s_barrier counts the waves that
// have reached any of them.  Every wave passes it once per level, in whichever body.
__device__ __forceinline__ void level_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// f(x-direction CPML in the tile, y-direction CPML in the wave's rows)
template <class F>
__device__ __forceinline__ void by_kind(const TileGeom &g, F &&f) {
    if (!g.xt) {
        if (!g.yt) f(std::false_type(), std::false_type());
        else f(std::false_type(), std::true_type());
    } else {
        if (!g.yt) f(std::true_type(), std::false_type());
        else f(std::true_type(), std::true_type());
    }
}

// Receivers in rows [lo, hi) of the calling wave's R rows: an entry per cell,
// -1 none, the receiver's index where the cell has one, -2 - q where it has
// several (q: its first place in the shot's sorted list).  Returns the mask
// of rows that have receivers in this shot.  Only the calling wave reads the
// entries, after a workgroup barrier.
constexpr int kNoRec = -1;

template <int R>
__device__ __forceinline__ unsigned rec_table(ColdRef cold, int s, int NY, int Rn, int j0, int lo,
                                              int hi, int x0, int (*tab)[64]) {
    unsigned mask = 0;
    const int *rr = cold->g.rrow + (size_t)s * (NY + 1);
    const int *rcol = cold->g.rcol + (size_t)s * Rn, *ridx = cold->g.ridx + (size_t)s * Rn;
    const int first = max(lo, j0), end = min(hi, j0 + R);
    for (int j = first; j < end; ++j) {
        const int a = ldc(rr, j), b = ldc(rr, j + 1);
        if (a == b) continue;
        mask |= 1u << (j - j0);
        tab[j - j0][lane_id()] = kNoRec;
        for (int q = a + lane_id(); q < b; q += 64) {
            const int c = ldg(rcol, q), x = c - x0;
            if (x < 0 || x > 63 || (q > a && ldg(rcol, q - 1) == c)) continue;
            tab[j - j0][x] = (q + 1 < b && ldg(rcol, q + 1) == c) ? -2 - q : ldg(ridx, q);
        }
    }
    return mask;
}

// y-direction CPML constants of N rows from j0 on, and the mask of the rows
// that lie in it.
template <int N>
__device__ __forceinline__ unsigned rows_pml(ColdRef cold, int j0, int NY, int npml, float ch,
                                             float rdy, bool any, RowPml (&rp)[N]) {
    unsigned m = 0;
#pragma unroll
    for (int r = 0; r < N; ++r) {
        rp[r] = RowPml{ch * rdy, rdy, 0.f, 0.f, 0.f, 0.f};
        if (any && yrow(j0 + r, NY, npml) >= 0) {
            m |= 1u << r;
            rp[r] = row_pml(cold, j0 + r, ch, rdy);
        }
    }
    return m;
}

// ---------------------------------------------------------------------------
// Forward: nlev <= D levels of k_fwd's step (fwi_stream.hip).
template <int R>
struct FwdTile {
    float E[R], Hx[R], Hy[R], Ca[R], Cs[R];
    float phx[R], phy[R], pex[R], pey[R];
    float hup, phxu;             // Hx and its memory of the row above the wave's
    RowPml rp[R + 1];            // rows j0 - 1 .. j0 + R - 1
    unsigned yp;                 // bit r: rp[r] lies in the y-direction CPML
    ColPml c;
    bool xp;
    float ch;

    // one level of the wave's rows; eup, edn: Ez of the rows above and below
    template <bool XP, bool YP>
    __device__ __forceinline__ void level(float eup, float edn) {
        {
            const float d = E[0] - eup;
            hup = fmaf(-rp[0].chy, d, hup);
            if (YP && (yp & 1)) {
                phxu = fmaf(rp[0].bHy, phxu, rp[0].aHy * d);
                hup = fmaf(-ch, phxu, hup);
            }
        }
        float hprev = hup;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float pE = E[r];
            const bool ypr = YP && (yp >> (r + 1) & 1);
            const RowPml &q = rp[YP ? r + 1 : 0];
            // stages 2-3: H to n+l+1/2
            const float dEy = (r + 1 < R ? E[r + 1 < R ? r + 1 : r] : edn) - pE;
            const float dEx = from_right(pE) - pE;
            float hx = fmaf(-q.chy, dEy, Hx[r]);
            float hy = fmaf(c.chx, dEx, Hy[r]);
            if (ypr) {
                phx[r] = fmaf(q.bHy, phx[r], q.aHy * dEy);
                hx = fmaf(-ch, phx[r], hx);
            }
            if (XP && xp) {
                phy[r] = fmaf(c.bHx, phy[r], c.aHx * dEx);
                hy = fmaf(ch, phy[r], hy);
            }
            // stages 4-5: E to n+l+1
            const float dHy = hy - from_left(hy);
            const float dHx = hx - hprev;
            float curl = fmaf(dHy, c.cxE, -(dHx * q.cyE));
            if (XP && xp) {
                pex[r] = fmaf(c.bEx, pex[r], c.aEx * dHy);
                curl += pex[r];
            }
            if (ypr) {
                pey[r] = fmaf(q.bEy, pey[r], q.aEy * dHx);
                curl -= pey[r];
            }
            E[r] = fmaf(Ca[r], pE, Cs[r] * curl);
            Hx[r] = hx;
            Hy[r] = hy;
            hprev = hx;
        }
    }
};

template <int D, int R, int NW, int LEV, bool XP, bool YP>
__device__ __forceinline__ void fwd_tile_kind(const FwdStreamArgs &a, const TileGeom &g,
                                              float (*xch)[NW][2][64], int (*rtab)[R][64]) {
    ColdRef cold = (ColdRef)a.cold;
    const int lane = lane_id(), s = g.s, i = g.i, j0 = g.j0;
    const int NY = a.NY, P = a.pitch, npml = a.npml;
    const size_t so = (size_t)s * a.plane;
    const float *Ein = a.E_in + so, *Hxin = a.Hx_in + so, *Hyin = a.Hy_in + so;
    FwdTile<R> f;
    f.ch = a.ch;
    f.xp = g.cx >= 0;
    f.hup = f.phxu = 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int j = j0 + r;
        f.E[r] = f.Hx[r] = f.Hy[r] = f.Ca[r] = f.Cs[r] = 0.f;
        if (j >= 0 && j < NY && g.inx) {
            const unsigned k = (unsigned)(j * P + i);
            f.E[r] = ldg(Ein, k);
            f.Hx[r] = ldg(Hxin, k);
            f.Hy[r] = ldg(Hyin, k);
            f.Ca[r] = ldg(a.Ca, k);
            f.Cs[r] = ldg(a.Cs, k);
        }
    }
    const bool up = g.wave > 0 && j0 - 1 >= 0 && j0 - 1 < NY && g.inx;
    if (up) f.hup = ldg(Hxin, (unsigned)((j0 - 1) * P + i));
    const PsiPtr pin{a.psi_in, a.psi_y, a.psi_x}, pout{a.psi_out, a.psi_y, a.psi_x};
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int j = j0 + r, ry = yrow(j, NY, npml);
        f.phx[r] = f.phy[r] = f.pex[r] = f.pey[r] = 0.f;
        if (YP && ry >= 0 && g.inx) {
            f.phx[r] = ldg(pin.phx(s, a.ys), (unsigned)(ry * P + i));
            f.pey[r] = ldg(pin.pey(s, a.ys), (unsigned)(ry * P + i));
        }
        if (XP && f.xp && j >= 0 && j < NY) {
            f.phy[r] = ldg(pin.phy(s, a.xs), (unsigned)(j * a.W + g.cx));
            f.pex[r] = ldg(pin.pex(s, a.xs), (unsigned)(j * a.W + g.cx));
        }
    }
    if (YP && up && yrow(j0 - 1, NY, npml) >= 0)
        f.phxu = ldg(pin.phx(s, a.ys), (unsigned)(yrow(j0 - 1, NY, npml) * P + i));
    f.c = XP ? col_pml(cold, i, g.inx, a.ch, a.rdx)
               : ColPml{a.ch * a.rdx, a.rdx, 0.f, 0.f, 0.f, 0.f};
    f.yp = rows_pml(cold, j0 - 1, NY, npml, a.ch, a.rdy, YP, f.rp);
    // source and receivers of the tile
    const int sr = ldc<int>(cold->g.src_ij, 2 * s + 1) - j0;
    const bool slane = i == ldc<int>(cold->g.src_ij, 2 * s);
    const bool src = sr >= 0 && sr < R;
    const float *wav = cold->g.wavelet + (size_t)s * a.nt + a.n;
    unsigned rmask = 0;
    if (a.record)
        rmask = rec_table<R>(cold, s, NY, a.R, j0, max(g.y0, ldc<int>(cold->g.rspan, 2 * s)),
                             min(g.y1, ldc<int>(cold->g.rspan, 2 * s + 1) + 1), g.x0,
                             rtab[g.wave]);
    float *el = LEV ? a.E_lev + so : nullptr;
    const int olo = g.y0 - j0, ohi = g.y1 - j0;      // owned rows of the wave

    auto record = [&](int l) {
        float *tr = cold->traces + ((size_t)s * a.nt + a.n + l) * a.R;
        for (unsigned m = rmask; m; m &= m - 1) {
            const int r = __builtin_ctz(m);
            const int v = rtab[g.wave][r][lane];
            const float e = pick(f.E, r);
            if (!g.own || v == kNoRec) continue;
            if (v >= 0) {
                stg(tr, (unsigned)v, e);
            } else {
                const int *rcol = cold->g.rcol + (size_t)s * a.R;
                const int end = ldc(cold->g.rrow + (size_t)s * (NY + 1), j0 + r + 1);
                for (int q = -2 - v; q < end && ldg(rcol, q) == i; ++q)
                    stg(tr, (unsigned)ldg(cold->g.ridx + (size_t)s * a.R, q), e);
            }
        }
    };
    for (int l = 0; l < a.nlev; ++l) {
        const int b = l & 1;
        xch[b][g.wave][0][lane] = f.E[0];
        xch[b][g.wave][1][lane] = f.E[R - 1];
        const float w = src ? ldc(wav, l) : 0.f;
        level_barrier();
        const float eup = g.wave > 0 ? xch[b][g.wave - 1][1][lane] : 0.f;
        const float edn = g.wave < NW - 1 ? xch[b][g.wave + 1][0][lane] : 0.f;
        if (rmask) record(l);                        // stage 1
        f.template level<XP, YP>(eup, edn);
        if (src) {                                   // stage 6
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (r == sr && slane) f.E[r] = fmaf(-(f.Cs[r] * w), a.src_scale, f.E[r]);
        }
        if (LEV) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                if (!(r >= olo && r < ohi && g.own)) continue;
                // The history of the problems that take large tiles outgrows the
                // caches (24 shots of 552 x 296: 122.2 -> 120.8 ms per gradient;
                // batch of 12: 273.6 -> 269.2), that of small ones does not
                // (one shot of 260 x 160: 5.41 -> 5.45 ms)
                const unsigned k = (unsigned)((j0 + r) * P + i);
                if (NW * R == kTileRowsLarge) stg_nt(el, k, f.E[r]);
                else stg(el, k, f.E[r]);
            }
            el += a.lev_stride;
        }
    }
    const int ie = anew(i), ce = anew(g.cx);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (!(r >= olo && r < ohi && g.own)) continue;
        const int j = j0 + r;
        const unsigned k = (unsigned)(j * P + ie);
        if (!LEV) stg(a.E_out + so, k, f.E[r]);
        stg(a.Hx_out + so, k, f.Hx[r]);
        stg(a.Hy_out + so, k, f.Hy[r]);
        const int ry = yrow(j, NY, npml);
        if (YP && ry >= 0) {
            stg(pout.phx(s, a.ys), (unsigned)(ry * P + ie), f.phx[r]);
            stg(pout.pey(s, a.ys), (unsigned)(ry * P + ie), f.pey[r]);
        }
        if (XP && f.xp) {
            stg(pout.phy(s, a.xs), (unsigned)(j * a.W + ce), f.phy[r]);
            stg(pout.pex(s, a.xs), (unsigned)(j * a.W + ce), f.pex[r]);
        }
    }
}

// Each kind of wave (tile with or without x-direction CPML columns, rows with
// or without y-direction CPML) runs a body of its own from the loads to the
// stores: nothing per lane is live where they part.  All pass as many barriers
// (level_barrier).
template <int D, int R, int NW, int LEV>
__device__ __forceinline__ void fwd_tile(const FwdStreamArgs &a, int blk) {
    __shared__ float xch[2][NW][2][64];
    __shared__ int rtab[NW][R][64];
    const TileGeom g = tile_geom<D, R, NW>(a.tl, a.S, a.NX, a.NY, a.npml, blk);
    by_kind(g, [&](auto xt, auto yt) {
        fwd_tile_kind<D, R, NW, LEV, decltype(xt)::value, decltype(yt)::value>(a, g, xch, rtab);
    });
}

template <int D, int R, int NW, int LEV>
__global__ __launch_bounds__(64 * NW) void k_fwd_tile(FwdStreamArgs a) {
    fwd_tile<D, R, NW, LEV>(a, xcd_logical(blockIdx.x, gridDim.x));
}

template <int D, int R, int NW, int LEV>
__global__ __launch_bounds__(64 * NW) void k_fwd_tile_tab(const FwdStreamArgs *tab,
                                                          const unsigned *boff, int nm) {
    const unsigned lb = (unsigned)xcd_logical(blockIdx.x, gridDim.x);
    const int m = table_entry(boff, nm, lb);
    const FwdStreamArgs a = load_const(tab, m);
    fwd_tile<D, R, NW, LEV>(a, (int)(lb - ldc(boff, m)));
}

// ---------------------------------------------------------------------------
// Adjoint: nlev <= D levels of k_adj's step (fwi_stream.hip), level l taking
// lambda^{n+1} to lambda^n for n = n_top-1-l.  The imaging sums of a pass are
// added to S1, S2 whenever n reaches a multiple of a.group, as passes of
// a.group levels would add them: the sums of the first group wait in LDS
// (`grp`) for the end of the pass, which then adds both groups' in order.
// The update coefficients of the tile live in LDS as well; both keep the
// registers to what every level works on.
template <int R>
struct AdjTile {
    float L[R], Hx[R], Hy[R], en[R], a1[R], a2[R];
    float phx[R], phy[R], pex[R], pey[R];
    float hup, phxu, peyu, peyd;     // the rows above and below the wave's
    RowPml rp[R + 2];                // rows j0 - 1 .. j0 + R
    unsigned yp;
    ColPml c;
    bool xp;
    float ch;

    // one level; ca, cs: the coefficients of the wave's rows (stride 64), of
    // which cs also holds the rows above and below; add(r, le): the adjoint
    // source of row r added to le
    template <bool XP, bool YP, class Add>
    __device__ __forceinline__ void level(const float *ca, const float *cs, float lup, float ldn,
                                          Add add) {
        // transposed E and H steps of the row above, as the wave above does
        const float gu = cs[-64] * lup;
        float ldy = -gu * rp[0].cyE;
        if (YP && (yp & 1)) {
            const float ty = peyu - gu;
            ldy = fmaf(rp[0].aEy, ty, ldy);
            peyu = rp[0].bEy * ty;
        }
        float gc = cs[0] * L[0];
        float ldyn = -gc * rp[YP ? 1 : 0].cyE;
        if (YP && (yp >> 1 & 1)) {
            const float ty = pey[0] - gc;
            ldyn = fmaf(rp[1].aEy, ty, ldyn);
            pey[0] = rp[1].bEy * ty;
        }
        hup = hup + (ldy - ldyn);
        float ldey_prev = -hup * rp[0].chy;
        if (YP && (yp & 1)) {
            const float t2 = fmaf(-ch, hup, phxu);
            ldey_prev = fmaf(rp[0].aHy, t2, ldey_prev);
            phxu = rp[0].bHy * t2;
        }
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float pL = L[r];
            const bool ypr = YP && (yp >> (r + 1) & 1);
            const RowPml &q = rp[YP ? r + 1 : 0];
            // A1: transposed E step; LDy of the next row
            const float gr = gc;
            float ldx = gr * c.cxE;
            ldy = ldyn;
            if (XP && xp) {
                const float tx = pex[r] + gr;
                ldx = fmaf(c.aEx, tx, ldx);
                pex[r] = c.bEx * tx;
            }
            const int rn = r + 1 < R ? r + 1 : r;
            gc = cs[64 * (r + 1)] * (r + 1 < R ? L[rn] : ldn);
            ldyn = -gc * rp[YP ? r + 2 : 0].cyE;
            if (YP && (yp >> (r + 2) & 1)) {
                float &py = r + 1 < R ? pey[rn] : peyd;
                const float ty = py - gc;
                ldyn = fmaf(rp[r + 2].aEy, ty, ldyn);
                py = rp[r + 2].bEy * ty;
            }
            const float lhy = Hy[r] + (ldx - from_right(ldx));
            const float lhx = Hx[r] + (ldy - ldyn);
            // A2: transposed H step
            float ldex = lhy * c.chx;
            if (XP && xp) {
                const float t1 = fmaf(ch, lhy, phy[r]);
                ldex = fmaf(c.aHx, t1, ldex);
                phy[r] = c.bHx * t1;
            }
            float ldey = -lhx * q.chy;
            if (ypr) {
                const float t2 = fmaf(-ch, lhx, phx[r]);
                ldey = fmaf(q.aHy, t2, ldey);
                phx[r] = q.bHy * t2;
            }
            float le = fmaf(ca[64 * r], pL, from_left(ldex) - ldex) + (ldey_prev - ldey);
            ldey_prev = ldey;
            le = add(r, le);                         // A3
            // imaging
            a1[r] = fmaf(en[r], le - pL, a1[r]);
            a2[r] = fmaf(en[r], le + pL, a2[r]);
            L[r] = le;
            Hx[r] = lhx;
            Hy[r] = lhy;
        }
    }
};

template <int D, int R, int NW, bool XP, bool YP>
__device__ __forceinline__ void adj_tile_kind(const AdjStreamArgs &a, const TileGeom &g,
                                              float (*xch)[NW][2][64],
                                              float (*cc)[NW * R + 2][64],
                                              float (*grp)[NW * R - 2 * D][64 - 2 * D],
                                              int (*rtab)[R][64]) {
    ColdRef cold = (ColdRef)a.cold;
    const int lane = lane_id(), s = g.s, i = g.i, j0 = g.j0, row = g.wave * R;
    const int NY = a.NY, P = a.pitch, npml = a.npml;
    const size_t so = (size_t)s * a.plane;
    const float *Lin = a.L_in + so, *Hxin = a.LHx_in + so, *Hyin = a.LHy_in + so;
    const int olo = g.y0 - j0, ohi = g.y1 - j0;      // owned rows of the wave
    AdjTile<R> f;
    f.ch = a.ch;
    f.xp = g.cx >= 0;
    f.hup = f.phxu = f.peyu = f.peyd = 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int j = j0 + r;
        float ca = 0.f, cs = 0.f;
        f.L[r] = f.Hx[r] = f.Hy[r] = f.a1[r] = f.a2[r] = 0.f;
        if (j >= 0 && j < NY && g.inx) {
            const unsigned k = (unsigned)(j * P + i);
            f.L[r] = ldg(Lin, k);
            f.Hx[r] = ldg(Hxin, k);
            f.Hy[r] = ldg(Hyin, k);
            ca = ldg(a.Ca, k);
            cs = ldg(a.Cs, k);
        }
        cc[0][row + 1 + r][lane] = ca;
        cc[1][row + 1 + r][lane] = cs;
    }
    if (g.wave == 0) cc[1][0][lane] = 0.f;
    if (g.wave == NW - 1) cc[1][NW * R + 1][lane] = 0.f;
    // forward Ez^n of level l for the cells the tile owns
    const float *el = a.E_lev + (size_t)(a.n_top - 1 - a.n_base) * a.lev_stride + so;
    auto load_en = [&]() {
#pragma unroll
        for (int r = 0; r < R; ++r)
            f.en[r] = (r >= olo && r < ohi && g.own) ? ldg(el, (unsigned)((j0 + r) * P + i)) : 0.f;
    };
    load_en();
    const bool up = g.wave > 0 && j0 - 1 >= 0 && j0 - 1 < NY && g.inx;
    if (up) f.hup = ldg(Hxin, (unsigned)((j0 - 1) * P + i));
    const PsiPtr pin{a.psi_in, a.psi_y, a.psi_x}, pout{a.psi_out, a.psi_y, a.psi_x};
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int j = j0 + r, ry = yrow(j, NY, npml);
        f.phx[r] = f.phy[r] = f.pex[r] = f.pey[r] = 0.f;
        if (YP && ry >= 0 && g.inx) {
            f.phx[r] = ldg(pin.phx(s, a.ys), (unsigned)(ry * P + i));
            f.pey[r] = ldg(pin.pey(s, a.ys), (unsigned)(ry * P + i));
        }
        if (XP && f.xp && j >= 0 && j < NY) {
            f.phy[r] = ldg(pin.phy(s, a.xs), (unsigned)(j * a.W + g.cx));
            f.pex[r] = ldg(pin.pex(s, a.xs), (unsigned)(j * a.W + g.cx));
        }
    }
    if (YP) {
        const int ru = yrow(j0 - 1, NY, npml), rd = yrow(j0 + R, NY, npml);
        if (up && ru >= 0) {
            f.phxu = ldg(pin.phx(s, a.ys), (unsigned)(ru * P + i));
            f.peyu = ldg(pin.pey(s, a.ys), (unsigned)(ru * P + i));
        }
        if (g.wave < NW - 1 && g.inx && rd >= 0)
            f.peyd = ldg(pin.pey(s, a.ys), (unsigned)(rd * P + i));
    }
    f.c = XP ? col_pml(cold, i, g.inx, a.ch, a.rdx)
               : ColPml{a.ch * a.rdx, a.rdx, 0.f, 0.f, 0.f, 0.f};
    f.yp = rows_pml(cold, j0 - 1, NY, npml, a.ch, a.rdy, YP, f.rp);
    const int sr = ldc<int>(cold->g.src_ij, 2 * s + 1) - j0;
    const bool slane = g.own && i == ldc<int>(cold->g.src_ij, 2 * s);
    const bool sadj = cold->src_adjoint && sr >= max(0, olo) && sr < min(R, ohi);
    // adjoint sources act in the halo too
    const unsigned rmask =
        rec_table<R>(cold, s, NY, a.R, j0, ldc<int>(cold->g.rspan, 2 * s),
                     ldc<int>(cold->g.rspan, 2 * s + 1) + 1, g.x0, rtab[g.wave]);
    bool two = false;    // a first group waits in grp (passes hold at most two groups)

    const float *ca = &cc[0][row + 1][lane], *cs = &cc[1][row + 1][lane];
    {
        for (int l = 0; l < a.nlev; ++l) {
            const int b = l & 1, n = a.n_top - 1 - l;
            xch[b][g.wave][0][lane] = f.L[0];
            xch[b][g.wave][1][lane] = f.L[R - 1];
            level_barrier();
            const float lup = g.wave > 0 ? xch[b][g.wave - 1][1][lane] : 0.f;
            const float ldn = g.wave < NW - 1 ? xch[b][g.wave + 1][0][lane] : 0.f;
            if (sadj && slane)
                stg(cold->src_adjoint + (size_t)s * a.nt, (unsigned)n,
                    -cs[64 * sr] * pick(f.L, sr) * a.src_scale);
            f.template level<XP, YP>(
                ca, cs, lup, ldn, [&](int r, float le) {
                    if (!(rmask >> r & 1)) return le;
                    const int v = rtab[g.wave][r][lane];
                    const float *res = cold->residual + ((size_t)s * a.nt + n) * a.R;
                    if (v >= 0) {
                        le += ldg(res, (unsigned)v);
                    } else if (v != kNoRec) {
                        const int *rcol = cold->g.rcol + (size_t)s * a.R;
                        const int end = ldc(cold->g.rrow + (size_t)s * (NY + 1), j0 + r + 1);
                        for (int k = -2 - v; k < end && ldg(rcol, k) == i; ++k)
                            le += ldg(res, (unsigned)ldg(cold->g.ridx + (size_t)s * a.R, k));
                    }
                    return le;
                });
            if (l + 1 == a.nlev) break;
            el -= a.lev_stride;
            load_en();
            if ((n & (a.group - 1)) == 0) {
                two = true;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    if (r >= olo && r < ohi && g.own) {
                        grp[0][row + r - D][lane - D] = f.a1[r];
                        grp[1][row + r - D][lane - D] = f.a2[r];
                    }
                    f.a1[r] = f.a2[r] = 0.f;
                }
            }
        }
    }
    const int ie = anew(i), ce = anew(g.cx);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (!(r >= olo && r < ohi && g.own)) continue;
        const int j = j0 + r;
        const unsigned k = (unsigned)(j * P + ie);
        stg(a.L_out + so, k, f.L[r]);
        stg(a.LHx_out + so, k, f.Hx[r]);
        stg(a.LHy_out + so, k, f.Hy[r]);
        float s1 = ldg(a.S1 + so, k), s2 = ldg(a.S2 + so, k);
        if (two) {
            s1 += grp[0][row + r - D][lane - D];
            s2 += grp[1][row + r - D][lane - D];
        }
        stg(a.S1 + so, k, s1 + f.a1[r]);
        stg(a.S2 + so, k, s2 + f.a2[r]);
        const int ry = yrow(j, NY, npml);
        if (YP && ry >= 0) {
            stg(pout.phx(s, a.ys), (unsigned)(ry * P + ie), f.phx[r]);
            stg(pout.pey(s, a.ys), (unsigned)(ry * P + ie), f.pey[r]);
        }
        if (XP && f.xp) {
            stg(pout.phy(s, a.xs), (unsigned)(j * a.W + ce), f.phy[r]);
            stg(pout.pex(s, a.xs), (unsigned)(j * a.W + ce), f.pex[r]);
        }
    }
}

template <int D, int R, int NW>
__device__ __forceinline__ void adj_tile(const AdjStreamArgs &a, int blk) {
    __shared__ float xch[2][NW][2][64];
    __shared__ float cc[2][NW * R + 2][64];          // Ca, Cs; a row above, a row below
    __shared__ float grp[2][NW * R - 2 * D][64 - 2 * D];
    __shared__ int rtab[NW][R][64];
    const TileGeom g = tile_geom<D, R, NW>(a.tl, a.S, a.NX, a.NY, a.npml, blk);
    by_kind(g, [&](auto xt, auto yt) {
        adj_tile_kind<D, R, NW, decltype(xt)::value, decltype(yt)::value>(a, g, xch, cc, grp, rtab);
    });
}

template <int D, int R, int NW>
__global__ __launch_bounds__(64 * NW) void k_adj_tile(AdjStreamArgs a) {
    adj_tile<D, R, NW>(a, xcd_logical(blockIdx.x, gridDim.x));
}

template <int D, int R, int NW>
__global__ __launch_bounds__(64 * NW) void k_adj_tile_tab(const AdjStreamArgs *tab,
                                                          const unsigned *boff, int nm) {
    const unsigned lb = (unsigned)xcd_logical(blockIdx.x, gridDim.x);
    const int m = table_entry(boff, nm, lb);
    const AdjStreamArgs a = load_const(tab, m);
    adj_tile<D, R, NW>(a, (int)(lb - ldc(boff, m)));
}

// Tile shapes: rows per wave and waves per workgroup for each tile height.
template <class F>
hipError_t for_tile(int rows, F f) {
    if (rows == kTileRowsSmall)
        return f(std::integral_constant<int, 4>(), std::integral_constant<int, 8>());
    if (rows == kTileRowsLarge)
        return f(std::integral_constant<int, 4>(), std::integral_constant<int, 16>());
    return hipErrorInvalidValue;
}

}  // namespace

hipError_t launch_fwd_tile(const FwdStreamArgs &a, hipStream_t st) {
    if (a.nlev < 1 || a.nlev > kTileLevels) return hipErrorInvalidValue;
    const dim3 grid(stream_blocks(a.S, a.tl));
    return for_tile(a.tl.tile, [&](auto r, auto nw) {
        constexpr int R = decltype(r)::value, NW = decltype(nw)::value;
        if (a.E_lev)
            hipLaunchKernelGGL((k_fwd_tile<kTileLevels, R, NW, 1>), grid, dim3(64 * NW), 0, st, a);
        else
            hipLaunchKernelGGL((k_fwd_tile<kTileLevels, R, NW, 0>), grid, dim3(64 * NW), 0, st, a);
        return hipGetLastError();
    });
}

hipError_t launch_adj_tile(const AdjStreamArgs &a, hipStream_t st) {
    if (a.nlev < 1 || a.nlev > kTileLevels) return hipErrorInvalidValue;
    const dim3 grid(stream_blocks(a.S, a.tl));
    return for_tile(a.tl.tile, [&](auto r, auto nw) {
        constexpr int R = decltype(r)::value, NW = decltype(nw)::value;
        hipLaunchKernelGGL((k_adj_tile<kTileLevels, R, NW>), grid, dim3(64 * NW), 0, st, a);
        return hipGetLastError();
    });
}

hipError_t launch_fwd_tile_table(const FwdStreamArgs *tab, const unsigned *boff, int nm,
                                 unsigned nblocks, int rows, int lev, hipStream_t st) {
    return for_tile(rows, [&](auto r, auto nw) {
        constexpr int R = decltype(r)::value, NW = decltype(nw)::value;
        if (lev)
            hipLaunchKernelGGL((k_fwd_tile_tab<kTileLevels, R, NW, 1>), dim3(nblocks),
                               dim3(64 * NW), 0, st, tab, boff, nm);
        else
            hipLaunchKernelGGL((k_fwd_tile_tab<kTileLevels, R, NW, 0>), dim3(nblocks),
                               dim3(64 * NW), 0, st, tab, boff, nm);
        return hipGetLastError();
    });
}

hipError_t launch_adj_tile_table(const AdjStreamArgs *tab, const unsigned *boff, int nm,
                                 unsigned nblocks, int rows, hipStream_t st) {
    return for_tile(rows, [&](auto r, auto nw) {
        constexpr int R = decltype(r)::value, NW = decltype(nw)::value;
        hipLaunchKernelGGL((k_adj_tile_tab<kTileLevels, R, NW>), dim3(nblocks), dim3(64 * NW), 0,
                           st, tab, boff, nm);
        return hipGetLastError();
    });
}

}  // namespace fwi
