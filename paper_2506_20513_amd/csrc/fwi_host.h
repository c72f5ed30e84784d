// Host-side building blocks of the FWI library shared by the single-problem
// entry points (fwi_host.cpp) and the batched plans (fwi_batch.cpp):
// validation, workspace layout, pointers into the workspace, geometry
// upload and the argument blocks of the stencil kernels.  Internal; not
// part of the C ABI.
#pragma once

#include "fwi.h"
#include "fwi_internal.h"

namespace fwi {
namespace host {

inline size_t align_up(size_t v) { return (v + kAlign - 1) / kAlign * kAlign; }

// Validate the grid and geometry and derive the dimensions (FWI_* status).
int make_dims(const fwi_grid *grid, const fwi_geom *geom, Dims &d);
// Checkpoint interval minimising checkpoint plus segment-buffer memory.
int stream_depth(const Dims &d);
int choose_k(const Dims &d, int depth);
// The decomposition of the stencil passes (stored in L): tiles or streams, by the
// shots of the whole call (`all`), of which `groups` share the chip.
void make_tiling(const Dims &all, Layout &L, int groups = 1);
// Whether a call of that many cells, streaming lanes' cells and tiles of the large
// height (over all shots) runs on tiles; a problem's such lanes' cells and tiles; the
// height for that many tiles in flight; whether the streaming sweep's stores of that
// many cells, on grids of at most `grid` cells, pass the caches by; tiles of height
// `rows` for both kernels; the streaming decomposition.
bool use_tiles(int depth, bool traces_only, long long cells, long long lanes, long long tiles);
long long lane_cells(const Dims &d, int depth);
long long tile_count(const Dims &d);
int pick_tile(long long tiles);
bool far_stores(long long cells, long long grid);
void set_tiles(Layout &L, int rows);
void set_streams(Layout &L, int groups = 1);
// Row bands of height `rows` for both kernels (batched plans).
void fixed_bands(Layout &L, int rows, int depth);
// Workspace layout for a save mode (-1: fwi_gradient); k > 0 forces the
// checkpoint interval (a multiple of the streaming depth).  With `shared`,
// one shot group's layout from byte `start` (see make_group_layout).
int make_layout(const Dims &d, int mode, Layout &L, int k = 0, int depth = 0, size_t start = 0,
                const Layout *shared = nullptr, int s0 = 0);

// A gradient's shots in G groups run concurrently (fwi_host.cpp).
constexpr int kMaxShotGroups = 4;
struct GroupLayout {
    int G;
    int s0[kMaxShotGroups + 1];   // first shot of each group, then S
    Layout shared;                // arrays shared by the groups (all S shots)
    Layout grp[kMaxShotGroups];
    size_t total;
};
int make_group_layout(const Dims &d, int G, GroupLayout &GL);
int auto_shot_groups(const Dims &d);
int gradient_workspace(const Dims &d, size_t &bytes);

// Pointers into the workspace.
struct Ptrs {
    char *base;
    const Layout *L;
    float *f(size_t off) const { return reinterpret_cast<float *>(base + off); }
    int *i(size_t off) const { return reinterpret_cast<int *>(base + off); }
    Profiles prof() const {
        const Dims &d = L->d;
        float *p = f(L->off_prof);
        Profiles q;
        q.bEx = p; q.aEx = p + d.NX; q.kEx = p + 2 * d.NX;
        q.bHx = p + 3 * d.NX; q.aHx = p + 4 * d.NX; q.kHx = p + 5 * d.NX;
        float *y = p + 6 * d.NX;
        q.bEy = y; q.aEy = y + d.NY; q.kEy = y + 2 * d.NY;
        q.bHy = y + 3 * d.NY; q.aHy = y + 4 * d.NY; q.kHy = y + 5 * d.NY;
        return q;
    }
    // A State laid out at `off`: [E][Hx][Hy][phx][phy][pex][pey] (E only when
    // with_e).
    State state(size_t off, bool with_e) const {
        const Dims &d = L->d;
        const size_t S = (size_t)d.S;
        const size_t field = align_up(S * d.plane * sizeof(float));
        const size_t xs = align_up(S * d.xs * sizeof(float));
        const size_t ys = align_up(S * d.ys * sizeof(float));
        State st;
        size_t o = off;
        st.E = nullptr;
        if (with_e) { st.E = f(o); o += field; }
        st.Hx = f(o); o += field;
        st.Hy = f(o); o += field;
        st.phx = f(o); o += ys;
        st.phy = f(o); o += xs;
        st.pex = f(o); o += xs;
        st.pey = f(o);
        return st;
    }
    // Checkpoint c: the state of step c K, E first.
    State checkpoint(int c) const {
        const size_t off = L->off_ckpt + (size_t)c * L->ckpt_stride;
        State st = state(off + align_up((size_t)L->d.S * L->d.plane * sizeof(float)), false);
        st.E = f(off);
        return st;
    }
    float *slot(int k) const {
        const Dims &d = L->d;
        return f(L->off_slots) + (size_t)k * d.S * d.plane;
    }
};

#define FWI_TRY(expr)                                   \
    do {                                                \
        hipError_t e_ = (expr);                         \
        if (e_ != hipSuccess) return FWI_EHIP;          \
    } while (0)

// Geometry tables, band table and cold arguments to the workspace (waits for
// the copies, so the host arrays may be released on return).
int upload_geometry(const Ptrs &P, const fwi_geom *g, const StreamCold &cold, hipStream_t st);
int zero_state(const State &s, const Dims &d, bool with_e, hipStream_t st);
Tiling tiling(const Ptrs &P);       // forward kernel
Tiling tiling_adj(const Ptrs &P);   // adjoint kernel
StreamCold make_cold(const Ptrs &P, const fwi_geom *g, float *traces, const float *residual,
                     float *src_adjoint);
FwdStreamArgs fwd_args(const Ptrs &P);
// the H / CPML states a forward pass reads and writes
void set_states(FwdStreamArgs &a, const State &in, const State &out);
AdjStreamArgs adj_args(const Ptrs &P);

}  // namespace host
}  // namespace fwi
