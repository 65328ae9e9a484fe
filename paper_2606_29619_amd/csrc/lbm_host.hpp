// lbm_host.hpp -- host-side internals shared by the solver and the request server: error
// reporting, the workspace layout, the solver handle and the tile geometry.
#pragma once

#include "lbm.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <string>
#include <type_traits>

#include "lbm_device.hpp"

namespace lbmh {

inline thread_local std::string g_err;

inline int fail(int code, const char *fmt, ...) {
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return code;
}

#define HIP_TRY(expr)                                                                   \
    do {                                                                                \
        hipError_t e_ = (expr);                                                         \
        if (e_ != hipSuccess)                                                           \
            return fail(LBM_ERR_HIP, "%s failed: %s", #expr, hipGetErrorString(e_));    \
    } while (0)

#define LAUNCH_CHECK()                                                                  \
    do {                                                                                \
        hipError_t e_ = hipGetLastError();                                              \
        if (e_ != hipSuccess)                                                           \
            return fail(LBM_ERR_HIP, "kernel launch failed: %s", hipGetErrorString(e_)); \
    } while (0)

inline size_t align256(size_t x) { return (x + 255) & ~size_t(255); }

struct Layout {
    size_t f, eps, muD, muF, mask, m1[2], m2[2], vsnap, part, res;
    size_t bcell, bcode, bval;  // boundary-node list (wet-node boundaries)
    size_t m0, mx;              // (rho, v_0) records and a second velocity buffer (Picard)
    size_t deps;                // analytic porosity derivatives, D + D(D+1)/2 planes
    size_t tsolid;              // per-tile flag: a solid cell within one cell of the tile
    size_t tflat;               // per-tile flag: a porosity gradient somewhere in the tile
    size_t f2;                  // second population buffer (runs stepped in one launch)
    size_t base;                // bytes without f2: what a run needs at least
    size_t total;
};

// sp: bytes per population value; s: bytes per value of the static fields and moment records.
// ntiles: workgroups of the tiled passes (solid runs keep one flag byte per tile).
inline Layout make_layout(int Q, int D, size_t N, size_t sp, size_t s, bool solids, bool lagged,
                          size_t ntiles, size_t nbnodes = 0, bool picard = false,
                          bool analytic = false, bool second = false) {
    Layout L{};
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off = align256(off + bytes);
        return o;
    };
    // the population region also stages the FP64 inputs at creation (up to 4 arrays of N)
    L.f = take(std::max((size_t)Q * N * sp, 4 * N * sizeof(double)));
    L.eps = take(N * s);
    L.muD = take(N * s);
    L.muF = take(N * s);
    L.mask = solids ? take(N) : 0;
    // packed (rho, v^(1)) and (rho, v) records; the lagged scheme keeps a second pair so that
    // one step reads the previous records while it writes the new ones
    L.m1[0] = take(4 * N * s);
    L.m2[0] = take(4 * N * s);
    L.m1[1] = lagged ? take(4 * N * s) : L.m1[0];
    L.m2[1] = lagged ? take(4 * N * s) : L.m2[0];
    L.vsnap = take((size_t)D * N * s);
    L.part = take((size_t)lbm::kStatsBlocks * lbm::kStatsSlots * sizeof(double));
    L.res = take(lbm::kStatsSlots * sizeof(double));
    L.bcell = nbnodes ? take(nbnodes * sizeof(uint32_t)) : 0;
    L.bcode = nbnodes ? take(nbnodes * sizeof(uint32_t)) : 0;
    L.bval = nbnodes ? take(nbnodes * 4 * s) : 0;
    L.m0 = picard ? take(4 * N * s) : 0;
    L.mx = picard ? take(4 * N * s) : 0;
    L.deps = analytic ? take((size_t)(D + D * (D + 1) / 2) * N * s) : 0;
    L.tsolid = solids ? take(ntiles) : 0;
    L.tflat = analytic ? 0 : take(ntiles);
    L.base = off;
    L.f2 = second ? take((size_t)Q * N * sp) : 0;
    L.total = off;
    return L;
}

inline bool is_finite(double x) { return std::isfinite(x); }

// Form of a two-pass D2Q9 step: separate passes, or one launch of 8 x 8 or 32 x 8 tiles.
enum PlaneShape { kPlaneSeparate, kPlaneSmall, kPlaneLarge };

}  // namespace lbmh

struct lbm_solver {
    int lattice, D, Q, storage;
    int nx, ny, nz;
    int64_t N;
    bool solids;
    hipStream_t stream;
    char *ws;
    lbmh::Layout L;
    int64_t step;
    int phase;  // AA-pattern layout: 0 natural, 1 swapped
    int scheme;
    int cur;        // record pair that holds the previous step's moments (lagged scheme)
    bool have_prev; // whether that pair is valid (lagged scheme)
    double RT, nu_f, nu_eff_ref, eta_eff, b[3], rho0;
    int nu_eff_pow;
    int shift;          // 16-bit population shift (LBM_SHIFT_*)
    uint32_t nb;        // boundary nodes
    bool bc_outflow, bc_vp;  // outflow nodes, velocity or pressure nodes present
    bool bc_visc;            // face velocity nodes whose density takes the viscous term
    int bc_scheme, bc_rho_rule;
    int picard_iters;
    double picard_omega;
    bool analytic;      // analytic porosity derivatives in L.deps
    lbm::Tiling tiles;  // 256-cell tiles, blocked, in XCD-contiguous ranges: collision and others
    lbm::Tiling mtiles; // the same of the moment and lagged passes (see run_tiles)
    bool fused_vc;      // velocity correction inside the collision pass (k_collide_vc)
    // whole step in one launch (k_plane_step): phase 0 in L.f, phase 1 in L.f2
    lbmh::PlaneShape plane;
    bool solid_occ;     // runs with solids: under a quarter of the tiles solid-aware
    bool cached_mom, cached_col, cached_lag;  // cached population accesses (see lbm::cached)
    lbm::ZTiling ztiles;
    int device;         // HIP device current at creation
};

namespace lbmh {

// Lattice temperature in the arithmetic type.  In FP32 it is rounded so that 1 - RT is exact
// (RT' = 1 - fl(1 - fl(RT)), exact by Sterbenz's lemma): then the three factors 1 - P and
// (P -/+ xi)/2 of each axis of the product-form equilibrium sum to exactly 1 for a cell at rest.
// With the nearest float of 1/3 they sum to 1 - 3e-8 per axis, which drains about 1e-7 of the
// mass per step.  The change of RT is below 2 ulp (1.2e-7 relative for 1/3); FP64 keeps RT.
template <typename T>
T lattice_temperature(double RT) {
    if constexpr (std::is_same_v<T, float>) {
        const float rt = (float)RT;
        const float c = 1.0f - rt;  // rounded: 1 - rt needs one bit more than a float for 1/3
        return 1.0f - c;            // exact (Sterbenz), and 1 - (1 - c) == c
    } else {
        return (T)RT;
    }
}

template <typename T>
lbm::Phys<T> phys_of(const lbm_solver *h) {
    lbm::Phys<T> ph;
    ph.RT = lattice_temperature<T>(h->RT);
    ph.omr = (T)(1.0 - 3.0 * h->RT);
    ph.nu_ref = (T)h->nu_eff_ref;
    ph.eta_on = std::isnan(h->eta_eff) ? 0 : 1;
    ph.eta = ph.eta_on ? (T)h->eta_eff : T(0);
    ph.two_over_D = (T)(2.0 / (double)h->D);
    for (int a = 0; a < 3; ++a) ph.b[a] = (T)h->b[a];
    ph.nu_pow = h->nu_eff_pow;
    ph.rho0 = (T)h->rho0;
    ph.shift_a = h->shift == LBM_SHIFT_POROUS ? (float)h->rho0 : 0.0f;
    ph.shift_b = h->shift == LBM_SHIFT_POROUS ? 0.0f : (float)h->rho0;
    ph.deps = h->analytic ? reinterpret_cast<const T *>(h->ws + h->L.deps) : nullptr;
    ph.dN = (uint32_t)h->N;
    return ph;
}

inline lbm::Grid grid_of(const lbm_solver *h) { return lbm::Grid{h->nx, h->ny, h->nz, (uint32_t)h->N}; }


inline dim3 flat_grid(int64_t total) { return dim3((unsigned)((total + 255) / 256)); }

// Tiles of the fused correction-collision pass: tx x ty cells (nx % tx == 0, ny % ty == 0),
// marched through chunks of zc z-planes, the eight XCDs taking contiguous ranges of the
// x-fastest, then y, then chunk order (neighbouring tiles in y share their ring rows in the
// XCD's L2).  One workgroup fills a CU (LDS rings of 143 KB in FP32, 114 KB for the 16-bit
// forms, 146 KB in FP64), so the launch runs in rounds of 256 workgroups, 32 on each XCD, and
// takes rounds x (zc + 3) plane times: a chunk corrects and stages about three planes' worth
// before its first collision.  The chunk length with the smallest product is taken (the longest
// of equals, at most 128 planes).  As long as 256 workgroups allow, which it was before, leaves
// the second round nearly empty on many grids: 192^3 FP64 has 144 columns, 2 x 108 planes in
// 288 workgroups took 1.32 ms, 7 x 28 planes in 1008 take 0.82 ms; 256^3 keeps its two chunks of
// 128 planes.
inline lbm::ZTiling make_ztiling(int nx, int ny, int nz, int tx, int ty) {
    lbm::ZTiling z{};
    z.ntx = nx / tx;
    z.nty = ny / ty;
    const int64_t cols = (int64_t)z.ntx * z.nty;
    int64_t best = INT64_MAX;
    for (int zc = std::min(nz, 128); zc >= std::min(nz, 4); --zc) {
        const int nch = (nz + zc - 1) / zc;
        const int64_t per = (cols * nch + 7) / 8;
        const int64_t cost = (per + 31) / 32 * (zc + 3);
        if (cost >= best) continue;
        best = cost;
        z.zc = zc;
        z.nch = nch;
        z.per = (uint32_t)per;
    }
    return z;
}

// Width of the rectangular row tiles (256 x 1, 128 x 2 or 64 x 4 cells) of an nx x ny plane: the
// one with the fewest lanes past the grid's edges, times `factor` for each doubling of the width.
// Lanes past a row's end idle in a working wave; a row past the plane's edge is a wave that ends
// early and counts `edge` of one.
inline int tile_x(int nx, int ny, double factor, double edge, double *lanes = nullptr) {
    int best = 0;
    double cost = 0.0, f = 1.0;
    for (int tx = 64; tx <= 256; tx *= 2, f *= factor) {
        const int ty = 256 / tx;
        const double rows = (1 - edge) * ny + edge * ((ny + ty - 1) / ty * ty);
        const double c = f * ((nx + tx - 1) / tx * tx) * rows;
        if (best == 0 || c < cost) {
            cost = c;
            best = tx;
        }
    }
    if (lanes) *lanes = cost;
    return best;
}

// Width for the passes that stage nothing: a wider tile is worth 3 % of idle lanes per doubling
// (fewer tile edges in x).  us per step of the separate FP32 passes at widths 64 / 128 / 256: 320 x
// 192 x 150 823 / 828 / 1,023; 384 x 192 x 192 1,280 / 1,251 / 1,443; 448 x 160 x 100 617 / 659 /
// 650; 256 x 192 x 192 869 / 857 / 827; FP64 192^3 1,319 / 1,507 / 1,340.  Few rows, 64 and 256
// wide: FP32 192 x 1 x 4096 66 / 58, 448 x 3 x 2048 215 / 224, FP64 473 / 495.
inline int rect_tile_x(int nx, int ny) { return tile_x(nx, ny, 0.97, 0.12); }

// Tiles of the cell passes: rectangular tiles of tx cells along x, or packed rows, so that rows of,
// say, 70 cells do not leave most of a second wave idle.
inline lbm::Tiling make_tiling(int nx, int ny, int nz, bool packed, int tx) {
    if (packed) return lbm::packed_tiling(nx, ny, nz, nx >= 2 ? ~uint64_t(0) / (uint64_t)nx + 1 : 0);
    lbm::Tiling t{};
    t.tx = tx;
    t.ltx = t.tx == 256 ? 8 : (t.tx == 128 ? 7 : 6);
    t.ty = 256 / t.tx;
    t.ntx = (nx + t.tx - 1) / t.tx;
    t.nty = (ny + t.ty - 1) / t.ty;
    lbm::block_tiles(t, nz);
    return t;
}

// Tiles of the 16-bit moment and lagged passes without solids.
// Rectangular tiles stage the porosity of the decode (the 26 neighbours of a D3Q27 cell) in LDS.
// The narrowest has the smallest halo (64 x 4: 1,188 values, 256 x 1: 2,322), which the moment pass
// feels (256 x 192 x 192 FP16, widths 64 / 128 / 256: 161 / 173 / 184 us) and the lagged pass
// hardly (224^3 BF16 675 / 672 / 687 us) except on D2Q9, where it has less else to do (65,536 x 3:
// 7.4 and 9.4 us); but three of its four rows lie past the edge of a plane of one row, and each
// stages all the same (256 x 1 x 4096 FP16, 64 and 256 wide: moments 44 and 26 us, lagged 86 and
// 52; 512 x 3 x 2048 lagged 171 and 160).
// Packed rows (can_pack: a ragged D3Q27 run) read that porosity through the caches, at some three
// times the moment pass's time per lane under the porous shift and over twice the lagged pass's
// (packed and rectangular, 192 x 160 rows of 9 cells: moments 13 and 31 us, lagged 25 and 77; of
// 25: 33 and 30, 51 and 72; of 37: 46 and 30, 96 and 72; 256 x 256 rows of 30: lagged 159 and 146).
// The lattice-weight shift needs none of it, and packing pays from a fifth of idle lanes (192 x 160
// rows of 66: moments 28 and 52 us, of 17: 11 and 30; 150^3 lagged 184 and 206).
inline lbm::Tiling moment_tiles(int nx, int ny, int nz, bool d3, bool can_pack, bool lagged,
                                bool weights) {
    double lanes;
    const int tx = tile_x(nx, ny, lagged && d3 ? 1.01 : 1.07, 0.25, &lanes);
    const double packed = (weights ? 1.2 : (lagged ? 2.35 : 3.0)) * nx * ny;
    return make_tiling(nx, ny, nz, can_pack && packed < lanes, tx);
}

// Lanes of a pass over one plane, those past the grid's edges included.
inline int64_t tile_lanes(const lbm::Tiling &t) { return (int64_t)256 * t.ntx * t.nty; }

// Grid of a cell pass: workgroups of one tile, padded to the same number on each XCD.
inline dim3 tile_grid(const lbm::Tiling &t) { return dim3((unsigned)(8 * (int64_t)t.per)); }

template <typename T>
T *ws_ptr(const lbm_solver *h, size_t off) {
    return reinterpret_cast<T *>(h->ws + off);
}

// Offset of the population buffer that holds the current state.
inline size_t f_off(const lbm_solver *h) {
    return h->plane != kPlaneSeparate && h->phase ? h->L.f2 : h->L.f;
}

inline const uint8_t *mask_ptr(const lbm_solver *h) {
    return h->solids ? reinterpret_cast<const uint8_t *>(h->ws + h->L.mask) : nullptr;
}

inline const uint8_t *tsolid_ptr(const lbm_solver *h) {
    return h->solids ? reinterpret_cast<const uint8_t *>(h->ws + h->L.tsolid) : nullptr;
}

// Flat-tile flags exist for differenced porosity derivatives only (analytic runs: null).
inline const uint8_t *tflat_ptr(const lbm_solver *h) {
    return h->analytic ? nullptr : reinterpret_cast<const uint8_t *>(h->ws + h->L.tflat);
}

// Tiles of a run's passes.
struct RunTiles {
    lbm::Tiling cells;    // collision, velocity correction and the passes at creation and reading
    lbm::Tiling moments;  // moment and lagged passes
};
RunTiles run_tiles(const lbm_params *p);

// Which passes access the populations through the caches: all when the step's working set (bytes)
// stays in the Infinity Cache, and on rows that are no whole cache lines the collision of FP32 and
// 16-bit storage and the 16-bit moment and lagged passes, these two not on packed rows without
// solids (measured at lbm::cached; the largest sets that gained held 231 MB, the smallest that lost
// 280 MB).  There they lose like FP32's moment pass (FP16, lattice-weight shift, non-temporal and
// cached: 200^3 moments 120 and 135 us, 81 x 256 x 256 74 and 91; 81 x 192 x 160 lagged pass 111 and
// 121; with solids, 70 x 192 x 192 moments 101 and 92).
constexpr int64_t kCachedSet = 240 << 20;
struct CachedPasses {
    bool moments, collide, lagged;
};
inline CachedPasses cached_passes(int64_t set, int storage, bool ragged, bool staged_ragged) {
    if (set <= kCachedSet) return {true, true, true};
    const bool half = storage == LBM_F16_SHIFTED || storage == LBM_BF16_SHIFTED;
    return {half && staged_ragged, storage != LBM_F64 && ragged, half && staged_ragged};
}
inline void set_cached(lbm_solver *h, const CachedPasses &c) {
    h->cached_mom = c.moments;
    h->cached_col = c.collide;
    h->cached_lag = c.lagged;
}
// Bytes a step of the run works on: populations, static fields and records.
inline int64_t step_bytes(const lbm_solver *h) {
    const int s = h->storage == LBM_F64 ? 8 : 4;
    const int sp = h->storage == LBM_F64 ? 8 : (h->storage == LBM_F32 ? 4 : 2);
    return h->N * (h->Q * sp + (3 + (h->scheme == LBM_SCHEME_LAGGED ? 16 : 8)) * s);
}
// Rows of populations that are no whole cache lines, and such rows in runs that have solids or whose
// moment tiles are not packed.
inline bool ragged_lines(const lbm_solver *h) {
    const int sp = h->storage == LBM_F64 ? 8 : (h->storage == LBM_F32 ? 4 : 2);
    return (int64_t)h->nx * sp % 128 != 0;
}
inline bool staged_ragged(const lbm_solver *h) {
    return ragged_lines(h) && (h->solids || !h->mtiles.packed);
}

// Workspace layout of a run with the shape and options of p (validates them; host only).
int run_layout(const lbm_params *p, Layout *L);

// Enqueue one D2Q9 step of a run stepped in one launch (lbm_plane.hip).
void launch_plane_step(const lbm_solver *h);

// Enqueue the statistics of the current state into res (8 doubles, the lbm_stats slots) with the
// per-block partial sums in part, without synchronising; defined with the solver kernels.
int enqueue_stats(lbm_solver *h, double *part, double *res);

// The same, with the partial sums and the result in the solver's workspace.
inline int enqueue_stats(lbm_solver *h) {
    return enqueue_stats(h, ws_ptr<double>(h, h->L.part), ws_ptr<double>(h, h->L.res));
}

}  // namespace lbmh

