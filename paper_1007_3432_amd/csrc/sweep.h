// Host-side planning and launch of one Q = M^T M sweep with a given op.
#pragma once

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>

#include "cgtiles.h"
#include "internal.h"
#include "stencil.h"

namespace hub {

// Tile shapes of the fused d = 1 kernel: TX sites in x x TT slices.
enum D1Tile { kD1_256x8 = 0, kD1_128x8, kD1_64x8, kD1_256x4, kD1_256x16, kD1_128x16,
              kD1_256x2, kD1_256x1, kD1_128x4, kD1_64x4, kD1_Count };
struct D1Shape { int tx, tt; };
static constexpr D1Shape kD1Shapes[kD1_Count] = {
    {256, 8}, {128, 8}, {64, 8}, {256, 4}, {256, 16}, {128, 16},
    {256, 2}, {256, 1}, {128, 4}, {64, 4}};

// Tile shapes of the fused d = 3 kernel: whole rows of NX x TY x TZ, swept
// by blocks of `block` lanes.  Mixed-precision solves (and with them the
// serving kernel, which must take the same steps) use 256-lane tiles only.
enum D3Tile { kD3_8x8x8 = 0, kD3_16x4x4, kD3_16x8x8, kD3_32x4x4, kD3_32x8x4, kD3_64x4x4,
              kD3_16x8x4, kD3_32x8x8_512, kD3_64x4x4_512, kD3_64x8x4_512, kD3_16x8x8_512,
              kD3_32x8x4_512, kD3_32x4x4_512, kD3_16x8x4_512, kD3_8x8x8_512, kD3_Count };
struct D3Shape { int nx, ty, tz, block; };
static constexpr D3Shape kD3Shapes[kD3_Count] = {
    {8, 8, 8, 256}, {16, 4, 4, 256}, {16, 8, 8, 256}, {32, 4, 4, 256}, {32, 8, 4, 256},
    {64, 4, 4, 256}, {16, 8, 4, 256}, {32, 8, 8, 512}, {64, 4, 4, 512}, {64, 8, 4, 512},
    {16, 8, 8, 512}, {32, 8, 4, 512}, {32, 4, 4, 512}, {16, 8, 4, 512}, {8, 8, 8, 512}};

enum SweepKind { kSweepD1 = 0, kSweepD3, kSweepRows, kSweepGeneric };

// Positions a lane of the row tiles handles at most, and lanes of a block.
struct RowsLevel { int own, halo_x, halo_y; };
constexpr RowsLevel kRowsLevels[] = {{1, 2, 1}, {1, 3, 2}, {2, 4, 2}, {2, 7, 4}};
constexpr int kRowsLevelCount = 4, kRowsBlock = 512;
constexpr int kRowsLdsMax = 64 * 1024;  // two blocks and more per CU

// Pair tiles of the d = 1 sweep (FP64, nx even): TX sites x TT slices.
enum D1PTile { kD1P_512x2 = 0, kD1P_256x2, kD1P_128x2, kD1P_512x4, kD1P_512x1, kD1P_Count };
static constexpr D1Shape kD1PShapes[kD1P_Count] = {
    {512, 2}, {256, 2}, {128, 2}, {512, 4}, {512, 1}};

struct SweepPlan {
    int kind;      // SweepKind
    bool fused;    // single pass (all but kSweepGeneric)
    bool pair;     // kSweepD1 with the pair tile (variant is a D1PTile)
    int variant;   // D1Tile, D1PTile, D3Tile or level of the row tiles
    int tiles_x;   // d = 1
    int tiles_y, tiles_z, tc;  // d = 2, 3: tiles and slices per block
    int lds;       // row tiles: elements of LDS
    int ntiles;    // tiles of one sweep = deposits of its reductions
    int grid;      // blocks of the sweep kernel (pass 2 when generic)
};

// Tuning aids: HUB_D1_TILE=<TX>x<TT>,
// HUB_D3_TILE=<NX>x<TY>x<TZ>[@512], HUB_D3_TC=<slices per block>, HUB_SWEEP=generic.
inline const char* env_or_null(const char* k) { return std::getenv(k); }

inline int d1_tile_override() {
    static int v = [] {
        const char* e = env_or_null("HUB_D1_TILE");
        if (!e) return -1;
        for (int k = 0; k < kD1_Count; ++k) {
            char buf[32];
            std::snprintf(buf, sizeof(buf), "%dx%d", kD1Shapes[k].tx, kD1Shapes[k].tt);
            if (std::strcmp(buf, e) == 0) return k;
        }
        return -1;
    }();
    return v;
}

inline int d3_tile_override() {
    static int v = [] {
        const char* e = env_or_null("HUB_D3_TILE");
        if (!e) return -1;
        for (int k = 0; k < kD3_Count; ++k) {
            char buf[32];
            if (kD3Shapes[k].block == 256)
                std::snprintf(buf, sizeof(buf), "%dx%dx%d", kD3Shapes[k].nx, kD3Shapes[k].ty,
                              kD3Shapes[k].tz);
            else
                std::snprintf(buf, sizeof(buf), "%dx%dx%d@%d", kD3Shapes[k].nx, kD3Shapes[k].ty,
                              kD3Shapes[k].tz, kD3Shapes[k].block);
            if (std::strcmp(buf, e) == 0) return k;
        }
        return -1;
    }();
    return v;
}

inline int d1p_tile_override() {
    static int v = [] {
        const char* e = env_or_null("HUB_D1P_TILE");
        if (!e) return -1;
        if (std::strcmp(e, "off") == 0) return -2;
        for (int k = 0; k < kD1P_Count; ++k) {
            char buf[32];
            std::snprintf(buf, sizeof(buf), "%dx%d", kD1PShapes[k].tx, kD1PShapes[k].tt);
            if (std::strcmp(buf, e) == 0) return k;
        }
        return -1;
    }();
    return v;
}

inline int env_int(const char* k, int dflt) {
    const char* e = env_or_null(k);
    return e ? std::atoi(e) : dflt;
}

inline bool force_generic() {
    static bool v = [] {
        const char* e = env_or_null("HUB_SWEEP");
        return e && std::strcmp(e, "generic") == 0;
    }();
    return v;
}

// The row tiles for a geometry (p->kind stays kSweepGeneric when none fits):
// the cut with the fewest positions gone through per owned site, counting a
// slice per chunk for its prologue.
inline void plan_rows(const Geom& g, SweepPlan* p) {
    double best = 1e30;
    // Each tile height once: the next count of tiles that makes it smaller.
    auto next = [&](int t) { return t > 1 ? ceil_div(g.nx, t - 1) : g.nx + 1; };
    for (int cy = 1, ty = g.nx; cy <= g.nx; cy = next(ty)) {
        ty = ceil_div(g.nx, cy);
        if ((long long)ty * g.nx > 2 * kRowsBlock) continue;
        for (int cz = 1, tz = g.nx; cz <= (g.d == 3 ? g.nx : 1); cz = next(tz)) {
            tz = g.d == 3 ? ceil_div(g.nx, cz) : 1;
            const long long rows = (long long)ty * tz;
            if (rows * g.nx > 2 * kRowsBlock) continue;
            const int own = g.nx * (int)rows;
            const int hx = g.nx * (g.d == 3 ? rows_halo_x<3>(ty, tz) : rows_halo_x<2>(ty, tz));
            const int hy = g.nx * (g.d == 3 ? rows_halo_y<3>(ty, tz) : rows_halo_y<2>(ty, tz));
            const int lds = g.d == 3 ? rows_lds_elems<3>(g.nx, ty, tz)
                                     : rows_lds_elems<2>(g.nx, ty, tz);
            if (8 * lds > kRowsLdsMax) continue;  // FP64 also in the mixed solver
            // Where the halo is over three times the tile, two passes read less
            // (d = 3 90^3 x 6 64.0 us against 60.0; see also rows_pay).
            if (hx > 3 * own) continue;
            const int tiles = cy * cz;
            // About two blocks per CU, chunks of 2 to 16 slices (256, 768 and
            // 1024 blocks were up to 40% slower on one lattice or another).
            const long long tcl = ((long long)g.nt * tiles + 511) / 512;
            const int tc = (int)(tcl < 2 ? 2 : (tcl > 16 ? 16 : tcl));
            const int chunks = ceil_div(g.nt, tc);
            for (int l = 0; l < kRowsLevelCount; ++l) {
                const RowsLevel& K = kRowsLevels[l];
                if (own > K.own * kRowsBlock || hx > K.halo_x * kRowsBlock ||
                    hy > K.halo_y * kRowsBlock)
                    continue;
                // Waves of blocks over the chip, times what a block does.
                const double turns = std::ceil(tiles * chunks / 512.0);
                const double cost = turns * (tc + 1) * (3.0 * K.own + K.halo_x + 2.0 * K.halo_y + 2.0);
                if (cost >= best) continue;
                best = cost;
                p->kind = kSweepRows;
                p->variant = l;
                p->tiles_y = cy;
                p->tiles_z = cz;
                p->tc = tc;
                p->lds = lds;
                p->ntiles = p->grid = tiles * chunks;
            }
        }
    }
}

// Whether the row tiles of plan_rows are faster than two passes: the time of a
// block's march, X = turns * (slices + 1) * positions of a lane, against a line in
// the number of sites.  A turn is as many blocks as the chip holds: two per CU of
// those that need at most 128 registers a lane, else one.  (Taken as two for all
// of them, FP64 solves and Chebyshev factors came to the row tiles where they
// are up to 1.9 times slower, d = 3 72^3 x 7, and bare products up to 1.5 times.)
// The lines are drawn so that of 230 to 340 lattices measured (d = 2 with nx = 5
// to 1024, d = 3 with nx = 3 to 128, 2 to 600 slices) none is over 4% slower than
// in two passes (factors on 4^3 6%).  us, two passes and row tiles: bare FP64
// products, the two with their scratch vector, 63^3 x 17 92 and 70, 67^3 x 17 69
// and 76; factors 29^3 x 40 15.7 and 17.0 a sweep, x 100 43 and 35, FP64 CG 40^3 x 7 25
// and 28 an iteration, x 17 45 and 43; FP32 CG 72^3 x 3 107 and 86, x 7 85 and 93.
inline bool rows_pay(const Geom& g, const SweepPlan& p, bool f64, bool solve, bool factor) {
    const RowsLevel& K = kRowsLevels[p.variant];
    const bool bare = !solve && !factor, d2 = g.d == 2;
    bool two = true;  // blocks per CU
    switch (p.variant) {
        case 0: break;
        case 1: two = d2 || bare || !f64; break;
        case 2: two = bare ? !f64 || d2 : !f64 && d2; break;
        default: two = false;
    }
    const double V = g.V;
    double x = std::ceil(p.grid / (two ? 512.0 : 256.0)) * (p.tc + 1) *
               (3 * K.own + K.halo_x + 2 * K.halo_y + 2);
    if (bare) return x <= 112 + 1.4e-4 * V;
    if (!f64) return x <= 40 + 2.2e-4 * V;
    // Two blocks share their CU; the largest phase A spills.
    if (two && p.grid > 256) x *= 1.3;
    if (solve && p.variant == 3) x *= 1.3;
    // (From some 3.3 million sites on two passes go to HBM.)
    return x <= 28 + (V > 3.3e6 ? 1.3e-4 : 1.0e-4) * V;
}

// f64: the sweep's ops are FP64 throughout, so the pair tile may serve d = 1.
// solve: the plan of a solver (CG phase A and the true residual), which may
// take another d = 3 tile than the bare product.  factor: of a Chebyshev factor's
// sweeps, which have their scratch vector anyway.
inline SweepPlan plan_sweep(const Geom& g, bool f64, bool solve = false, bool factor = false) {
    SweepPlan p{};
    p.kind = kSweepGeneric;
    p.variant = -1;
    p.pair = false;
    const int pv = d1p_tile_override();
    if (!force_generic() && g.d == 1 && f64 && g.nx % 2 == 0 && pv != -2) {
        int v = pv;
        if (v < 0) v = g.nx >= 512 ? kD1P_512x2 : (g.nx >= 256 ? kD1P_256x2 : kD1P_128x2);
        p.kind = kSweepD1;
        p.pair = true;
        p.variant = v;
        p.tiles_x = ceil_div(g.nx, kD1PShapes[v].tx);
        p.ntiles = p.tiles_x * ceil_div(g.nt, kD1PShapes[v].tt);
        p.grid = p.ntiles;
    } else if (!force_generic() && g.d == 1) {
        int v = d1_tile_override();
        if (v < 0) v = g.nx >= 256 ? kD1_256x4 : (g.nx >= 128 ? kD1_128x4 : kD1_64x4);
        p.kind = kSweepD1;
        p.variant = v;
        p.tiles_x = ceil_div(g.nx, kD1Shapes[v].tx);
        p.ntiles = p.tiles_x * ceil_div(g.nt, kD1Shapes[v].tt);
        p.grid = p.ntiles;
    } else if (!force_generic() && g.d == 3) {
        int v = d3_tile_override();
        if (v >= 0 && (kD3Shapes[v].nx != g.nx || (!f64 && solve && kD3Shapes[v].block != 256)))
            v = -1;
        if (v < 0) {
            // Measured on MI355X (bare FP64 and FP32 sweeps on 8^3 x 80,
            // 16^3 x 160, 32^3 x 256, 64^3 x 32): FP64 sweeps run best on
            // 512-lane blocks for nx = 16, 32 (fewer registers per lane than
            // the 256-lane tiles, whose FP64 CG variant needs 256 VGPRs), bare
            // FP32 ones for nx = 32, 64; mixed-precision solves stay on
            // 256-lane tiles (their sums are laid out by tile).
            switch (g.nx) {
                case 8: v = kD3_8x8x8; break;
                case 16: v = f64 ? kD3_16x8x4_512 : kD3_16x4x4; break;
                // Eight planes of z a tile wherever its blocks fill the chip
                // (a lane's four sites in z give each other their neighbours):
                // bare product, 32x8x4 and 32x8x8, us: FP64 32^3 x 16 6.9 and
                // 8.6, x 24 7.9 and 8.5, x 25 8.9 and 8.5, x 64 16.4 and 14.4, x
                // 144 34.7 and 26.1, x 256 40 and 40; FP32 x 24 6.3 and 6.5, x 25
                // 6.9 and 6.6, x 256 24 and 20.6, x 257 33 and 31.  In FP64 a CU
                // holds one block of it, and two of 32x8x4, which fill the last
                // turn better: x 257 53 and 66, x 384 57 and 68, x 400 69 and 69,
                // x 512 73 and 76, x 513 86 and 100, x 640 116 and 126, but x 641
                // 129 and 124, x 768 138 and 131, x 900 174 and 164.
                case 32: {
                    const int last = (ceil_div(g.nt, 16) - 1) % 16;  // of 16 chunks a turn
                    const bool tall = g.nt >= 25 && (!f64 || g.nt <= 256 ||
                                                     (g.nt > 512 && last >= 8));
                    if (solve) v = f64 ? kD3_32x8x8_512 : kD3_32x8x4;
                    else v = tall ? kD3_32x8x8_512 : kD3_32x8x4_512;
                    break;
                }
                // Bare FP32 products on 512 lanes, unless the second chunk of 16
                // slices of their unrolled march would repeat half the first: 256
                // and 512 lanes, us, 64^3 x 16 18.1 and 17.6, x 17 19.2 and 25.8,
                // x 20 20.3 and 25.3, x 24 23.4 and 24.6, x 28 25.6 and 24.7, x 32
                // 28.4 and 25.1, x 33 43 and 38, x 64 51 and 47.
                case 64:
                    v = f64 || (!solve && (g.nt <= 16 || g.nt >= 26)) ? kD3_64x4x4_512
                                                                      : kD3_64x4x4;
                    break;
                default: v = -1;
            }
        }
        if (v >= 0) {
            const D3Shape sh = kD3Shapes[v];
            p.kind = kSweepD3;
            p.variant = v;
            p.tiles_y = g.nx / sh.ty;
            p.tiles_z = g.nx / sh.tz;
            const int tiles = p.tiles_y * p.tiles_z;
            // Slices per block: the sweeps ran best with about 128K lanes in
            // the grid (one 512-lane or two 256-lane blocks per CU), long
            // marches amortising each block's prologue slice.
            long long tcl = ((long long)g.nt * tiles * sh.block + 131071) / 131072;
            int tc = (int)(tcl < 2 ? 2 : (tcl > 16 ? 16 : tcl));
            tc = env_int("HUB_D3_TC", tc);
            if (tc < 1) tc = 1;
            p.tc = tc;
            p.ntiles = tiles * ceil_div(g.nt, tc);
            p.grid = p.ntiles;
        }
    }
    if (p.kind == kSweepGeneric && !force_generic() && g.d > 1) {
        // The search takes 1 to 3 us, as long as a launch: the last one of
        // each thread is kept, by the extents that it depends on.
        struct Last { int d, nx, nt; SweepPlan p; };
        static thread_local Last last{0, 0, 0, {}};
        if (last.d != g.d || last.nx != g.nx || last.nt != g.nt) {
            SweepPlan q = p;
            plan_rows(g, &q);
            last = {g.d, g.nx, g.nt, q};
        }
        if (last.p.kind == kSweepRows && rows_pay(g, last.p, f64, solve, factor)) p = last.p;
    }
    if (p.kind == kSweepGeneric) p.ntiles = p.grid = ceil_div(g.V, 256);
    p.fused = p.kind != kSweepGeneric;
    return p;
}

// Doubles of deposit space any reduction over this geometry may need:
// kMaxNP sums for each tile of the largest grid (sweep or element-wise).
inline int max_partials(const Geom& g) {
    const SweepPlan p = plan_sweep(g, false, true), q = plan_sweep(g, true),
                    r = plan_sweep(g, true, true);
    const int e = elem_tiles(g.V);
    int m = p.ntiles > e ? p.ntiles : e;
    m = q.ntiles > m ? q.ntiles : m;
    m = r.ntiles > m ? r.ntiles : m;
    return kMaxNP * m;
}

// Slices in flight per block of the d = 3 sweep.  Measured on MI355X: FP32
// ops gain from loading two slices ahead (the mixed-precision CG iteration
// on 32^3 x 256 with FP16 links: 75.6 -> 67.0 us); FP64 ops do not (the
// FP64 sweep and CG on the same lattice: 57.3 -> 58.9 us, 154 -> 159 us).
template <class Op>
constexpr int d3_prefetch_depth() {
    return sizeof(typename Op::acc_t) == 4 ? 2 : 1;
}

// Slices per block of the completely unrolled d = 3 march, with two slices in
// flight.  Only the bare products take it, on 512-lane tiles, from the plans
// whose blocks march the most slices: on 32x8x4 tiles FP64 32^3 x 256 58.0 -> 54
// us, FP32 32^3 x 256 28.5 -> 26.7, 64^3 x 32 29.2 -> 26.8.  The FP64 CG phase A would
// spill registers on it (140 -> 198 us per iteration), the mixed one gains
// nothing.  (17 slices, so that chunks do not start at multiples of 4 MiB: 51.4
// us on the first, but 56.0 for 52.5 on FP64 64^3 x 32 and 26.4 for 25.1 on
// 32^3 x 128.)
constexpr int kD3Unroll = 16;
inline bool d3_unrolled_ok(const Geom& g, const SweepPlan& P) {
    return P.tc == 16 && g.nt >= kD3Unroll;
}

template <class Op, int D, int L>
inline void launch_rows_l(const Geom& g, const SweepPlan& P, const Op& op, double* partials,
                          hipStream_t st) {
    constexpr RowsLevel K = kRowsLevels[L];
    k_mtm_rows<Op, D, K.own, K.halo_x, K.halo_y, kRowsBlock>
        <<<P.grid, kRowsBlock, (size_t)P.lds * sizeof(typename Op::acc_t), st>>>(
            g, op, P.tiles_y, P.tiles_z, P.tc, partials);
}
template <class Op, int D>
inline void launch_rows(const Geom& g, const SweepPlan& P, const Op& op, double* partials,
                        hipStream_t st) {
    switch (P.variant) {
        case 0: launch_rows_l<Op, D, 0>(g, P, op, partials, st); break;
        case 1: launch_rows_l<Op, D, 1>(g, P, op, partials, st); break;
        case 2: launch_rows_l<Op, D, 2>(g, P, op, partials, st); break;
        default: launch_rows_l<Op, D, 3>(g, P, op, partials, st); break;
    }
}

// One sweep: z = Q in, consumed by op.out().  y: scratch of g.V acc_t
// elements, used by the generic path only.  A reducing op's deposits go to
// partials; with finalize, a one-block kernel then adds them (op.finish),
// otherwise the next kernel does.
template <class Op>
hub_status launch_q(const Geom& g, const SweepPlan& P, const Op& op,
                    typename Op::acc_t* y, double* partials, hipStream_t st,
                    bool finalize = true) {
    if (P.kind == kSweepD1 && P.pair) {
        if constexpr (op_marches<Op>::value) {
            // The bare product takes the marching tile (8 slices per
            // wavefront, all but the last stage's loads issued up front) on
            // lattices of 2^19 sites and more, unless a pair tile is forced
            // for tuning.  Measured on MI355X: at 2^20 sites and above the
            // marching tile is faster (d=1 2048x512 streamed from HBM 8.0 ->
            // 6.8 us), at 2^18 and below the shorter chains of the two-slice
            // tile win (d=1 1024x256: 2.8 vs 4.2 us).  The plan's deposit
            // count is the pair tile's, so only ops without a reduction may
            // march.
            static_assert(!Op::kReduce, "a marching sweep leaves no pair-tile deposits");
            if (d1p_tile_override() < 0 && g.V >= (1 << 19)) {
                constexpr int kTS = 8, kPF = 8;
                const int tx = kD1PShapes[P.variant].tx;
                const int ntiles = P.tiles_x * ceil_div(g.nt, kTS);
                switch (tx) {
                    case 512:
                        k_mtm_d1m<Op, 512, kTS, kPF><<<ntiles, 256, 0, st>>>(g, op, P.tiles_x,
                                                                             ntiles, partials);
                        break;
                    case 256:
                        k_mtm_d1m<Op, 256, kTS, kPF><<<ntiles, 128, 0, st>>>(g, op, P.tiles_x,
                                                                             ntiles, partials);
                        break;
                    default:
                        k_mtm_d1m<Op, 128, kTS, kPF><<<ntiles, 64, 0, st>>>(g, op, P.tiles_x,
                                                                            ntiles, partials);
                        break;
                }
                HUB_HIP(hipGetLastError());
                return HUB_OK;
            }
        }
        if constexpr (op_has_pair<Op>::value) {
            switch (P.variant) {
#define HUB_D1P_CASE(K, TX, TT)                                                         \
    case K:                                                                             \
        k_mtm_d1p<Op, TX, TT><<<P.grid, TX / 2, 0, st>>>(g, op, P.tiles_x, P.ntiles,     \
                                                          partials);                     \
        break;
                HUB_D1P_CASE(kD1P_512x2, 512, 2)
                HUB_D1P_CASE(kD1P_256x2, 256, 2)
                HUB_D1P_CASE(kD1P_128x2, 128, 2)
                HUB_D1P_CASE(kD1P_512x4, 512, 4)
                HUB_D1P_CASE(kD1P_512x1, 512, 1)
#undef HUB_D1P_CASE
                default:
                    return set_error(HUB_E_INVALID, "internal: bad d=1 pair tile variant");
            }
        } else {
            return set_error(HUB_E_INVALID, "internal: op has no pair access");
        }
    } else if (P.kind == kSweepD1) {
        switch (P.variant) {
#define HUB_D1_CASE(K, TX, TT)                                                             \
    case K:                                                                                \
        k_mtm_d1<Op, TX, TT><<<P.grid, TX, 0, st>>>(g, op, P.tiles_x, P.ntiles, partials); \
        break;
            HUB_D1_CASE(kD1_256x8, 256, 8)
            HUB_D1_CASE(kD1_128x8, 128, 8)
            HUB_D1_CASE(kD1_64x8, 64, 8)
            HUB_D1_CASE(kD1_256x4, 256, 4)
            HUB_D1_CASE(kD1_256x16, 256, 16)
            HUB_D1_CASE(kD1_128x16, 128, 16)
            HUB_D1_CASE(kD1_256x2, 256, 2)
            HUB_D1_CASE(kD1_256x1, 256, 1)
            HUB_D1_CASE(kD1_128x4, 128, 4)
            HUB_D1_CASE(kD1_64x4, 64, 4)
#undef HUB_D1_CASE
            default:
                return set_error(HUB_E_INVALID, "internal: bad d=1 tile variant");
        }
    } else if (P.kind == kSweepD3) {
        if (g.nx != kD3Shapes[P.variant].nx)
            return set_error(HUB_E_INVALID, "internal: d=3 tile does not fit nx");
        switch (P.variant) {
#define HUB_D3_CASE(K, NX, TY, TZ, B)                                                    \
    case K:                                                                              \
        if constexpr (NX >= 32 && B == 512 && op_repeats<Op>::value) {                   \
            if (d3_unrolled_ok(g, P)) {                                                  \
                const int grid = P.tiles_y * P.tiles_z * ceil_div(g.nt, kD3Unroll);       \
                k_mtm_d3<Op, NX, TY, TZ, B, 2, kD3Unroll><<<grid, B, 0, st>>>(            \
                    g, op, P.tiles_y, P.tiles_z, kD3Unroll, partials);                    \
                break;                                                                   \
            }                                                                            \
        }                                                                                \
        if constexpr (B == 256 || sizeof(typename Op::acc_t) == 8 || !Op::kReduce)         \
            k_mtm_d3<Op, NX, TY, TZ, B, d3_prefetch_depth<Op>()>                          \
                <<<P.grid, B, 0, st>>>(g, op, P.tiles_y, P.tiles_z, P.tc, partials);      \
        else                                                                             \
            return set_error(HUB_E_INVALID, "internal: mixed solves take 256-lane tiles"); \
        break;
            HUB_D3_CASE(kD3_8x8x8, 8, 8, 8, 256)
            HUB_D3_CASE(kD3_16x4x4, 16, 4, 4, 256)
            HUB_D3_CASE(kD3_16x8x8, 16, 8, 8, 256)
            HUB_D3_CASE(kD3_32x4x4, 32, 4, 4, 256)
            HUB_D3_CASE(kD3_32x8x4, 32, 8, 4, 256)
            HUB_D3_CASE(kD3_64x4x4, 64, 4, 4, 256)
            HUB_D3_CASE(kD3_16x8x4, 16, 8, 4, 256)
            HUB_D3_CASE(kD3_32x8x8_512, 32, 8, 8, 512)
            HUB_D3_CASE(kD3_64x4x4_512, 64, 4, 4, 512)
            HUB_D3_CASE(kD3_64x8x4_512, 64, 8, 4, 512)
            HUB_D3_CASE(kD3_16x8x8_512, 16, 8, 8, 512)
            HUB_D3_CASE(kD3_32x8x4_512, 32, 8, 4, 512)
            HUB_D3_CASE(kD3_32x4x4_512, 32, 4, 4, 512)
            HUB_D3_CASE(kD3_16x8x4_512, 16, 8, 4, 512)
            HUB_D3_CASE(kD3_8x8x8_512, 8, 8, 8, 512)
#undef HUB_D3_CASE
            default:
                return set_error(HUB_E_INVALID, "internal: bad d=3 tile variant");
        }
    } else if (P.kind == kSweepRows) {
        if ((size_t)P.lds * sizeof(typename Op::acc_t) > kRowsLdsMax)
            return set_error(HUB_E_INVALID, "internal: row tile does not fit LDS");
        if (g.d == 2) launch_rows<Op, 2>(g, P, op, partials, st);
        else launch_rows<Op, 3>(g, P, op, partials, st);
    } else {
        if (!y) return set_error(HUB_E_INVALID, "internal: generic sweep needs scratch");
        const int grid = ceil_div(g.V, 256);
        k_gen_pass1<Op><<<grid, 256, 0, st>>>(g, op, y);
        k_gen_pass2<Op><<<grid, 256, 0, st>>>(g, op, y, partials);
    }
    if constexpr (Op::kReduce) {
        if (!partials) return set_error(HUB_E_INVALID, "internal: reduction needs deposits");
        if (finalize) k_finish_op<Op><<<1, 256, 0, st>>>(op, partials, P.ntiles);
    }
    HUB_HIP(hipGetLastError());
    return HUB_OK;
}

}  // namespace hub
