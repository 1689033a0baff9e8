// FP64 conjugate gradient on Q = M^T M (Sec. 4.1) with the whole solve
// resident on the chip: lattices too large for one workgroup and small enough
// that x, r, p, s = Q p and the links fit the registers of one block per CU.
//
// The last spatial dimension (z below; x itself for d = 1) and time are cut
// into Nz x Nt tiles, one block each; the other dimensions, `inner`, stay
// whole.  A lane keeps one inner index and every G-th (z, t) position of its
// block's tile.  The sums and the directions are arranged after Chronopoulos
// and Gear (1989), so that an iteration has one synchronisation of the grid:
//   1. w = Q r: r of tile and halo into LDS (P), y = M r on the tile and on
//      the sites around it that M^T reads into LDS (Y), w on the tile;
//   2. the tile's rim of w goes to global memory for the neighbours, and the
//      block's r.r and r.w to the grid sum (gridsum.h);
//   3. beta = r.r / (r.r before), p.Qp = r.w - beta r.r / (alpha before),
//      alpha = r.r / p.Qp; p = r + beta p, s = w + beta s, x += alpha p,
//      r -= alpha s.
//      On the halo, where w has come from the neighbours, s and r follow the
//      same recurrences: the block keeps the values that their owners have.
// The kernel ends when r.r meets tol, after a number of iterations, or when
// it cannot go on; the state is in memory then.  Convergence is decided
// between launches as in the other solvers: the true residual phi - Q x
// replaces r, and if it does not meet tol the iteration goes on from it,
// keeping p; the next p.Qp is then r.w + 2 beta r.s + beta^2 (p.Qp before), as
// r has lost its exact orthogonality to the step before.
//
// What bounds an iteration is the grid sum (2 to 2.5 us), the stores before
// and the halo read after it (1 us), and the LDS traffic of the stencils, where
// it was three kernels and 80 bytes a site of memory traffic.  Before and now,
// us an iteration: d = 1 256 x 128 9.4 and 3.0, 4096 x 128 15.2 and 4.3, 2048
// x 512 20.5 and 4.9; d = 2 33 x 60 11.9 and 3.4; d = 3 8^3 x 80 12.1 and 3.2,
// 16^3 x 128 17.2 and 5.8.  (Hestenes and Stiefel's arrangement, with two grid
// sums an iteration, took 4.5, 5.7, 7.0, 5.3, 4.8 and 11.0.)
#pragma once

#include <utility>

#include "gridsum.h"
#include "internal.h"

namespace hub {

// Positions a lane handles at most: its own sites, the sites around the tile
// where y is formed, and the halo of r.  Each level is a kernel; a lane holds
// 15 words for each of the first, 4 and 6 for each of the others, and two
// more for each of the first two where z is whole.  `whole`: that fits too.
struct ResLevel {
    int own, rim, halo;
    bool whole;
};
constexpr ResLevel kResLevels[] = {
    {1, 1, 2, true},   {2, 2, 4, true}, {3, 3, 6, true},   {4, 2, 3, true}, {4, 4, 10, true},
    {4, 6, 16, false}, {6, 3, 6, true}, {6, 5, 12, false}, {8, 2, 3, true}, {8, 4, 10, false}};
constexpr int kResLevelCount = 10;
constexpr int kResBlock = 512;

struct ResState {
    double rho;       // r.r before the step that r has taken last
    double alpha;     // of that step
    double pq;        // p.Qp of that step
    double phi2;
    double rho_true;  // |phi - Q x|^2 of the last recompute
    double rs;        // r.s after it
    int32_t iter;
    int32_t done;     // kRunning, kDoneIterConverged, kDoneBreakdown, kDoneMaxIter
    int32_t given_up;
    int32_t pad;
};

enum : int { kResFirst = 0, kResOn = 1, kResReplaced = 2 };

struct ResArgs {
    Geom g;
    int inner;   // sites of the dimensions that are not cut
    int Nz, Nt;  // tiles in z and time
    int G;       // (z, t) positions taken at a time: lanes / inner
    const double* A;
    const double* phi;
    double* x;
    double *R, *P, *S;  // r, p and s between launches
    double* W;   // 2 V: rim of w between blocks, in turns
    uint64_t* slots;
    ResState* st;
    double tol2;
    int max_iter;
    int iters;   // iterations of this launch at most
    int mode;    // kResFirst: starts the solve; kResReplaced: r was replaced
    int limit;   // reads before a wait is given up
};

// The index as the compiler sees it anew: neighbour addresses are formed where
// they are used, an add each, instead of being kept in registers (a dozen for
// every position) across the loop.
__device__ __forceinline__ int fresh(int i) {
    asm volatile("" : "+v"(i));
    return i;
}

// Values that have to be there at this point: the loads they come from are
// not held in registers beyond it.
__device__ __forceinline__ void settle(double& a, double& b) {
    asm volatile("" : "+v"(a), "+v"(b));
}

typedef __attribute__((address_space(3))) double lds_double;

template <int D, bool WHOLE, int KO, int KY, int KH>
__global__ __launch_bounds__(kResBlock) void k_cg_resident(ResArgs a) {
    constexpr int H = WHOLE ? 0 : 1;  // z halo of y; r has twice that
    extern __shared__ __align__(16) double res_lds[];
    const Geom& g = a.g;
    const int nz = g.nx, nt = g.nt, I = D == 1 ? 1 : a.inner;
    // Tiles next to each other in z, and then in time, are on the same XCD,
    // whose L2 then has most of what a block hands to its neighbours (16^3 x
    // 128 9.1 -> 5.9 us an iteration).
    const int tile = xcd_remap(blockIdx.x, gridDim.x);
    const int bz = tile % a.Nz, bt = tile / a.Nz;
    const int z0 = (int)((long long)bz * nz / a.Nz), Tz = (int)((long long)(bz + 1) * nz / a.Nz) - z0;
    const int t0 = (int)((long long)bt * nt / a.Nt), Tt = (int)((long long)(bt + 1) * nt / a.Nt) - t0;
    const int ZP = Tz + 4 * H, ZY = Tz + 2 * H;  // z extents of P and Y
    // LDS, in doubles from res_lds: the sums, P, Y, and one spare element that
    // positions past the end write.  Indices below are LDS byte addresses.
    constexpr int kP = GridSum::kLdsDoubles;
    const int base = (int)(uint32_t)(uintptr_t)(lds_double*)res_lds;
    const int kY = kP + ZP * (Tt + 2) * I, sink = base + 8 * (kY + ZY * (Tt + 1) * I);
    GridSum gs{a.slots, res_lds, a.limit, 0};
    auto lds = [](int byte) -> lds_double& { return *(lds_double*)(uintptr_t)(uint32_t)byte; };
    auto at = [](const double* v, int byte) {
        return reinterpret_cast<const double*>(reinterpret_cast<const char*>(v) + (uint32_t)byte);
    };
    auto at_w = [](double* v, int byte) {
        return reinterpret_cast<double*>(reinterpret_cast<char*>(v) + (uint32_t)byte);
    };

    const int grp = (int)threadIdx.x / I, m = (int)threadIdx.x - grp * I;
    const bool on = grp < a.G;
    // Inner neighbours of m.
    int in[4] = {0, 0, 0, 0};
    if constexpr (D >= 2) {
        const int cx = m % g.nx;
        in[0] = 8 * (cx + 1 == g.nx ? 1 - g.nx : 1);
        in[1] = 8 * (cx == 0 ? g.nx - 1 : -1);
    }
    if constexpr (D == 3) {
        const int cy = m / g.nx;
        in[2] = 8 * (cy + 1 == g.nx ? g.nx - I : g.nx);
        in[3] = 8 * (cy == 0 ? I - g.nx : -g.nx);
    }
    auto pidx = [&](int z, int t) { return base + 8 * (kP + ((t + 1) * ZP + z + 2 * H) * I + m); };
    auto yidx = [&](int z, int t) { return base + 8 * (kY + (t * ZY + z + H) * I + m); };
    // Site of (z, t) relative to the tile; images around the lattice wrap.
    auto site = [&](int z, int t) {
        int zz = (z0 + z) % nz, tt = (t0 + t) % nt;
        if (zz < 0) zz += nz;
        if (tt < 0) tt += nt;
        return 8 * (tt * g.vs + zz * I + m);
    };
    // Offsets of the z neighbours: +-I, or around the tile where z is whole.
    auto zup = [&](int z) { return 8 * (WHOLE && z == Tz - 1 ? -(Tz - 1) * I : I); };
    auto zdn = [&](int z) { return 8 * (WHOLE && z == 0 ? (Tz - 1) * I : -I); };

    // Own sites.  Positions past the end repeat the first one and are masked.
    int opi[KO], oyi[KO], ogi[KO];
    bool ook[KO], orim[KO];
    int ozu[KO], ozd[KO];  // used where z is whole
    double oa[KO], oap[KO];
    double x[KO], r[KO], p[KO], s[KO];
#pragma unroll
    for (int k = 0; k < KO; ++k) {
        int o = grp + a.G * k;
        ook[k] = on && o < Tz * Tt;
        if (!ook[k]) o = 0;
        const int z = o % Tz, t = o / Tz;
        opi[k] = pidx(z, t);
        oyi[k] = yidx(z, t);
        ogi[k] = site(z, t);
        orim[k] = ook[k] && (t == 0 || t == Tt - 1 || (H && (z < 2 || z >= Tz - 2)));
        ozu[k] = zup(z);
        ozd[k] = zdn(z);
        oa[k] = *at(a.A, ogi[k]);
        oap[k] = *at(a.A, site(z, t + 1));
    }
    // Sites around the tile where y is formed: z = -1, Tz on the tile's
    // slices, and the tile's z on the slice after it.
    int rpi[KY], ryi[KY];
    int rzu[KY], rzd[KY];
    double ra[KY];
    const int nrim = 2 * H * Tt + Tz;
#pragma unroll
    for (int k = 0; k < KY; ++k) {
        int o = grp + a.G * k;
        const bool ok = on && o < nrim;
        if (!ok) o = 0;
        int z, t;
        if (o < 2 * H * Tt) {
            t = o >> 1;
            z = (o & 1) ? Tz : -1;
        } else {
            t = Tt;
            z = o - 2 * H * Tt;
        }
        rpi[k] = pidx(z, t);
        ryi[k] = ok ? yidx(z, t) : sink;
        rzu[k] = zup(z);
        rzd[k] = zdn(z);
        ra[k] = *at(a.A, site(z, t));
    }
    // Halo of r: slices -1 and Tt over the z extent of y, and z = -2, -1, Tz,
    // Tz + 1 on the tile's slices.
    int hpi[KH], hgi[KH];
    double rh[KH], sh[KH];
    const int nhalo = 2 * ZY + 4 * H * Tt;
#pragma unroll
    for (int k = 0; k < KH; ++k) {
        int o = grp + a.G * k;
        const bool ok = on && o < nhalo;
        if (!ok) o = 0;
        int z, t;
        if (o < 2 * ZY) {
            const int up = o >= ZY;
            t = up ? Tt : -1;
            z = o - up * ZY - H;
        } else {
            const int e = o - 2 * ZY, j = e & 3;
            t = e >> 2;
            z = j < 2 ? j - 2 : Tz + j - 2;
        }
        hpi[k] = ok ? pidx(z, t) : sink;
        hgi[k] = site(z, t);
    }

    // Sum of v over the spatial neighbours of LDS index j.
    auto hop = [&](int j, int up, int dn) {
        if constexpr (!WHOLE) up = 8 * I, dn = -8 * I;
        double h = lds(j + up) + lds(j + dn);
        if constexpr (D >= 2) h += lds(j + in[0]) + lds(j + in[1]);
        if constexpr (D == 3) h += lds(j + in[2]) + lds(j + in[3]);
        return h;
    };
    // out = Q v on the own sites, for v there and vh on the halo.  Positions
    // are taken two at a time, so that a lane's loads in flight stay few.
    auto apply_q = [&](const double (&v)[KO], const double (&vh)[KH], double (&out)[KO]) {
#pragma unroll
        for (int k = 0; k < KO; ++k)
            if (ook[k]) lds(opi[k]) = v[k];
#pragma unroll
        for (int k = 0; k < KH; ++k) lds(hpi[k]) = vh[k];
        __syncthreads();
        double y[KO + (KO & 1)], yr[KY + (KY & 1)];
#pragma unroll
        for (int k = 0; k < KO; k += 2) {
            int j[2] = {};
#pragma unroll
            for (int e = 0; e < 2; ++e)
                if (k + e < KO) j[e] = fresh(opi[k + e]);
            y[k + 1] = 0.0;
#pragma unroll
            for (int e = 0; e < 2; ++e)
                if (k + e < KO)
                    y[k + e] = v[k + e] - g.kappa * hop(j[e], ozu[k + e], ozd[k + e]) +
                               oa[k + e] * lds(j[e] - 8 * ZP * I);
            settle(y[k], y[k + 1]);
        }
#pragma unroll
        for (int k = 0; k < KY; k += 2) {
            int j[2] = {};
#pragma unroll
            for (int e = 0; e < 2; ++e)
                if (k + e < KY) j[e] = fresh(rpi[k + e]);
            yr[k + 1] = 0.0;
#pragma unroll
            for (int e = 0; e < 2; ++e)
                if (k + e < KY)
                    yr[k + e] = lds(j[e]) - g.kappa * hop(j[e], rzu[k + e], rzd[k + e]) +
                                ra[k + e] * lds(j[e] - 8 * ZP * I);
            settle(yr[k], yr[k + 1]);
        }
#pragma unroll
        for (int k = 0; k < KO; ++k)
            if (ook[k]) lds(oyi[k]) = y[k];
#pragma unroll
        for (int k = 0; k < KY; ++k) lds(ryi[k]) = yr[k];
        __syncthreads();
#pragma unroll
        for (int k = 0; k < KO; k += 2) {
            int j[2] = {};
#pragma unroll
            for (int e = 0; e < 2; ++e)
                if (k + e < KO) j[e] = fresh(oyi[k + e]);
            double z[2] = {};
#pragma unroll
            for (int e = 0; e < 2; ++e)
                if (k + e < KO)
                    z[e] = y[k + e] - g.kappa * hop(j[e], ozu[k + e], ozd[k + e]) +
                           oap[k + e] * lds(j[e] + 8 * ZY * I);
            settle(z[0], z[1]);
#pragma unroll
            for (int e = 0; e < 2; ++e)
                if (k + e < KO) out[k + e] = ook[k + e] ? z[e] : 0.0;
        }
    };
    ResState c{};
    if (a.mode == kResFirst) {
#pragma unroll
        for (int k = 0; k < KO; ++k) {
            r[k] = ook[k] ? *at(a.phi, ogi[k]) : 0.0;
            x[k] = p[k] = s[k] = 0.0;
        }
#pragma unroll
        for (int k = 0; k < KH; ++k) {
            rh[k] = *at(a.phi, hgi[k]);
            sh[k] = 0.0;
        }
    } else {
        c = *a.st;
#pragma unroll
        for (int k = 0; k < KO; ++k) {
            r[k] = ook[k] ? *at(a.R, ogi[k]) : 0.0;
            p[k] = ook[k] ? *at(a.P, ogi[k]) : 0.0;
            s[k] = ook[k] ? *at(a.S, ogi[k]) : 0.0;
            x[k] = ook[k] ? *at(a.x, ogi[k]) : 0.0;
        }
#pragma unroll
        for (int k = 0; k < KH; ++k) {
            rh[k] = *at(a.R, hgi[k]);
            sh[k] = *at(a.S, hgi[k]);
        }
    }

    int mode = a.mode, n = 0;
    for (;;) {
        double w[KO];
        double* W = a.W + (size_t)(n & 1) * g.V;
        apply_q(r, rh, w);
        double part0 = 0.0, part1 = 0.0;
#pragma unroll
        for (int k = 0; k < KO; ++k) {
            if (orim[k]) agent_store(at_w(W, fresh(ogi[k])), w[k]);
            part0 += r[k] * r[k];
            part1 += r[k] * w[k];
        }
        gs.deposit(part0, part1);
        double rr, rw;
        if (!gs.wait(rr, rw)) {
            if (threadIdx.x == 0)
                __hip_atomic_store(&a.st->given_up, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            return;
        }
        double wh[KH];
#pragma unroll
        for (int k = 0; k < KH; ++k) wh[k] = agent_load(at(W, fresh(hgi[k])));
        if (mode == kResFirst) c.phi2 = rr;
        // (A residual just replaced has not met tol by the sum that decides.)
        if (!isfinite(rr)) c.done = kDoneBreakdown;
        else if (rr <= a.tol2 * c.phi2 && mode != kResReplaced) c.done = kDoneIterConverged;
        else if (c.iter >= a.max_iter) c.done = kDoneMaxIter;
        if (c.done != kRunning || n == a.iters) break;
        const double beta = mode == kResFirst ? 0.0 : rr / c.rho;
        double pq = rw;
        if (mode == kResOn) pq = rw - beta * rr / c.alpha;
        else if (mode == kResReplaced) pq = rw + 2.0 * beta * c.rs + beta * beta * c.pq;
        if (!(pq > 0.0) || !isfinite(pq)) {
            c.done = kDoneBreakdown;
            break;
        }
        const double alpha = rr / pq;
        c.pq = pq;
        c.alpha = alpha;
        c.rho = rr;
        mode = kResOn;
#pragma unroll
        for (int k = 0; k < KO; ++k) {
            p[k] = r[k] + beta * p[k];
            s[k] = w[k] + beta * s[k];
            x[k] = x[k] + alpha * p[k];
            r[k] = r[k] - alpha * s[k];
        }
#pragma unroll
        for (int k = 0; k < KH; ++k) {
            sh[k] = wh[k] + beta * sh[k];
            rh[k] = rh[k] - alpha * sh[k];
        }
        ++c.iter;
        ++n;
    }
#pragma unroll
    for (int k = 0; k < KO; ++k)
        if (ook[k]) {
            const int i = fresh(ogi[k]);
            *at_w(a.x, i) = x[k];
            *at_w(a.R, i) = r[k];
            *at_w(a.P, i) = p[k];
            *at_w(a.S, i) = s[k];
        }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        // Not given_up, which another block may write.
        a.st->rho = c.rho;
        a.st->alpha = c.alpha;
        a.st->pq = c.pq;
        a.st->phi2 = c.phi2;
        a.st->iter = c.iter;
        a.st->done = c.done;
    }
}

// The kernel of a dimension, level and cut (cgres_d1.hip, _d2, _d3).
using ResKernel = void (*)(ResArgs);
template <int D, int L>
ResKernel res_kernel_l(bool whole) {
    constexpr ResLevel K = kResLevels[L];
    if constexpr (K.whole)
        if (whole) return &k_cg_resident<D, true, K.own, K.rim, K.halo>;
    return &k_cg_resident<D, false, K.own, K.rim, K.halo>;
}
template <int D, int... L>
ResKernel res_kernel_of(int level, bool whole, std::integer_sequence<int, L...>) {
    ResKernel k = nullptr;
    (void)((level == L ? (k = res_kernel_l<D, L>(whole), true) : false) || ...);
    return k;
}
template <int D>
ResKernel res_kernel_d(int level, bool whole) {
    return res_kernel_of<D>(level, whole, std::make_integer_sequence<int, kResLevelCount>());
}
ResKernel res_kernel_d1(int level, bool whole);
ResKernel res_kernel_d2(int level, bool whole);
ResKernel res_kernel_d3(int level, bool whole);

}  // namespace hub
