// One block's tile of a lattice that stays resident on the chip, for the
// solvers that keep their vectors in registers (cgres.h): where its sites and
// halo lie, Q = M^T M on it through LDS, and the exchange of halos between the
// blocks of the grid.
//
// The last spatial dimension (z below; x itself for d = 1) and time are cut
// into Nz x Nt tiles, one block each; the other dimensions, `inner`, stay
// whole.  A lane keeps one inner index and every G-th (z, t) position of its
// block's tile.  Q v: v of tile and halo go into LDS (P), y = M v on the tile
// and on the sites around it that M^T reads into LDS (Y), and the lane has
// (M^T y) at its own sites.
//
// Exchange.  A block stores the rim of a vector for its neighbours in one of
// two buffers, taken in turns.  Where a grid sum follows (CG), that is the
// synchronisation; elsewhere the block raises a flag when its stores have
// arrived, and a neighbour waits for the flags of the tiles around it.  A
// buffer is free again by then: whoever has raised its next flag, or gone into
// the next sum, has read it.  Stores and loads are agent-scope relaxed atomics
// (gridsum.h), every wait is bounded.  (Values that carry the synchronisation
// themselves, as the slots of the grid sum do, need a mark stored over each
// after it has been read.  A product of the preconditioned solver took, with
// them and with flags: 16^3 x 128 4.9 and 4.7 us, 2048 x 512 4.1 and 3.3, 8^3 x
// 80 2.2 and 2.7; an iteration of CG 0.3 us more with them.)
#pragma once

#include "gridsum.h"
#include "internal.h"

namespace hub {

// Positions a lane handles at most: its own sites, the sites around the tile
// where y is formed, and the halo.  Each level is a kernel; in CG a lane
// holds 13 words for each of the first, 4 and 6 for each of the others, and
// two more for each of the first two where z is whole.  `whole`: that fits too.
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
    double rho;       // preconditioned: r.z of the last step
    double phi2;
    double rho_true;  // |phi - Q x|^2 of the last recompute
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
    double *R, *P;  // r and p between launches
    double* W;   // 2 V: rims between blocks
    uint64_t* flags;  // kMaxResidentBlocks, 64 bytes apart, 0 when a launch starts
    uint64_t* slots;
    ResState* st;
    double tol2;
    int max_iter;
    int iters;   // iterations of this launch at most
    int mode;    // kResFirst: starts the solve; kResReplaced: r was replaced
    int limit;   // reads before a wait is given up
    const double* f;  // preconditioned: c2, c1, c0 of each factor
    int nf;           // and their number
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

__device__ __forceinline__ lds_double& lds_at(int byte) {
    return *(lds_double*)(uintptr_t)(uint32_t)byte;
}
__device__ __forceinline__ const double* at(const double* v, int byte) {
    return reinterpret_cast<const double*>(reinterpret_cast<const char*>(v) + (uint32_t)byte);
}
__device__ __forceinline__ double* at_w(double* v, int byte) {
    return reinterpret_cast<double*>(reinterpret_cast<char*>(v) + (uint32_t)byte);
}

template <int D, bool WHOLE, int KO, int KY, int KH>
struct ResTile {
    static constexpr int H = WHOLE ? 0 : 1;  // z halo of y; v has twice that
    // LDS, in doubles: the sums, the give-up mark, P, Y, and one spare element
    // that positions past the end write.  Indices are LDS byte addresses.
    static constexpr int kMark = GridSum<kGridSumMax>::kLdsDoubles, kP = kMark + 1;

    double kappa;
    int I, ZP, ZY;  // inner sites; z extents of P and Y
    int base;
    double* W;
    size_t V;
    int turn;        // rims handed over in this launch
    uint64_t* flag;  // this block's
    const uint64_t* near_flag;  // of a tile around this one, a lane each
    int limit;
    // Own sites.  Positions past the end repeat the first one and are masked.
    int opi[KO], oyi[KO], ogi[KO];
    bool ook[KO], orim[KO];
    int ozu[KO], ozd[KO];  // used where z is whole
    double oa[KO], oap[KO];
    // Sites around the tile where y is formed.
    int rpi[KY], ryi[KY], rzu[KY], rzd[KY];
    double ra[KY];
    // Halo of v.
    int hpi[KH], hgi[KH];
    int in[4];  // inner neighbours

    __device__ __forceinline__ void init(const ResArgs& a, double* lds) {
        const Geom& g = a.g;
        const int nz = g.nx, nt = g.nt;
        kappa = g.kappa;
        I = D == 1 ? 1 : a.inner;
        W = a.W;
        V = (size_t)g.V;
        turn = 0;
        limit = a.limit;
        // Tiles next to each other in z, and then in time, are on the same XCD,
        // whose L2 then has most of what a block hands to its neighbours (CG on
        // 16^3 x 128 9.1 -> 5.9 us an iteration).
        const int tile = xcd_remap(blockIdx.x, gridDim.x);
        const int bz = tile % a.Nz, bt = tile / a.Nz;
        const int z0 = (int)((long long)bz * nz / a.Nz),
                  Tz = (int)((long long)(bz + 1) * nz / a.Nz) - z0;
        const int t0 = (int)((long long)bt * nt / a.Nt),
                  Tt = (int)((long long)(bt + 1) * nt / a.Nt) - t0;
        ZP = Tz + 4 * H;
        ZY = Tz + 2 * H;
        base = (int)(uint32_t)(uintptr_t)(lds_double*)lds;
        const int kY = kP + ZP * (Tt + 2) * I, sink = base + 8 * (kY + ZY * (Tt + 1) * I);
        const int grp = (int)threadIdx.x / I, m = (int)threadIdx.x - grp * I;
        const bool on = grp < a.G;
        // The tiles that hold z0 - 2, z0 - 1, z0, z0 + Tz, z0 + Tz + 1 on t0 - 1,
        // t0, t0 + Tt (images wrap): a lane each.
        {
            const int c = (int)threadIdx.x % 15, j = c % 5, i = c / 5;
            const int zc = ((z0 + (j < 3 ? j - 2 : Tz + j - 3)) % nz + nz) % nz;
            const int tc = ((t0 + (i < 2 ? i - 1 : Tt)) % nt + nt) % nt;
            const int near = ((zc + 1) * a.Nz - 1) / nz + a.Nz * (((tc + 1) * a.Nt - 1) / nt);
            near_flag = a.flags + near * kSlotStride;
            flag = a.flags + tile * kSlotStride;
        }
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
        // y around the tile: z = -1, Tz on the tile's
        // slices, and the tile's z on the slice after it.
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
        // Halo: slices -1 and Tt over the z extent of y, and z = -2, -1, Tz,
        // Tz + 1 on the tile's slices.
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
        if (threadIdx.x == 0) lds_at(base + 8 * kMark) = 0.0;
        __syncthreads();
    }

    // Sum of v over the spatial neighbours of LDS index j.
    __device__ __forceinline__ double hop(int j, int up, int dn) const {
        if constexpr (!WHOLE) up = 8 * I, dn = -8 * I;
        double h = lds_at(j + up) + lds_at(j + dn);
        if constexpr (D >= 2) h += lds_at(j + in[0]) + lds_at(j + in[1]);
        if constexpr (D == 3) h += lds_at(j + in[2]) + lds_at(j + in[3]);
        return h;
    }

    // out = Q v on the own sites, for v there and vh on the halo.  Positions
    // are taken two at a time, so that a lane's loads in flight stay few.
    __device__ __forceinline__ void apply_q(const double (&v)[KO], const double (&vh)[KH],
                                            double (&out)[KO]) {
#pragma unroll
        for (int k = 0; k < KO; ++k)
            if (ook[k]) lds_at(opi[k]) = v[k];
#pragma unroll
        for (int k = 0; k < KH; ++k) lds_at(hpi[k]) = vh[k];
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
                    y[k + e] = v[k + e] - kappa * hop(j[e], ozu[k + e], ozd[k + e]) +
                               oa[k + e] * lds_at(j[e] - 8 * ZP * I);
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
                    yr[k + e] = lds_at(j[e]) - kappa * hop(j[e], rzu[k + e], rzd[k + e]) +
                                ra[k + e] * lds_at(j[e] - 8 * ZP * I);
            settle(yr[k], yr[k + 1]);
        }
#pragma unroll
        for (int k = 0; k < KO; ++k)
            if (ook[k]) lds_at(oyi[k]) = y[k];
#pragma unroll
        for (int k = 0; k < KY; ++k) lds_at(ryi[k]) = yr[k];
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
                    z[e] = y[k + e] - kappa * hop(j[e], ozu[k + e], ozd[k + e]) +
                           oap[k + e] * lds_at(j[e] + 8 * ZY * I);
            settle(z[0], z[1]);
#pragma unroll
            for (int e = 0; e < 2; ++e)
                if (k + e < KO) out[k + e] = ook[k + e] ? z[e] : 0.0;
        }
    }

    // The rim of v for the neighbours.
    __device__ __forceinline__ void publish(const double (&v)[KO]) {
        double* to = W + (size_t)(turn & 1) * V;
#pragma unroll
        for (int k = 0; k < KO; ++k)
            if (orim[k]) agent_store(at_w(to, fresh(ogi[k])), v[k]);
        ++turn;
    }

    // Waits until the neighbours have published as often as this block.  False
    // when the wait was given up: the block must end then.  All lanes.
    __device__ __forceinline__ bool exchange() {
        wait_stores();
        __syncthreads();
        if (threadIdx.x < 64) {
            if (threadIdx.x == 0)
                __hip_atomic_store(flag, (uint64_t)turn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            bool here = false;
            for (int n = 0; n < limit && !here; ++n)
                here = __all(__hip_atomic_load(near_flag, __ATOMIC_RELAXED,
                                               __HIP_MEMORY_SCOPE_AGENT) >= (uint64_t)turn);
            if (!here && threadIdx.x == 0) lds_at(base + 8 * kMark) = 1.0;
        }
        __syncthreads();
        return lds_at(base + 8 * kMark) == 0.0;
    }

    // The halo of what was published last, after exchange() or a grid sum.
    __device__ __forceinline__ void fetch(double (&vh)[KH]) const {
        const double* from = W + (size_t)((turn - 1) & 1) * V;
#pragma unroll
        for (int k = 0; k < KH; ++k) vh[k] = agent_load(at(from, fresh(hgi[k])));
    }
};

}  // namespace hub
