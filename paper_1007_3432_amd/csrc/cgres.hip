// Host side of the resident CG solve (cgres.h): how a lattice is cut into
// blocks, and the launches of a solve.
#include <algorithm>
#include <cmath>
#include <cstdlib>
#include <mutex>

#include "cgres.h"

namespace hub {

namespace {

struct ResPlan {
    int Nz = 0, Nt = 0, G = 0, inner = 0, level = -1;
    int threads = 0;
    size_t lds = 0;
    double us = 0;  // estimated time of an iteration
    bool whole() const { return Nz == 1; }
    int blocks() const { return Nz * Nt; }
};

constexpr size_t kResLdsMax = 160 * 1024;

// The cut with the smallest estimated iteration: the grid sum (1.75 us and 3
// ns a block), barriers, stores and the halo read (0.9 us), and the LDS
// accesses of the positions that a level's code goes through, 4 cycles each
// for a wavefront at 2.4 GHz; the levels that do not fit with z whole are at
// the register limit and measured 1 us slower than that.  Fitted over 70 cuts of
// ten lattices, to within 0.6 us, with one vector more in the lane's registers;
// as it is now, us an iteration, estimated and measured: d = 1 4096 x 128 4.0 and
// 4.2, 2048 x 512 4.4 and 4.8, d = 2 33 x 60 3.3 and 3.4, 128 x 60 6.2 and 6.6, d = 3
// 8^3 x 80 3.3 and 3.3, 16^3 x 128 4.9 and 5.8, x 160 6.3 and 6.4.  level < 0: the
// lattice does not fit.
ResPlan plan_resident(const Geom& g, int max_blocks) {
    ResPlan best;
    const int inner = g.vs / g.nx;
    if (inner > kResBlock || g.V > (1 << 21)) return best;
    const int G = kResBlock / inner;
    const int threads = (G * inner + 63) / 64 * 64;
    for (int Nz = 1; Nz <= std::min(g.nx, max_blocks); ++Nz) {
        const int H = Nz == 1 ? 0 : 1;
        const int Tz = ceil_div(g.nx, Nz);
        for (int Nt = 1; Nt <= std::min(g.nt, max_blocks / Nz); ++Nt) {
            const int Tt = ceil_div(g.nt, Nt);
            const int own = ceil_div(Tz * Tt, G), rim = ceil_div(2 * H * Tt + Tz, G),
                      halo = ceil_div(2 * (Tz + 2 * H) + 4 * H * Tt, G);
            const size_t lds =
                8 * (GridSum<kGridSumMax>::kLdsDoubles + 2 + (size_t)inner * ((size_t)(Tz + 4 * H) * (Tt + 2) +
                                           (size_t)(Tz + 2 * H) * (Tt + 1)));
            if (lds > kResLdsMax) continue;
            for (int l = 0; l < kResLevelCount; ++l) {
                const ResLevel& K = kResLevels[l];
                if (own > K.own || rim > K.rim || halo > K.halo || (Nz == 1 && !K.whole)) continue;
                const double acc = K.own * (4.0 * g.d + 4) + K.rim * (2.0 * g.d + 3) + K.halo;
                const double us = 2.65 + 0.003 * Nz * Nt + acc * (threads / 64) * 4 / 2400.0 +
                                  (K.whole ? 0.0 : 1.0);
                if (best.level >= 0 && us >= best.us) continue;
                best.Nz = Nz;
                best.Nt = Nt;
                best.G = G;
                best.inner = inner;
                best.level = l;
                best.threads = threads;
                best.lds = lds;
                best.us = us;
            }
        }
    }
    return best;
}

ResKernel res_kernel(const Geom& g, const ResPlan& p, bool pcg) {
    switch (g.d) {
        case 1: return res_kernel_d1(p.level, p.whole(), pcg);
        case 2: return res_kernel_d2(p.level, p.whole(), pcg);
        default: return res_kernel_d3(p.level, p.whole(), pcg);
    }
}

constexpr int kFlagWords = kMaxResidentBlocks * kSlotStride;

// Empty slots, flags down, nothing given up, still running.
__global__ __launch_bounds__(256) void k_res_reset(uint64_t* slots, uint64_t* flags, ResState* st) {
    for (int k = blockIdx.x * 256 + threadIdx.x; k < (int)kSlotWords; k += gridDim.x * 256)
        slots[k] = kSlotEmpty;
    for (int k = blockIdx.x * 256 + threadIdx.x; k < kFlagWords; k += gridDim.x * 256) flags[k] = 0;
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        st->given_up = 0;
        st->done = kRunning;
    }
}

// r = phi - z, and the deposits of |r|^2.
__global__ __launch_bounds__(256) void k_res_recompute(const double* __restrict__ phi,
                                                       const double* __restrict__ z,
                                                       double* __restrict__ r, int V,
                                                       double* partials) {
    double part[1] = {0.0};
    for (int i = blockIdx.x * 256 + threadIdx.x; i < V; i += gridDim.x * 256) {
        const double d = phi[i] - z[i];
        r[i] = d;
        part[0] += d * d;
    }
    deposit<256, 1>(part, partials, blockIdx.x);
}

__global__ __launch_bounds__(256) void k_res_recompute_finish(const double* partials, int n,
                                                              ResState* st) {
    double tot[1];
    reduce_deposits<256, 1>(partials, n, tot);
    if (threadIdx.x == 0) st->rho_true = tot[0];
}

// Products with Q of one launch: 1 to 2 ms.  The blocks fill the registers or the
// LDS of their CUs, so that a kernel of another stream which does not fit beside
// them, or whose stream shares a hardware queue with this one, starts only
// between launches.  A product on 16^3 x 32 beside a solve on 16^3 x 128 waited
// for 5.9 ms at most with 1000 products a launch and for 1.8 with 300 (with the
// multi-kernel solver for 0.9 to 1.9 where the queue was shared, else for 0.1).
// A launch costs some 50 us: solves alone take 2 to 3% more than with 1000.
constexpr int kResChunk = 300;

// Reads of a grid sum's slots before a wait is given up (about half a second).
int res_read_limit() {
    const char* e = std::getenv("HUB_CG_RESIDENT_READS");
    return e ? std::max(1, std::atoi(e)) : 1 << 19;
}

bool res_enabled() {
    const char* e = std::getenv("HUB_CG_RESIDENT");
    return !(e && e[0] == '0');
}

}  // namespace

// One launch at a time on a device: its blocks wait for each other, so all
// must find a place.
FairLock& resident_lock(int device) {
    static FairLock lock[64];
    return lock[device & 63];
}

hub_status cg_solve_resident(const Geom& g, const double* sigma, const double* phi, double* x,
                             const hub_cg_opts& o, const double* factors, int nf,
                             hub_cg_stats* out, hipStream_t st, bool* ran) {
    *ran = false;
    const bool pcg = nf > 0;
    if (!res_enabled()) return HUB_OK;
    int dev = 0, cus = 0, coop = 0;
    HUB_HIP(hipGetDevice(&dev));
    HUB_HIP(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
    HUB_HIP(hipDeviceGetAttribute(&coop, hipDeviceAttributeCooperativeLaunch, dev));
    if (!coop) return HUB_OK;
    const ResPlan p = plan_resident(g, std::min(cus, kMaxResidentBlocks));
    if (p.level < 0) return HUB_OK;
    const ResKernel kern = res_kernel(g, p, pcg);
    HUB_HIP(hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                                (int)kResLdsMax));

    auto al = [](size_t b) { return (b + 255) & ~size_t(255); };
    const size_t vb = al(8 * (size_t)g.V);
    const size_t sb = al(8 * (kSlotWords + kFlagWords)), fb = al(24 * (size_t)nf);
    char* ws = nullptr;
    hub_status r = solver_workspace(5 * vb + sb + 256 + fb, &ws);
    if (r != HUB_OK) return r;
    SolverHost host;
    r = solver_host(&host);
    if (r != HUB_OK) return r;
    ResArgs a{};
    a.g = g;
    a.inner = p.inner;
    a.Nz = p.Nz;
    a.Nt = p.Nt;
    a.G = p.G;
    a.A = (const double*)ws;
    a.R = (double*)(ws + vb);
    a.P = (double*)(ws + 2 * vb);
    a.W = (double*)(ws + 3 * vb);  // two vectors
    a.slots = (uint64_t*)(ws + 5 * vb);
    a.flags = a.slots + kSlotWords;
    a.st = (ResState*)(ws + 5 * vb + sb);
    a.f = (double*)(ws + 5 * vb + sb + 256);
    a.nf = nf;
    if (pcg)
        HUB_HIP(hipMemcpyAsync((void*)a.f, factors, 24 * (size_t)nf, hipMemcpyHostToDevice, st));
    a.phi = phi;
    a.x = x;
    a.tol2 = o.tol * o.tol;
    a.max_iter = o.max_iter;
    a.iters = std::max(1, kResChunk / (2 * nf + 1));
    a.mode = kResFirst;
    a.limit = res_read_limit();
    static_assert(sizeof(ResState) <= sizeof(CGScalars), "snapshot buffer");
    ResState* s = (ResState*)host.snap;

    auto fetch = [&]() -> hub_status {
        HUB_HIP(hipMemcpyAsync(s, a.st, sizeof(ResState), hipMemcpyDeviceToHost, st));
        HUB_HIP(hipStreamSynchronize(st));
        return HUB_OK;
    };
    // r = phi - Q x with the operator's own kernels; once or twice a solve.
    auto recompute = [&]() -> hub_status {
        double *y = a.W, *z = a.W + g.V;
        hub_status q = launch_apply_M(g, a.A, HUB_F64, HUB_F64, x, y, 0, st);
        if (q == HUB_OK) q = launch_apply_M(g, a.A, HUB_F64, HUB_F64, y, z, 1, st);
        if (q != HUB_OK) return q;
        const int blocks = std::min(256, ceil_div(g.V, 256));
        double* part = (double*)a.slots;  // refilled before the next launch
        static_assert(256 <= kSlotWords, "deposits fit the slots");
        k_res_recompute<<<blocks, 256, 0, st>>>(phi, z, a.R, g.V, part);
        k_res_recompute_finish<<<1, 256, 0, st>>>(part, blocks, a.st);
        HUB_HIP(hipGetLastError());
        return fetch();
    };
    r = launch_links(g, sigma, ws, HUB_F64, st);
    if (r != HUB_OK) return r;
    // What the caller has queued on its stream ends before the lock is taken:
    // other threads' solves do not wait for it (a solve of 2 ms beside a thread
    // with 260 ms queued: 241 ms, and 4 with the wait here), nor for what it may
    // wait for itself.
    HUB_HIP(hipStreamSynchronize(st));
    HUB_HIP(hipEventRecord(host.t0, st));
    int done = kRunning, recomputes = 0;
    while (done == kRunning) {
        {
            std::lock_guard<FairLock> lk(resident_lock(dev));
            k_res_reset<<<8, 256, 0, st>>>(a.slots, a.flags, a.st);
            void* args[] = {&a};
            const hipError_t e = hipLaunchCooperativeKernel(
                (const void*)kern, dim3(p.blocks()), dim3(p.threads), args, (unsigned)p.lds, st);
            if (e != hipSuccess) {
                // Refused, as where another process of this GPU holds the
                // right to such launches.  An error of earlier work is
                // reported here instead.
                (void)hipGetLastError();
                HUB_HIP(hipStreamSynchronize(st));
                return HUB_OK;
            }
            r = fetch();
            if (r != HUB_OK) return r;
        }
        // A breakdown is left to the multi-kernel solver as well: it decides, and
        // counts its steps, as it does for the lattices that come to it first.
        if (s->given_up || s->done == kDoneBreakdown) return HUB_OK;
        done = s->done;
        a.mode = kResOn;
        if (done != kDoneIterConverged) continue;
        if (s->phi2 == 0.0) {
            s->rho_true = 0.0;
            done = kDoneConverged;
            break;
        }
        r = recompute();
        if (r != HUB_OK) return r;
        ++recomputes;
        if (s->rho_true <= a.tol2 * s->phi2) done = kDoneConverged;
        else if (!std::isfinite(s->rho_true)) return HUB_OK;
        else if (s->iter >= o.max_iter) done = kDoneMaxIter;
        else done = kRunning;
        a.mode = kResReplaced;
    }
    if (s->done > kDoneConverged) {
        r = recompute();
        if (r != HUB_OK) return r;
    }
    HUB_HIP(hipEventRecord(host.t1, st));
    HUB_HIP(hipStreamSynchronize(st));
    float ms = 0.0f;
    HUB_HIP(hipEventElapsedTime(&ms, host.t0, host.t1));
    *ran = true;
    hub_cg_stats stats{};
    stats.iters = s->iter;
    stats.reliable_updates = recomputes;
    stats.true_rel_resid = s->phi2 > 0 ? std::sqrt(s->rho_true / s->phi2) : 0.0;
    stats.ms = ms;
    stats.status = done == kDoneConverged ? HUB_OK : HUB_E_NOCONV;
    if (out) *out = stats;
    if (stats.status != HUB_OK)
        return set_error(HUB_E_NOCONV,
                         "CG did not converge: %d iterations, true relative residual %.3e",
                         s->iter, stats.true_rel_resid);
    return HUB_OK;
}

}  // namespace hub
