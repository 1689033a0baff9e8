// Shared device/host definitions of libhub (gfx950).
#pragma once

#include <hip/hip_runtime.h>
#include <hip/hip_fp16.h>
#include <stdint.h>

#include "hub.h"

namespace hub {

// n / d for 0 <= n < 2^31 and 1 <= d < 2^31 by one multiply and a shift
// (rounded-up multiplier, after Granlund and Montgomery 1994): with
// s = ceil(log2 d) and m = ceil(2^(32+s) / d), m d = 2^(32+s) + e with
// 0 <= e < d, so n m / 2^(32+s) exceeds n / d by less than n / 2^(32+s) <
// 1 / (2d), which never reaches the next integer.  The one-lane-per-site
// kernels need two to four divisions per site for its coordinates; as
// integer divisions those cost more than the kernels' memory traffic.
struct FastDiv {
    uint64_t m;  // <= 2^33
    int sh;      // 32 + s
};

inline FastDiv make_fastdiv(uint32_t d) {
    int s = 0;
    while ((1ull << s) < d) ++s;
    return {((1ull << (32 + s)) + d - 1) / d, 32 + s};
}

__host__ __device__ __forceinline__ int fdiv(int n, const FastDiv& f) {
    return (int)(((uint64_t)(uint32_t)n * f.m) >> f.sh);
}

// Lattice geometry and operator constants, passed to kernels by value.
struct Geom {
    int d;          // spatial dimensions
    int nx;         // spatial extent
    int nt;         // time slices
    int vs;         // nx^d
    int V;          // vs * nt
    double kappa;   // dtau * t_hop
    double lscale;  // exp(dtau * mu)
    double b;       // Hubbard-Stratonovich coupling sqrt(2 (exp(-dtau U) - 1))
    FastDiv fnx;    // division by nx
    FastDiv fvs;    // division by vs
};

// Device-resident solver state of one CG solve.  Every field is written by
// exactly one thread: thread 0 of a one-block finalize kernel, or an
// initialisation kernel.
struct CGScalars {
    double rho;        // current iterated r.r (FP64 accumulation)
    double rho_prev;   // r.r of the previous iteration
    double alpha;      // step length still to be added to x (0 once folded)
    double beta;       // p_new = gamma r + beta p_old
    double gamma;      // 1 except right after a reliable update
    double phi2;       // |phi|^2
    double tol2phi2;   // tol^2 |phi|^2
    double rho_true;   // |phi - Q x|^2 of the last true-residual recompute
    double rho_ru;     // r.r right after the last reliable update
    double delta2;     // reliable update once rho < delta2 * rho_ru (0: never)
    double pq;         // last p.Qp
    double rr;         // preconditioned CG: iterated r.r (rho holds r.z)
    int32_t iter;      // iterations completed
    int32_t max_iter;
    int32_t done;      // see kDone* below
    int32_t reliable_updates;
    int32_t restart;   // preconditioned CG: next beta is 0 (fresh residual)
    int32_t pad[3];
};

enum : int32_t {
    kRunning = 0,
    kDoneIterConverged = 1,  // iterated residual met tol, or dropped by
                             // delta since the last reliable update: recompute
    kDoneConverged = 2,      // true residual met tol
    kDoneBreakdown = 3,      // p.Qp <= 0 or a non-finite scalar
    kDoneMaxIter = 4,
};

// When the fold / true-residual kernels run.
enum : int32_t {
    kModeReliable = 0,  // periodic reliable update: run while done <= 1
    kModeCheck = 1,     // verify an iterated convergence: run iff done == 1
    kModeFinal = 2,     // end of solve: always run
};

__host__ __device__ inline int ceil_div(int a, int b) { return (a + b - 1) / b; }

#if defined(__HIP_DEVICE_COMPILE__) || defined(__HIPCC__)
// Workgroups are dispatched round-robin over the 8 XCDs of an MI355X, each
// with its own L2.  Map hardware block ids so that every XCD receives a
// contiguous range of logical tiles: neighbouring tiles (which share halo
// sites) then hit in the same L2.
__device__ inline int xcd_remap(int bid, int nblocks) {
    constexpr int kXcd = 8;
    const int q = nblocks / kXcd, r = nblocks % kXcd;
    const int x = bid % kXcd, k = bid / kXcd;
    return x * q + (x < r ? x : r) + k;
}

// Wrap an index that is at most one period out of [0, n).
__device__ inline int wrap1(int v, int n) {
    return v < 0 ? v + n : (v >= n ? v - n : v);
}

// v of the lane that a DPP control names (all lanes have a source there).
template <int CTRL>
__device__ __forceinline__ double dpp_move(double v) {
    const long long w = __builtin_bit_cast(long long, v);
    const int lo = (int)w, hi = (int)(w >> 32);
    const int rlo = __builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xf, 0xf, false);
    const int rhi = __builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xf, 0xf, false);
    return __builtin_bit_cast(double, (long long)(((unsigned long long)(unsigned)rhi << 32) |
                                                  (unsigned)rlo));
}

// v_i + v_{i xor 32} (HALF = 32) or v_i + v_{i xor 16} (HALF = 16): the swap
// of two copies of v leaves one addend of every lane in each copy.
template <int HALF>
__device__ __forceinline__ double swap_add(double v) {
    const long long w = __builtin_bit_cast(long long, v);
    const unsigned lo = (unsigned)w, hi = (unsigned)(w >> 32);
    auto sw = [](unsigned x) {
        if constexpr (HALF == 32) return __builtin_amdgcn_permlane32_swap(x, x, false, false);
        else return __builtin_amdgcn_permlane16_swap(x, x, false, false);
    };
    const auto l = sw(lo), h = sw(hi);
    const double a = __builtin_bit_cast(
        double, (long long)(((unsigned long long)h[0] << 32) | l[0]));
    const double b = __builtin_bit_cast(
        double, (long long)(((unsigned long long)h[1] << 32) | l[1]));
    return a + b;
}

// Sum over a 64-wide wavefront, result valid in every lane.  The tree of the
// xor butterfly (32, 16, 8, 4, 2, 1), whose every step adds the same two
// numbers in all lanes that share them, so that its bits do not depend on how
// the numbers travel: as register moves (lane swaps, DPP rotations and quad
// permutations) a step costs a few cycles, as an LDS permute a round trip of
// over a hundred.  After the step of 8 the values repeat every 8 lanes of a
// row, so a rotation by 4 brings the lane of i xor 4.
__device__ inline double wave_sum(double v) {
    v = swap_add<32>(v);
    v = swap_add<16>(v);
    v += dpp_move<0x128>(v);  // row_ror:8
    v += dpp_move<0x124>(v);  // row_ror:4
    v += dpp_move<0x4e>(v);   // quad_perm 2,3,0,1
    v += dpp_move<0xb1>(v);   // quad_perm 1,0,3,2
    return v;
}

// Deterministic block sum (fixed tree); result valid in thread 0.
template <int BLOCK>
__device__ inline double block_sum(double v) {
    static_assert(BLOCK % 64 == 0 && BLOCK <= 1024, "block must be whole waves");
    __shared__ double red[BLOCK / 64];
    v = wave_sum(v);
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    __syncthreads();  // red[] may still be read by a previous call
    if (lane == 0) red[wid] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 0; w < BLOCK / 64; ++w) s += red[w];
    }
    return s;
}

// Sum of n deposits of NP values (deposit b at partials[NP*b + k]) in a
// fixed order: thread t adds deposits t, t+BLOCK, ... (four at a time, the
// loads issued together), then the block tree.  Every caller that sums the
// same deposits gets the same bits.  Result in thread 0.  Callers read the
// deposits after a kernel boundary or a grid barrier, so plain loads see
// them.
template <int BLOCK, int NP>
__device__ inline void reduce_deposits(const double* partials, int n, double (&total)[NP]) {
#pragma unroll
    for (int k = 0; k < NP; ++k) {
        double s = 0.0;
        int b = threadIdx.x;
        for (; b + 3 * BLOCK < n; b += 4 * BLOCK) {
            const double v0 = partials[NP * b + k];
            const double v1 = partials[NP * (b + BLOCK) + k];
            const double v2 = partials[NP * (b + 2 * BLOCK) + k];
            const double v3 = partials[NP * (b + 3 * BLOCK) + k];
            s += v0;
            s += v1;
            s += v2;
            s += v3;
        }
        for (; b < n; b += BLOCK) s += partials[NP * b + k];
        total[k] = block_sum<BLOCK>(s);
    }
}

// The sum of n single-value deposits in exactly the order of
// reduce_deposits<256, 1> (so with the same bits), computed by a block of
// any multiple of 64 lanes: its waves take the four 64-lane groups of a
// 256-lane block in turn.  Result in every thread.  Lets a kernel of any
// block size reduce the previous kernel's deposits itself and get what a
// one-block finalize would.
__device__ inline double reduce_deposits_canon(const double* partials, int n) {
    constexpr int B = 256;
    __shared__ double red[4];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
    const int nw = (int)(blockDim.x >> 6);
    __syncthreads();  // red[] may still be read by a previous call
    for (int vw = wid; vw < 4; vw += nw) {
        double s = 0.0;
        int b = vw * 64 + lane;
        for (; b + 3 * B < n; b += 4 * B) {
            const double v0 = partials[b];
            const double v1 = partials[b + B];
            const double v2 = partials[b + 2 * B];
            const double v3 = partials[b + 3 * B];
            s += v0;
            s += v1;
            s += v2;
            s += v3;
        }
        for (; b < n; b += B) s += partials[b];
        s = wave_sum(s);
        if (lane == 0) red[vw] = s;
    }
    __syncthreads();
    double tot = 0.0;
#pragma unroll
    for (int w = 0; w < 4; ++w) tot += red[w];
    return tot;
}

// After r.r: rho, beta, iteration count; ask for a true-residual recompute
// when rho meets tol or has dropped by delta^2 since the last one.
__device__ __forceinline__ void finish_phaseB(CGScalars* sc, double total) {
    if (!isfinite(total)) {
        sc->done = kDoneBreakdown;
        return;
    }
    sc->rho_prev = sc->rho;
    sc->rho = total;
    sc->beta = total / sc->rho_prev;
    sc->iter += 1;
    if (total <= sc->tol2phi2 || total < sc->delta2 * sc->rho_ru)
        sc->done = kDoneIterConverged;
    else if (sc->iter >= sc->max_iter)
        sc->done = kDoneMaxIter;
}

// The sum of n <= 256 single-value deposits in the order of
// reduce_deposits<256, 1>, so with its bits, by every wavefront for itself:
// all loads at once and no barrier, so that nothing else the kernel has to
// load waits for it.
__device__ __forceinline__ double reduce_deposits_wave(const double* __restrict__ partials,
                                                       int n) {
    constexpr int kG = 4;  // wavefronts of the 256-lane block whose order this is
    const int lane = threadIdx.x & 63;
    double v[kG];
#pragma unroll
    for (int k = 0; k < kG; ++k) v[k] = partials[min(64 * k + lane, n - 1)];
    double tot = 0.0;
#pragma unroll
    for (int k = 0; k < kG; ++k) tot += wave_sum(64 * k + lane < n ? v[k] : 0.0);
    return tot;
}

// The same for n <= 512, shared among the wavefronts of the block: a quarter
// of the sums each in 256 lanes, for one barrier.  Once in a kernel.
__device__ __forceinline__ double reduce_deposits_block(const double* __restrict__ partials,
                                                        int n) {
    constexpr int kG = 4;
    __shared__ double red[kG];
    const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = (int)(blockDim.x >> 6);
    for (int k = wid; k < kG; k += nw) {
        const int b = 64 * k + lane;
        const double v0 = partials[min(b, n - 1)], v1 = partials[min(b + 64 * kG, n - 1)];
        double s = b < n ? v0 : 0.0;
        s += b + 64 * kG < n ? v1 : 0.0;
        s = wave_sum(s);
        if (lane == 0) red[k] = s;
    }
    __syncthreads();
    double tot = 0.0;
#pragma unroll
    for (int k = 0; k < kG; ++k) tot += red[k];
    return tot;
}

// Who adds the deposits that a sweep takes over from the kernel before it:
// each wavefront (kByWave, at most 256), the block (kByBlock, at most 512), or
// a launch of its own before it (kByNone).  The wavefronts where one solve has
// the chip to itself, us an iteration by wave and by block: d = 1 32 x 64 7.8
// and 8.4, 256 x 128 8.3 and 8.4.  The block with more deposits (20^3 x 96, 375
// of them: 16.4 and 16.1) and where blocks of many solves share the CUs, whose
// wavefronts would issue four times the sums (eight served solves 258 and 246
// ms).
enum SumsBy { kByNone = 0, kByWave, kByBlock };
inline int sums_by(int n, bool shared) {
    return n > 512 ? kByNone : n > 256 || shared ? kByBlock : kByWave;
}

// The solver state as words, one a lane: a block that hands the state on loads
// its lane's word beside its other loads, puts the new values in and stores it,
// where a copy by one lane would add a load's latency to the kernel.
constexpr int kStateWords = sizeof(CGScalars) / 8;
static_assert(kStateWords <= 64 && offsetof(CGScalars, iter) % 8 == 0 &&
                  offsetof(CGScalars, max_iter) == offsetof(CGScalars, iter) + 4 &&
                  offsetof(CGScalars, done) % 8 == 0 &&
                  offsetof(CGScalars, reliable_updates) == offsetof(CGScalars, done) + 4,
              "pairs of 32-bit fields that share a word");
__device__ __forceinline__ void put_word(uint64_t& w, size_t offset, double v) {
    if (threadIdx.x == offset / 8) w = (uint64_t)__double_as_longlong(v);
}
__device__ __forceinline__ void put_word(uint64_t& w, size_t offset, int lo, int hi) {
    if (threadIdx.x == offset / 8) w = (uint64_t)(uint32_t)hi << 32 | (uint32_t)lo;
}

// finish_phaseB by every block for itself: the state left in *from and its
// n r.r deposits give what a sweep has to know of the next state, and the lead
// block writes that state to *to.
// A solve that has ended stays as it is.
struct NextState {
    double beta;
    int iter, done;
};
template <int BY>
__device__ __forceinline__ NextState phaseB_take(const CGScalars* __restrict__ from,
                                                 CGScalars* __restrict__ to,
                                                 const double* __restrict__ dep_rr, int n,
                                                 bool lead) {
    const bool writes = lead && threadIdx.x < kStateWords;
    uint64_t w = 0;
    if (writes) w = reinterpret_cast<const uint64_t*>(from)[threadIdx.x];
    const double rho = from->rho, tol = from->tol2phi2, drop = from->delta2 * from->rho_ru;
    const int max_iter = from->max_iter, updates = from->reliable_updates;
    NextState s{from->beta, from->iter, from->done};
    double rr;
    if constexpr (BY == kByWave) rr = reduce_deposits_wave(dep_rr, n);
    else rr = reduce_deposits_block(dep_rr, n);
    if (s.done == kRunning) {
        if (!isfinite(rr)) {
            s.done = kDoneBreakdown;
        } else {
            s.beta = rr / rho;
            s.iter += 1;
            s.done = rr <= tol || rr < drop ? kDoneIterConverged
                                            : s.iter >= max_iter ? kDoneMaxIter : kRunning;
            put_word(w, offsetof(CGScalars, rho), rr);
            put_word(w, offsetof(CGScalars, rho_prev), rho);
            put_word(w, offsetof(CGScalars, beta), s.beta);
            put_word(w, offsetof(CGScalars, iter), s.iter, max_iter);
        }
        put_word(w, offsetof(CGScalars, done), s.done, updates);
    }
    if (writes) reinterpret_cast<uint64_t*>(to)[threadIdx.x] = w;
    return s;
}

// Largest number of sums any reduction deposits per tile.
constexpr int kMaxNP = 2;

// Block sums of one tile into deposit slot `slot`.  Grid reductions are two
// kernels: every tile deposits its sums, then a one-block kernel adds the
// deposits in tile order (reduce_deposits) and updates the solver scalars.
// The kernel boundary in between is the device-wide synchronisation; on
// MI355X it costs about a launch, far less than per-block release fences
// and same-address atomics inside one kernel.
template <int BLOCK, int NP>
__device__ inline void deposit(const double (&part)[NP], double* partials, int slot) {
    double bs[NP];
#pragma unroll
    for (int k = 0; k < NP; ++k) bs[k] = block_sum<BLOCK>(part[k]);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int k = 0; k < NP; ++k)
            __hip_atomic_store(&partials[NP * slot + k], bs[k], __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
    }
}

#endif

}  // namespace hub
