// Sums over all blocks of one resident grid, and data handed from block to
// block, without a kernel boundary.
//
// Every block owns one 8-byte slot in each of three sets.  A sum deposits the
// block's part in its slot of the current set and then reads all slots of the
// set until none holds the empty mark, so that one store and one load carry
// both the barrier and the data.  A block that has seen a full set knows that
// every block has finished reading the set before it; it marks its own slot
// of that one empty again, two sums before it is next written.  All blocks
// add the slots in the same order and get the same bits.
//
// Stores and loads of slots and of handed-over data are agent-scope relaxed
// atomics: they go through to, and come from, the memory that all eight L2s
// share, so no cache has to be written back or invalidated (a release fence
// at every block costs tens of microseconds on this chip).  Order, where it
// is needed, comes from waiting for the stores' acknowledgement, after the
// block's own sums are formed (before them: 2.70 and 2.61 us an iteration of
// CG at 5^3 x 20, 4.33 and 4.24 at d = 1 4096 x 128).  Measured with
// slots 64 bytes apart: 1.8 us a sum over 16 blocks, 2.0 us over 64, 2.5 us
// over 256; 8 bytes apart 3.4 us over 256, whose deposits then share lines.
//
// Every wait is bounded: after `limit` reads the block gives up, which ends
// its kernel, and so the others' in turn.
#pragma once

#include "common.h"

namespace hub {

constexpr uint64_t kSlotEmpty = ~0ull;  // a NaN that no sum deposits
constexpr int kSlotStride = 8;          // slots 64 bytes apart
constexpr int kMaxResidentBlocks = 256;
constexpr size_t kSlotWords = size_t(3) * kMaxResidentBlocks * kSlotStride;

__device__ __forceinline__ void agent_store(double* p, double v) {
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ double agent_load(const double* p) {
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// Waits until every store of this wavefront has reached the shared memory.
__device__ __forceinline__ void wait_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Sums of N values over a wavefront, with the bits of wave_sum: the swap that
// brings the other half's addends can bring those of two values at once, each
// in its own half, so that four values take 7 adds and 7 moves instead of 24.
// Value k's sum is left in the lanes l with sum_of<N>(l) = k.
template <int N>
__device__ __forceinline__ int sum_of(int lane) {
    return N == 1 ? 0 : N == 2 ? lane >> 5 : (lane >> 5) + 2 * ((lane >> 4) & 1);
}
// v of the lower and w of the upper HALF of every 2 HALF lanes, each added to
// its value in the other half.
template <int HALF>
__device__ __forceinline__ double swap_add2(double v, double w) {
    const long long a = __builtin_bit_cast(long long, v), b = __builtin_bit_cast(long long, w);
    auto sw = [](unsigned x, unsigned y) {
        if constexpr (HALF == 32) return __builtin_amdgcn_permlane32_swap(x, y, false, false);
        else return __builtin_amdgcn_permlane16_swap(x, y, false, false);
    };
    const auto l = sw((unsigned)a, (unsigned)b);
    const auto h = sw((unsigned)(a >> 32), (unsigned)(b >> 32));
    return __builtin_bit_cast(double, (long long)((unsigned long long)h[0] << 32 | l[0])) +
           __builtin_bit_cast(double, (long long)((unsigned long long)h[1] << 32 | l[1]));
}
template <int N>
__device__ __forceinline__ double wave_sums(const double (&v)[N]) {
    static_assert(N == 1 || N == 2 || N == 4, "");
    if constexpr (N == 1) return wave_sum(v[0]);
    double s;
    if constexpr (N == 4) s = swap_add2<16>(swap_add2<32>(v[0], v[1]), swap_add2<32>(v[2], v[3]));
    else s = swap_add<16>(swap_add2<32>(v[0], v[1]));
    s += dpp_move<0x128>(s);  // as in wave_sum
    s += dpp_move<0x124>(s);
    s += dpp_move<0x4e>(s);
    s += dpp_move<0xb1>(s);
    return s;
}

// N sums at a time: one, or pairs whose two slots lie side by side in a block's
// line.  A wavefront reads a pair with 16-byte loads, as many requests as for
// one sum (four sums with 8-byte loads, a wavefront each: 1.3 us more).
// Each slot carries its own mark, so that of a pair either may come first.
constexpr int kGridSumMax = 4;
template <int N>
struct GridSum {
    static_assert(N == 1 || (N % 2 == 0 && N <= kGridSumMax && N <= kSlotStride), "pairs");
    static constexpr int kPair = N == 1 ? 1 : 2, kReaders = N / kPair;
    static constexpr int kMaxWaves = 8;
    static constexpr int kLdsDoubles = N * kMaxWaves + N + kReaders;
    uint64_t* slots;  // kSlotWords words, all kSlotEmpty when the kernel starts
    double* lds;      // kLdsDoubles
    int limit;
    int turn;         // set of the next sums

    __device__ __forceinline__ uint64_t* slot(int set, int block, int which) const {
        return slots + ((size_t)set * kMaxResidentBlocks + block) * kSlotStride + which;
    }

    // Deposits this block's sums of v; what the block has stored with
    // agent_store is then visible to whoever sees the deposit.  All lanes of
    // a block of kReaders to kMaxWaves wavefronts.
    __device__ __forceinline__ void deposit(const double (&v)[N]) {
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        const double part = wave_sums(v);
        if ((lane & (64 / N - 1)) == 0) lds[kMaxWaves * sum_of<N>(lane) + w] = part;
        wait_stores();  // on their way while the sums were formed
        __syncthreads();
        if (lane < kPair && w < kReaders) {
            const int which = kPair * w + lane;
            double s = 0.0;
            const int nw = (int)(blockDim.x >> 6);
#pragma unroll
            for (int k = 0; k < kMaxWaves; ++k) s += k < nw ? lds[kMaxWaves * which + k] : 0.0;
            uint64_t u = (uint64_t)__double_as_longlong(s);
            if (s != s) u = 0x7ff8000000000000ull;
            __hip_atomic_store(slot(turn, blockIdx.x, which), u, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        }
    }

    // The sums over all blocks, the same bits in every lane of each.  False
    // when the wait was given up: the block must end then.  All lanes.
    __device__ __forceinline__ bool wait(double (&total)[N]) {
        constexpr int kPer = kMaxResidentBlocks / 64;
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        double* tot = lds + N * kMaxWaves;
        if (w < kReaders) {
            const int nb = (int)gridDim.x;
            const uint64_t* set = slot(turn, 0, kPair * w);
            uint64_t u[kPer][kPair];
            bool full = false;
            for (int n = 0; n < limit; ++n) {
                bool ok = true;
#pragma unroll
                for (int j = 0; j < kPer; ++j)  // past the last block: its slot again
                    load(set + min(lane + 64 * j, nb - 1) * kSlotStride, u[j]);
#pragma unroll
                for (int j = 0; j < kPer; ++j)
#pragma unroll
                    for (int k = 0; k < kPair; ++k) ok = ok && u[j][k] != kSlotEmpty;
                if (__all(ok)) {
                    full = true;
                    break;
                }
            }
            double s[kPair];
#pragma unroll
            for (int k = 0; k < kPair; ++k) {
                s[k] = 0.0;
#pragma unroll
                for (int j = 0; j < kPer; ++j)
                    s[k] += lane + 64 * j < nb ? __longlong_as_double((long long)u[j][k]) : 0.0;
            }
            const double t = wave_sums(s);
            if ((lane & (64 / kPair - 1)) == 0) {
                const int which = kPair * w + sum_of<kPair>(lane);
                tot[which] = t;
                if (lane == 0) tot[N + w] = full ? 1.0 : 0.0;
                // the set before this one
                __hip_atomic_store(slot(turn == 0 ? 2 : turn - 1, blockIdx.x, which), kSlotEmpty,
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        __syncthreads();
        bool all = true;
#pragma unroll
        for (int k = 0; k < N; ++k) total[k] = tot[k];
#pragma unroll
        for (int k = 0; k < kReaders; ++k) all = all && tot[N + k] != 0.0;
        turn = turn == 2 ? 0 : turn + 1;
        return all;
    }

  private:
    __device__ __forceinline__ void load(const uint64_t* p, uint64_t (&u)[1]) const {
        u[0] = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // Agent scope (sc1); not kept from one read to the next.
    __device__ __forceinline__ void load(const uint64_t* p, uint64_t (&u)[2]) const {
        constexpr int kAgentScope = 16, kRawBuffer = 0x00027000;
        asm volatile("" ::: "memory");
        const auto rsrc = __builtin_amdgcn_make_buffer_rsrc((void*)slots, 0, (int)(8 * kSlotWords),
                                                            kRawBuffer);
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(
            rsrc, (int)((const char*)p - (const char*)slots), 0, kAgentScope);
        u[0] = (uint64_t)(uint32_t)v[1] << 32 | (uint32_t)v[0];
        u[1] = (uint64_t)(uint32_t)v[3] << 32 | (uint32_t)v[2];
    }
};

}  // namespace hub
