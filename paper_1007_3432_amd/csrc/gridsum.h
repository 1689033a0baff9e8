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

// Two sums at a time, each with its own slot in a block's line.
struct GridSum {
    static constexpr int kMaxWaves = 8;
    static constexpr int kLdsDoubles = 2 * kMaxWaves + 4;
    uint64_t* slots;  // kSlotWords words, all kSlotEmpty when the kernel starts
    double* lds;      // kLdsDoubles
    int limit;
    int turn;         // set of the next sums

    __device__ __forceinline__ uint64_t* slot(int set, int block, int which) const {
        return slots + ((size_t)set * kMaxResidentBlocks + block) * kSlotStride + which;
    }

    // Deposits this block's sums of v0 and v1; what the block has stored with
    // agent_store is then visible to whoever sees the deposit.  All lanes of
    // a block of two to kMaxWaves wavefronts.
    __device__ __forceinline__ void deposit(double v0, double v1) {
        v0 = wave_sum(v0);
        v1 = wave_sum(v1);
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        if (lane == 0) {
            lds[w] = v0;
            lds[kMaxWaves + w] = v1;
        }
        wait_stores();  // on their way while the sums were formed
        __syncthreads();
        if (lane == 0 && w < 2) {
            double s = 0.0;
            const int nw = (int)(blockDim.x >> 6);
#pragma unroll
            for (int k = 0; k < kMaxWaves; ++k) s += k < nw ? lds[kMaxWaves * w + k] : 0.0;
            uint64_t u = (uint64_t)__double_as_longlong(s);
            if (s != s) u = 0x7ff8000000000000ull;
            __hip_atomic_store(slot(turn, blockIdx.x, w), u, __ATOMIC_RELAXED,
                               __HIP_MEMORY_SCOPE_AGENT);
        }
    }

    // The sums over all blocks, the same bits in every lane of each.  False
    // when the wait was given up: the block must end then.  All lanes.
    __device__ __forceinline__ bool wait(double& total0, double& total1) {
        constexpr int kPer = kMaxResidentBlocks / 64;
        const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
        if (w < 2) {  // a wavefront for each sum
            const int nb = (int)gridDim.x;
            const uint64_t* set = slot(turn, 0, w);
            uint64_t u[kPer];
            bool full = false;
            for (int n = 0; n < limit; ++n) {
                bool ok = true;
#pragma unroll
                for (int j = 0; j < kPer; ++j)  // past the last block: its slot again
                    u[j] = __hip_atomic_load(set + min(lane + 64 * j, nb - 1) * kSlotStride,
                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
                for (int j = 0; j < kPer; ++j) ok = ok && u[j] != kSlotEmpty;
                if (__all(ok)) {
                    full = true;
                    break;
                }
            }
            double s = 0.0;
#pragma unroll
            for (int j = 0; j < kPer; ++j)
                s += lane + 64 * j < nb ? __longlong_as_double((long long)u[j]) : 0.0;
            s = wave_sum(s);
            if (lane == 0) {
                lds[2 * kMaxWaves + w] = s;
                lds[2 * kMaxWaves + 2 + w] = full ? 1.0 : 0.0;
                // the set before this one
                __hip_atomic_store(slot(turn == 0 ? 2 : turn - 1, blockIdx.x, w), kSlotEmpty,
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        __syncthreads();
        total0 = lds[2 * kMaxWaves];
        total1 = lds[2 * kMaxWaves + 1];
        turn = turn == 2 ? 0 : turn + 1;
        return lds[2 * kMaxWaves + 2] != 0.0 && lds[2 * kMaxWaves + 3] != 0.0;
    }
};

}  // namespace hub
