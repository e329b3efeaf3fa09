// sweep.h -- the chunk step of the multi-candidate neighbourhood sweeps, used
// by the trace and the operator-log kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "layout.h"

namespace dtr {

// the lanes whose predicate holds (straight from the compare's mask)
__device__ __forceinline__ uint64_t ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

// a wave-uniform lane mask as this lane's predicate
__device__ __forceinline__ bool lane_in(uint64_t m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

// Keep the compiler from moving memory accesses across (one wavefront's
// accesses to LDS, and to a device-memory address, execute in order, so
// nothing has to be waited for).
__device__ __forceinline__ void lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// One chunk of 64 nodes, a node per lane, in an order in which every node's
// sources have smaller lane numbers: (s0, s1) holds the lane's sources in the
// chunk, a bit each (none for a node that takes part in no walk), (m0, m1)
// the candidates that have reached the node from outside the chunk, a bit
// each, and c0 its cost, below 2^28.  Nodes are taken one after another,
// eight to a step: a node's set is complete when its turn comes; it joins the
// sets of the later lanes that have it as a source, and lane i adds the
// node's cost and counts it if candidate i is in the set.  Steps that nothing
// has reached are skipped.  About eleven vector instructions a node.
__device__ __forceinline__ void sweep_chunk(uint32_t &m0, uint32_t &m1, uint32_t s0, uint32_t s1, uint32_t c0,
                                            uint64_t &sum, int32_t &cnt)
{
    constexpr int STEP = 8;
#pragma unroll
    for (int st = 0; st < WAVE / STEP; st++) {
        const uint64_t act = ballot((m0 | m1) != 0);
        if (!((act >> (STEP * st)) & ((1u << STEP) - 1))) continue;
        uint32_t part = 0;           // eight costs below 2^28 each
#pragma unroll
        for (int j = 0; j < STEP; j++) {
            const int k = STEP * st + j;
            const uint32_t b0 = __builtin_amdgcn_readlane(m0, k), b1 = __builtin_amdgcn_readlane(m1, k);
            const uint32_t to = (uint32_t)((int32_t)((k < 32 ? s0 : s1) << (31 - (k & 31))) >> 31);
            m0 |= to & b0;
            m1 |= to & b1;
            const bool in = lane_in((uint64_t)b0 | ((uint64_t)b1 << 32));
            const uint32_t ck = __builtin_amdgcn_readlane(c0, k);
            part += in ? ck : 0;
            cnt += in ? 1 : 0;
        }
        sum += part;
    }
}

// all lanes' bits joined into pend (uniform)
__device__ __forceinline__ void join_masks(uint64_t &pend, uint64_t to)
{
    for (uint64_t q; (q = ballot(to != 0));) {
        const int32_t j = __builtin_ctzll(q);
        const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)to, j);
        const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(to >> 32), j);
        const uint64_t t = (uint64_t)lo | ((uint64_t)hi << 32);
        pend |= t;
        to &= ~t;
    }
}

}  // namespace dtr
