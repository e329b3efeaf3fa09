// score.h -- exact score comparison at float cost, and the wavefront
// reductions it needs; used by the trace and the operator-log kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "sweep.h"

namespace dtr {

typedef unsigned __int128 u128;

// lane j's value (j wave-uniform)
__device__ __forceinline__ uint64_t readlane64(uint64_t v, int32_t j)
{
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, j);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(v >> 32), j);
    return ((uint64_t)hi << 32) | lo;
}

// x's minimum over the lanes that are not NaN (uniform): row shifts, then the
// rows' results passed on, a few cycles a step where a shuffle goes through LDS
__device__ __forceinline__ float wave_min(float x)
{
    auto step = [&](auto ctrl, auto rows) {
        const int v = __builtin_bit_cast(int, x);
        x = fminf(x, __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(v, v, ctrl.value, rows.value, 0xF, false)));
    };
    using std::integral_constant;
    step(integral_constant<int, 0x111>(), integral_constant<int, 0xF>());    // row_shr:1
    step(integral_constant<int, 0x112>(), integral_constant<int, 0xF>());    // row_shr:2
    step(integral_constant<int, 0x114>(), integral_constant<int, 0xF>());    // row_shr:4
    step(integral_constant<int, 0x118>(), integral_constant<int, 0xF>());    // row_shr:8
    step(integral_constant<int, 0x142>(), integral_constant<int, 0xA>());    // row_bcast:15 into rows 1 and 3
    step(integral_constant<int, 0x143>(), integral_constant<int, 0xC>());    // row_bcast:31 into rows 2 and 3
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, x), WAVE - 1));
}

// x summed over the lanes (uniform), as wave_min
__device__ __forceinline__ uint64_t wave_add(uint64_t x)
{
    auto step = [&](auto ctrl, auto rows) {
        const int lo = (int)(uint32_t)x, hi = (int)(uint32_t)(x >> 32);
        const uint32_t a = (uint32_t)__builtin_amdgcn_update_dpp(0, lo, ctrl.value, rows.value, 0xF, false);
        const uint32_t b = (uint32_t)__builtin_amdgcn_update_dpp(0, hi, ctrl.value, rows.value, 0xF, false);
        x += (uint64_t)a | ((uint64_t)b << 32);
    };
    using std::integral_constant;
    step(integral_constant<int, 0x111>(), integral_constant<int, 0xF>());
    step(integral_constant<int, 0x112>(), integral_constant<int, 0xF>());
    step(integral_constant<int, 0x114>(), integral_constant<int, 0xF>());
    step(integral_constant<int, 0x118>(), integral_constant<int, 0xF>());
    step(integral_constant<int, 0x142>(), integral_constant<int, 0xA>());
    step(integral_constant<int, 0x143>(), integral_constant<int, 0xC>());
    return readlane64(x, WAVE - 1);
}

// a strictly better (lower score) than b; ties go to the smaller id
__device__ __forceinline__ bool better(uint64_t na, u128 da, int32_t ia, uint64_t nb, u128 db, int32_t ib)
{
    u128 l = (u128)na * db;
    u128 r = (u128)nb * da;
    if (l != r) return l < r;
    return ia < ib;
}

// Scores are N / (da * db) with N < 2^64 and da * db < 2^76.  A float
// estimate decides every comparison whose two estimates differ by more than a
// factor 1 -+ 2^-16; the rest (near ties, exact ties, 0/0) are decided
// exactly by 128-bit cross-multiplication, so the outcome is always that of
// the exact comparison.  Error of the estimate: each u64f conversion rounds
// twice (the high and low 32-bit halves, then the fused sum), under
// (1 + 2^-24)^2 - 1 < 2^-22.9; the product da * db adds one rounding
// (2^-24), v_rcp_f32 at most 1 ulp (2^-23) and the final product one
// rounding (2^-24): in all below 3 * 2^-22.9 + 2^-23 + 2 * 2^-24 < 2^-20.4.
// Two estimates within the margin can therefore never be ordered wrongly by
// the float test: (1 - 2^-16) (1 + 2^-24) (1 + 2^-20.4)^2 < 1.
constexpr float FILTER_LO = 1.0f - 0x1p-16f;
constexpr float FILTER_HI = 1.0f + 0x1p-16f;

__device__ __forceinline__ float u64f(uint64_t x)
{
    return fmaf((float)(uint32_t)(x >> 32), 4294967296.0f, (float)(uint32_t)x);
}

__device__ __forceinline__ float score_est(uint64_t N, uint64_t da, uint64_t db)
{
    return u64f(N) * __builtin_amdgcn_rcpf(u64f(da) * u64f(db));   // 0 -> inf, 0/0 -> NaN
}

__device__ __forceinline__ bool better_exact(uint64_t na, uint64_t daa, uint64_t dba, int32_t ia, uint64_t nb,
                                             uint64_t dab, uint64_t dbb, int32_t ib)
{
    return better(na, (u128)daa * dba, ia, nb, (u128)dab * dbb, ib);
}

struct Best {
    float sc, lo, hi;    // estimated score of the best and its decision bounds
    uint64_t N, da, db;
    int32_t id, slot, have;
};

// keep the candidate if valid and better than the current best
__device__ __forceinline__ void take(Best &b, bool valid, float sc, uint64_t N, uint64_t da, uint64_t db, int32_t id,
                                     int32_t slot)
{
    const bool dec_better = sc < b.lo;
    const bool dec_worse = sc > b.hi;
    bool t = valid && (!b.have || dec_better);
    const bool close = valid && b.have && !dec_better && !dec_worse;
    if (ballot(close)) {
        if (close) t = better_exact(N, da, db, id, b.N, b.da, b.db, b.id);
    }
    b.sc = t ? sc : b.sc;
    b.lo = t ? sc * FILTER_LO : b.lo;
    b.hi = t ? sc * FILTER_HI : b.hi;
    b.N = t ? N : b.N;
    b.da = t ? da : b.da;
    b.db = t ? db : b.db;
    b.id = t ? id : b.id;
    b.slot = t ? slot : b.slot;
    b.have = t ? 1 : b.have;
}

// the lane that holds the exact (score, id) minimum of the lanes' bests
// (uniform; -1: none): the smallest estimate bounds the winner, and only the
// lanes within the filter margin of it (usually one) are compared exactly
__device__ __forceinline__ int32_t best_lane(const Best &best)
{
    const float thr = wave_min(best.have ? best.sc : __builtin_inff()) * FILTER_HI;
    uint64_t m = ballot(best.have && !(best.sc > thr));     // NaN estimates stay in
    if (!m) return -1;
    int32_t w = __builtin_ctzll(m);
    for (m &= m - 1; m; m &= m - 1) {
        const int32_t j = __builtin_ctzll(m);
        if (better_exact(readlane64(best.N, j), readlane64(best.da, j), readlane64(best.db, j),
                         __builtin_amdgcn_readlane(best.id, j), readlane64(best.N, w), readlane64(best.da, w),
                         readlane64(best.db, w), __builtin_amdgcn_readlane(best.id, w)))
            w = j;
    }
    return w;
}

}  // namespace dtr
