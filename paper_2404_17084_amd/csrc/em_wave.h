// Wavefront-level helpers for device code (wave64, gfx950).
#pragma once

#include <hip/hip_runtime.h>

#include "em_internal.h"

namespace em {

// Slot of this lane in a wave-wide push (lanes in the mask, or with want = true,
// in lane order); count (wave-uniform) grows by the number of pushing lanes.  Call in
// wave-uniform control flow.
__device__ __forceinline__ int wave_push(uint64_t m, int &count)
{
    const int slot = __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, (unsigned)count));
    count += __popcll(m);
    return slot;
}
__device__ __forceinline__ int wave_push(bool want, int &count)
{
    return wave_push(__builtin_amdgcn_ballot_w64(want), count);
}

// Set lanes of mask m below this lane.
__device__ __forceinline__ int lanes_below(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

// Orders LDS writes of one wavefront before its later reads by other lanes.
__device__ __forceinline__ void lds_sync_wave()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Reduction of a double over the wavefront by data-parallel primitives (three
// vector instructions a step, against two trips through the LDS crossbar),
// wave-uniform; `identity` stands in for lanes without a partner.
template <class Op>
__device__ __forceinline__ double wave_reduce(double v, double identity, Op op)
{
    const uint64_t id = (uint64_t)__double_as_longlong(identity);
#define EM_DPP_STEP(ctrl, rows)                                                                               \
    {                                                                                                         \
        const uint64_t b = (uint64_t)__double_as_longlong(v);                                                 \
        const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)id, (int)(uint32_t)b, ctrl,   \
                                                                  rows, 0xf, false);                          \
        const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(id >> 32), (int)(b >> 32), ctrl, rows, \
                                                                  0xf, false);                                \
        v = op(v, __longlong_as_double((int64_t)(((uint64_t)hi << 32) | lo)));                                \
    }
    EM_DPP_STEP(0xB1, 0xf)   // quad_perm 1,0,3,2
    EM_DPP_STEP(0x4E, 0xf)   // quad_perm 2,3,0,1
    EM_DPP_STEP(0x141, 0xf)  // row_half_mirror
    EM_DPP_STEP(0x140, 0xf)  // row_mirror: every row of 16 has its result
    EM_DPP_STEP(0x142, 0xa)  // row_bcast15 into rows 1 and 3
    EM_DPP_STEP(0x143, 0xc)  // row_bcast31 into rows 2 and 3
#undef EM_DPP_STEP
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(b >> 32), 63);
    return __longlong_as_double((int64_t)(((uint64_t)hi << 32) | lo));
}

// S_a is summed in 2^-52 fixed point with 64-bit integer atomics (each term
// rounded by at most 2^-53, the sum exact, so it does not depend on the order
// of the additions, and a pair's term can be replaced by adding the difference).
__device__ __forceinline__ unsigned long long fixed52(double f)
{
    return (unsigned long long)__double2ll_rn(f * 4503599627370496.0);
}

// This workgroup's copy of the counters (em_internal.h).
__device__ __forceinline__ unsigned long long *counter_copy(unsigned long long *counters)
{
    return counters + (blockIdx.x % (unsigned)kCounterCopies) * (unsigned)kCounterStride;
}

// Logical index of this workgroup in an XCD-aware order.  Workgroups are
// dispatched round-robin over the 8 XCDs (workgroup b to XCD b mod 8); this
// gives XCD x a contiguous run of logical indices (x * per + min(x, rem) ...,
// per = nb / 8, rem = nb mod 8), so neighbouring work shares one L2.  A
// bijection of [0, nb).
__device__ __forceinline__ unsigned xcd_block(unsigned b, unsigned nb)
{
    const unsigned x = b & 7u, k = b >> 3, per = nb >> 3, rem = nb & 7u;
    return x * per + (x < rem ? x : rem) + k;
}

}  // namespace em
