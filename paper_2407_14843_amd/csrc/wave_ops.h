// Operations over the lanes of one wavefront that several kernels share.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace themis {

// Orders the LDS traffic of one wavefront: what its lanes wrote before is
// visible to all its lanes after (a wavefront's LDS operations complete in
// order; this only keeps the compiler from moving them across).
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Inclusive prefix sums (MIN = false) or running minima (MIN = true) over segments
// of `width` consecutive lanes (a power of two; q = lane within its segment), with
// the data-parallel primitives instead of LDS permutes: shifts by 1, 2, 4, 8 inside
// each row of 16 lanes (a lane whose source lies outside its row, or its segment,
// takes the identity), then the last lane of a row of 16 broadcast to the next row
// (32-lane segments: rows 1 and 3) and lane 31 to rows 2 and 3 (64).
template <bool MIN, int CTRL, int ROWS>
__device__ __forceinline__ uint32_t scan_step(uint32_t x, bool keep)
{
    uint32_t t = (uint32_t)__builtin_amdgcn_update_dpp(MIN ? -1 : 0, (int)x, CTRL, ROWS, 0xF, false);
    if (!keep) t = MIN ? 0xFFFFFFFFu : 0u;
    return MIN ? (t < x ? t : x) : x + t;
}

template <bool MIN>
__device__ __forceinline__ uint32_t segmented_scan(uint32_t x, uint32_t q, uint32_t width)
{
    // segments shorter than a row of 16: a shift must not reach into the segment before
    const bool narrow = width < 16u;
    if (width > 1u) x = scan_step<MIN, 0x111, 0xF>(x, !narrow || q >= 1u);
    if (width > 2u) x = scan_step<MIN, 0x112, 0xF>(x, !narrow || q >= 2u);
    if (width > 4u) x = scan_step<MIN, 0x114, 0xF>(x, !narrow || q >= 4u);
    if (width > 8u) x = scan_step<MIN, 0x118, 0xF>(x, true);
    if (width > 16u) x = scan_step<MIN, 0x142 /* row_bcast:15 */, 0xA>(x, true);
    if (width > 32u) x = scan_step<MIN, 0x143 /* row_bcast:31 */, 0xC>(x, true);
    return x;
}

// The whole wavefront as one segment.
template <bool MIN>
__device__ __forceinline__ uint32_t wave_scan(uint32_t x)
{
    return segmented_scan<MIN>(x, 0u, 64u);
}

// The value of the lane below; lane 0 gets `first`.
__device__ __forceinline__ uint32_t from_lane_below(uint32_t x, uint32_t first)
{
    return (uint32_t)__builtin_amdgcn_update_dpp((int)first, (int)x, 0x138 /* wave_shr:1 */, 0xF, 0xF,
                                                 false);
}

__device__ __forceinline__ uint32_t lane_value(uint32_t x, int lane)
{
    return (uint32_t)__builtin_amdgcn_readlane((int)x, lane);
}

// A butterfly over groups of `width` lanes (a power of two): calls f(of) for partners at
// distance 1, 2, 4, ..; of(x) is the partner's x.  What f makes of a lane's values and its
// partner's has to be the same for both.  Within 16 lanes by data-parallel primitives:
// after the steps before it, a mirrored half row is as good as a distance of 4, a
// mirrored row as one of 8.
template <int CTRL>
__device__ __forceinline__ uint32_t mirrored(uint32_t x)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, false);
}
template <typename F>
__device__ __forceinline__ void with_partners(int width, F f)
{
    if (width > 1) f([](uint32_t x) { return mirrored<0xB1 /* quad_perm:[1,0,3,2] */>(x); });
    if (width > 2) f([](uint32_t x) { return mirrored<0x4E /* quad_perm:[2,3,0,1] */>(x); });
    if (width > 4) f([](uint32_t x) { return mirrored<0x141 /* row_half_mirror */>(x); });
    if (width > 8) f([](uint32_t x) { return mirrored<0x140 /* row_mirror */>(x); });
    // (swapped with itself, a value comes back as the lane's and its partner's)
    if (width > 16) f([](uint32_t x) {
        const auto both = __builtin_amdgcn_permlane16_swap(x, x, false, false);
        return both[0] ^ both[1] ^ x;
    });
    if (width > 32) f([](uint32_t x) {
        const auto both = __builtin_amdgcn_permlane32_swap(x, x, false, false);
        return both[0] ^ both[1] ^ x;
    });
}

// Sum over all lanes, the same in every lane (and known to be).
__device__ __forceinline__ uint32_t wave_sum(uint32_t x) { return lane_value(wave_scan<false>(x), 63); }

}  // namespace themis
