// Data exchanged between the 64 lanes of a wavefront without the LDS crossbar (HIP, gfx950): data-parallel moves within
// rows of sixteen lanes, row and half swaps above.  A shuffle takes some 100 cycles there and back, and the steps of a sort,
// a sum or a scan wait for each other.  All lanes have to be active.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace eck {

// the value of the lane whose number differs in bit `stride` (a power of two, known after unrolling)
__device__ __forceinline__ uint32_t lane_exchange(uint32_t v, uint32_t stride)
{
    const int x = (int)v;
    switch (stride) {
    case 1: return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, true);  // quad_perm 1 0 3 2
    case 2: return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0x4E, 0xF, 0xF, true);  // quad_perm 2 3 0 1
    case 4: return (uint32_t)__builtin_amdgcn_mov_dpp(__builtin_amdgcn_mov_dpp(x, 0x141, 0xF, 0xF, true), 0x1B, 0xF, 0xF, true); // row_half_mirror, quad_perm 3 2 1 0
    case 8: return (uint32_t)__builtin_amdgcn_mov_dpp(x, 0x128, 0xF, 0xF, true); // row_ror:8
    case 16: {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false); // even rows twice, odd rows twice
        return threadIdx.x & 16 ? r[0] : r[1];
    }
    default: {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false); // lower half twice, upper half twice
        return threadIdx.x & 32 ? r[0] : r[1];
    }
    }
}
__device__ __forceinline__ uint64_t lane_exchange(uint64_t v, uint32_t stride)
{
    return ((uint64_t)lane_exchange((uint32_t)(v >> 32), stride) << 32) | lane_exchange((uint32_t)v, stride);
}
__device__ __forceinline__ double lane_exchange(double v, uint32_t stride)
{
    return __builtin_bit_cast(double, lane_exchange(__builtin_bit_cast(uint64_t, v), stride));
}

// the least of a wavefront's values, in every lane
__device__ __forceinline__ uint32_t wave_least(uint32_t v)
{
#pragma unroll
    for (uint32_t stride = 1; stride < 64; stride <<= 1) v = min(v, lane_exchange(v, stride));
    return v;
}

// the largest of a wavefront's values, none of them a NaN, in every lane
__device__ __forceinline__ double wave_most(double v)
{
    auto two = [](uint32_t hi, uint32_t lo) { return __builtin_bit_cast(double, (uint64_t)hi << 32 | lo); };
#pragma unroll
    for (uint32_t stride = 1; stride < 16; stride <<= 1) v = __builtin_fmax(v, lane_exchange(v, stride));
    {
        const uint64_t u = __builtin_bit_cast(uint64_t, v); // (both sides of a pair arrive in both of its lanes)
        const auto hi = __builtin_amdgcn_permlane16_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
        const auto lo = __builtin_amdgcn_permlane16_swap((uint32_t)u, (uint32_t)u, false, false);
        v = __builtin_fmax(two(hi[0], lo[0]), two(hi[1], lo[1]));
    }
    const uint64_t u = __builtin_bit_cast(uint64_t, v);
    const auto hi = __builtin_amdgcn_permlane32_swap((uint32_t)(u >> 32), (uint32_t)(u >> 32), false, false);
    const auto lo = __builtin_amdgcn_permlane32_swap((uint32_t)u, (uint32_t)u, false, false);
    return __builtin_fmax(two(hi[0], lo[0]), two(hi[1], lo[1]));
}

// the value of one lane (the same for all), in every lane
__device__ __forceinline__ int64_t lane_value(int64_t v, int lane)
{
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, lane), hi = (uint32_t)__builtin_amdgcn_readlane((int)(v >> 32), lane);
    return (int64_t)((uint64_t)hi << 32 | lo);
}
__device__ __forceinline__ int64_t last_lane(int64_t v) { return lane_value(v, 63); }

// sums over the lanes up to and including each: within rows, then the last lane of a row to the next row, then of the first
// two rows to the others
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t moved(uint32_t v) // zero where nothing arrives
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xF, false);
}
template <int CTRL, int ROWS>
__device__ __forceinline__ int64_t moved(int64_t v)
{
    return (int64_t)((uint64_t)moved<CTRL, ROWS>((uint32_t)(v >> 32)) << 32 | moved<CTRL, ROWS>((uint32_t)v));
}
template <class V>
__device__ __forceinline__ V wave_prefix_sum(V v)
{
    v += moved<0x111, 0xF>(v); // row_shr:1
    v += moved<0x112, 0xF>(v); // row_shr:2
    v += moved<0x114, 0xF>(v); // row_shr:4
    v += moved<0x118, 0xF>(v); // row_shr:8
    v += moved<0x142, 0xA>(v); // row_bcast:15 to rows 1 and 3
    v += moved<0x143, 0xC>(v); // row_bcast:31 to rows 2 and 3
    return v;
}

} // namespace eck
