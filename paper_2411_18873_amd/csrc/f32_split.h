// fp32 numbers as sums of three bfloat16 ones (HIP, gfx950), for products of fp32 matrices on the bfloat16 matrix cores.
//
// Rounded to nearest, x = x0 + x1 + x2 exactly, with |x1| <= 2^-9 |x| and |x2| <= 2^-18 |x|, for |x| >= 2^-110 and zero: below
// that the last part falls under the least bfloat16, and what is lost grows from 2^-22 of the number at 2^-112 to 2^-10 at 2^-124.
// Of the nine products of two such sums the six largest are kept; the others are below 2^-25 of the product together, less than
// the rounding of an fp32 product.  A number that is not finite, or rounds to infinity, has a NaN among its parts.
//
// What keeps a layer's sums as good as fp32 ones: no input below 2^-40 and no weight below 2^-50 but zeros.  Then no product
// is below 2^-90, so the rounding of a sum of them (2^-114) hides what the parts of a small output lose (2^-134), and an output
// that is a bias alone has its parts if the bias is not below 2^-100.  Models with other weights, and candidates with other
// features, are worked out in fp32 products.
//
// Weights of a layer ([K][H], row-major) as operands of v_mfma_f32_16x16x32_bf16, rows = units (lane = 16 p + c holds A[c][8p ..
// 8p + 7], B[8p .. 8p + 7][c], D[4p + q][c] in register q): fragments [unit tile][group of 32 inputs][part][lane][8], zeros past K
// and H.
#pragma once
#include "eck_internal.h"

namespace eck {
namespace split {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int PARTS = 3;

__host__ __device__ inline uint32_t tiles_of(int H) { return (uint32_t)(H + 15) / 16; }
__host__ __device__ inline uint32_t groups_of(int K) { return (uint32_t)(K + 31) / 32; }
// fragments (all parts) of the two hidden layers, 64 lanes each
__host__ __device__ inline uint32_t fragments1(int F, int H1) { return tiles_of(H1) * groups_of(F); }
__host__ __device__ inline uint32_t fragments2(int H1, int H2) { return tiles_of(H2) * groups_of(H1); }
__host__ __device__ inline uint32_t fragments(int F, int H1, int H2) { return fragments1(F, H1) + fragments2(H1, H2); }
// behind the fragments a byte for each, not zero where it holds a weight outside the range (or its unit's bias is); whole words
__host__ __device__ inline uint32_t flag_words(int F, int H1, int H2) { return (fragments(F, H1, H2) + 3) / 4; }
inline uint64_t packed_bytes(int F, int H1, int H2) { return (uint64_t)fragments(F, H1, H2) * PARTS * 1024 + 4 * flag_words(F, H1, H2); }

constexpr uint32_t LEAST_INPUT = 0x2B800000, LEAST_WEIGHT = 0x26800000, LEAST_BIAS = 0x0D800000; // 2^-40, 2^-50, 2^-100
// the order of magnitudes as numbers, zero last; x lies below `least` (a float's bits) and is no zero if this is below
// magnitude_order(least)
__host__ __device__ inline uint32_t magnitude_order(uint32_t bits) { return (bits << 1) - 1; }

// the parts of two numbers, two to a word
__device__ __forceinline__ void split_two(float a, float b, uint32_t (&part)[PARTS])
{
#pragma unroll
    for (int i = 0; i < PARTS; ++i) {
        const bf16x2 two = {(__bf16)a, (__bf16)b};
        part[i] = __builtin_bit_cast(uint32_t, two);
        a -= __uint_as_float(part[i] << 16);
        b -= __uint_as_float(part[i] & 0xFFFF0000u);
    }
}

// lane `lane` of fragment `frag` of a model's layers: eight weights, split (all lanes of a wavefront)
__device__ __forceinline__ void pack_lane(const float *__restrict__ w1, const float *__restrict__ b1, const float *__restrict__ w2,
                                          const float *__restrict__ b2, int F, int H1, int H2, uint32_t frag, uint32_t lane,
                                          unsigned char *__restrict__ packed)
{
    const uint32_t n1 = fragments1(F, H1);
    const bool second = frag >= n1;
    const float *w = second ? w2 : w1;
    const int K = second ? H1 : F, H = second ? H2 : H1;
    const uint32_t f = second ? frag - n1 : frag, groups = groups_of(K), unit = 16 * (f / groups) + (lane & 15);
    const uint32_t k0 = 32 * (f % groups) + 8 * (lane >> 4);
    u32x4 out[PARTS];
    bool outside = false;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float two[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const uint32_t k = k0 + 2 * e + i;
            two[i] = k < (uint32_t)K && unit < (uint32_t)H ? w[(uint64_t)k * H + unit] : 0.0f;
            const uint32_t order = magnitude_order(__float_as_uint(two[i]));
            // (from the second bound on, infinity in bfloat16)
            outside |= order < magnitude_order(LEAST_WEIGHT) || (order >= magnitude_order(0x7F7F8000) && order != 0xFFFFFFFFu);
        }
        uint32_t part[PARTS];
        split_two(two[0], two[1], part);
#pragma unroll
        for (int i = 0; i < PARTS; ++i) out[i][e] = part[i];
    }
#pragma unroll
    for (int i = 0; i < PARTS; ++i) reinterpret_cast<u32x4 *>(packed)[((uint64_t)frag * PARTS + i) * 64 + lane] = out[i];
    if (k0 == 0 && unit < (uint32_t)H) {
        const uint32_t order = magnitude_order(__float_as_uint((second ? b2 : b1)[unit]));
        outside |= (!second && order < magnitude_order(LEAST_BIAS)) || (order >= magnitude_order(0x7F800000) && order != 0xFFFFFFFFu);
    }
    const uint64_t any = __ballot(outside);
    if (lane == 0) packed[(uint64_t)fragments(F, H1, H2) * PARTS * 1024 + frag] = any != 0;
}

} // namespace split
} // namespace eck
