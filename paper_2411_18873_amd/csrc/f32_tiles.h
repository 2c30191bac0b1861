// The fp32 matrix-core kernels of the refit (HIP, gfx950): the tile layout and the loads of a layer's weights.
//
// v_mfma_f32_16x16x4_f32, fp32 operands and accumulation.  The network is evaluated transposed, rows = hidden units
// (A = weights), columns = candidates or minibatch rows (B = activations).  Lane = 16 p + c (quarter p):
//   A (16 x 4):  lane holds A[c][p]      B (4 x 16): lane holds B[p][c]
//   D (16 x 16): lane holds D[4p + q][c] in register q
// The reduction runs in groups of sixteen units: in step t of group g quarter p supplies unit 16g + 4p + t, so the four
// steps of a group take one 16-byte LDS read per lane for B, and a D tile is one 16-byte LDS write.  Activations sit in
// LDS as [unit / 4][column][unit % 4]: reads and writes touch 16 bytes times consecutive columns, no conflicts.
//
// A wavefront takes a slice of 16 J units of a layer, J <= 4, as J tiles whose rows interleave: row c of tile j is unit
// J c + j of the slice, so that one load of J consecutive weights per lane serves J tiles, and the 4 J values a lane
// holds of a column are consecutive units: value e = 0 .. 4 J - 1 at quarter p is unit first + 4 J p + e, in register
// e / J of tile e % J.
#pragma once
#include "eck_internal.h"

namespace eck {
namespace f32 {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef int i32x3 __attribute__((ext_vector_type(3)));
typedef int i32x2 __attribute__((ext_vector_type(2)));

constexpr int RSRC_FLAGS = 0x00020000; // buffer descriptor: raw 32-bit data

struct F32Layer {
    const float *w, *b; // [K][H] row-major, [H]
    int K, H;
};

// One wavefront's part of a layer: units first .. first + 16 J - 1.  Those past H get weights from the next row of the
// matrix -- or, in its last row, from what follows in the parameter vector: at most 63 floats on, within the moments that
// always follow -- and are never used.
template <int J>
struct Slice {
    const F32Layer &l;
    int first, p, c;
    __amdgpu_buffer_rsrc_t weights;
    uint32_t lane_bytes; // of this lane's weights in the rows of quarter p, from the first row of a group

    __device__ Slice(const F32Layer &layer, int first_unit, int p_, int c_) : l(layer), first(first_unit), p(p_), c(c_)
    {
        weights = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(l.w), 0, (l.K * l.H + 64) * 4, RSRC_FLAGS);
        lane_bytes = 4u * (uint32_t)(4 * p * l.H + first + J * c);
    }

    // The weights of step t of group g: quarter p wants row 16g + 4p + t.  A scalar row offset and one 32-bit lane
    // offset: no vector instructions.
    __device__ __forceinline__ void row(int g, int t, float (&a)[J]) const
    {
        const int row_bytes = (16 * g + t) * l.H * 4;
        if constexpr (J == 4) {
            const i32x4 f = __builtin_amdgcn_raw_buffer_load_b128(weights, lane_bytes, row_bytes, 0);
#pragma unroll
            for (int j = 0; j < J; ++j) a[j] = __int_as_float(f[j]);
        } else if constexpr (J == 3) {
            const i32x3 f = __builtin_amdgcn_raw_buffer_load_b96(weights, lane_bytes, row_bytes, 0);
#pragma unroll
            for (int j = 0; j < J; ++j) a[j] = __int_as_float(f[j]);
        } else if constexpr (J == 2) {
            const i32x2 f = __builtin_amdgcn_raw_buffer_load_b64(weights, lane_bytes, row_bytes, 0);
#pragma unroll
            for (int j = 0; j < J; ++j) a[j] = __int_as_float(f[j]);
        } else {
            a[0] = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(weights, lane_bytes, row_bytes, 0));
        }
    }

    // The last group of a reduction that is not a multiple of sixteen: rows past K read as zero.
    __device__ __forceinline__ void partial_group(int g, float (&a)[4][J]) const
    {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int j = 0; j < J; ++j) {
                const int k = 16 * g + 4 * p + t;
                const float v = l.w[(int64_t)min(k, l.K - 1) * l.H + min(first + J * c + j, l.H - 1)];
                a[t][j] = k < l.K ? v : 0.0f;
            }
    }
};

} // namespace f32
} // namespace eck
