// Internal declarations shared by the translation units of libeck (HIP, gfx950).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "eck.h"

#define ECK_HIP_TRY(expr)                       \
    do {                                        \
        if ((expr) != hipSuccess) {             \
            (void)hipGetLastError();            \
            return ECK_EDEVICE;                 \
        }                                       \
    } while (0)

namespace eck {

constexpr int NAX = 5;      // axis slots: four spatial, one reduction
constexpr int RED_AXIS = 4; // GEMM/BGEMM: (B, M, N, -, K); CONV2D: (N, K_out, H_out, W_out, C)

// Everything the enumerate / feature kernels need about one space; passed by value.
struct SpaceParams {
    int32_t kind, op, n_genes, n_split;
    uint32_t radix[8];
    int32_t split_axis[NAX];   // axis slot of split gene s
    uint32_t table_off[NAX];   // first entry of split gene s in the concatenated table
    uint32_t table_total;      // entries in the concatenated table
    uint32_t ext[NAX];         // true extents per axis slot
    uint32_t R, S, stride;
    uint32_t elem_bytes;
    uint32_t hw_num_cu, hw_wave, hw_lds_bytes, hw_max_threads_cu, hw_max_blocks_cu;
    int32_t vec_axis;          // spatial axis whose innermost level is contiguous in memory
    uint64_t true_out, true_red, flop_useful, compulsory_bytes, compulsory_in_bytes;
    float const_x[6];          // transformed per-space constants: features 0, 22, 60, 61, 62, 63
};

// bytes before the tables in a space's device copy
constexpr size_t kDevHeader = (sizeof(SpaceParams) + 15) & ~(size_t)15;

inline hipStream_t as_stream(void *s) { return reinterpret_cast<hipStream_t>(s); }

} // namespace eck

struct eck_space {
    eck_problem pb;
    eck::SpaceParams prm;
    std::vector<uint16_t> tables; // [table_total][4]
    uint32_t table_n[eck::NAX];
    uint64_t size;                // 0 when it overflows
    unsigned char *d_blob = nullptr; // device copy [SpaceParams, padded to kDevHeader | tables], made on first use
    int device = -1;
};

struct eck_model {
    int32_t n_layers;
    int32_t widths[4];
    int32_t dtype;
    uint64_t n_params;
    uint64_t off_w[3], off_b[3]; // offsets of W_l and b_l in theta
    float *d_state = nullptr;    // [theta | m | v | t]  (3P+1 floats)
    void *d_packed = nullptr;    // weights in matrix-core fragment order; BF16: + bias/output vectors, fp32: in three parts
    uint64_t packed_bytes = 0;
    float *d_copies = nullptr;   // fp32 models whose refits run by a crew: the weights as its steps read them (behind d_packed)
    int device = -1;
};

namespace eck {
// What a scoring launch needs to reduce its scores to the least legal one per segment of seg_len candidates as well
struct MinArgs {
    const uint8_t *legal; // or NULL: all legal
    uint64_t seg_len;
    uint32_t *min_key;    // [n / seg_len], preset to 0xFFFFFFFF
    uint32_t tiles_per_seg; // bf16 kernel: seg_len / (candidates per tile) when that is whole (set by the launcher), else 0
};

// order-preserving key of a float: unsigned comparison of keys = comparison of the numbers
__device__ __forceinline__ uint32_t score_order_key(float x)
{
    const uint32_t u = __float_as_uint(x);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Block barrier that orders LDS traffic only, for kernels whose wavefronts exchange nothing but LDS data: loads of weights for a
// later phase stay on their way across it (__syncthreads() would wait for them).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Adam on a parameter (bias-corrected, no weight decay).  The corrections' divisions are worked out once a step: a division or
// square root is a dozen instructions, and three and one of them a parameter were most of what a weights phase does once its
// sums are there.
struct AdamScales {
    float m, v; // lr / (1 - beta1^t), 1 / sqrt(1 - beta2^t)
};
// of the step behind `done` ones (whole, any number a float holds) and step_in_call more: the powers by squaring (a dozen
// multiplications for two double-precision pow() of most of a microsecond; a few units in the last place of a double).  Of 2^32 steps
// and more, the powers of every beta below 1 that a float holds are nothing beside 1.
__device__ __forceinline__ AdamScales adam_scales(float lr, float beta1, float beta2, float done, int step_in_call)
{
    uint32_t t = (uint32_t)fmin((double)done + step_in_call + 1, 4294967295.0);
    double power1 = 1.0, power2 = 1.0, square1 = beta1, square2 = beta2;
    for (; t; t >>= 1) {
        if (t & 1) {
            power1 *= square1;
            power2 *= square2;
        }
        square1 *= square1;
        square2 *= square2;
    }
    return {(float)((double)lr / (1.0 - power1)), (float)(1.0 / sqrt(1.0 - power2))};
}
struct AdamNext {
    float w, m, v;
};
__device__ __forceinline__ AdamNext adam_next(float w, float m, float v, float g, float beta1, float beta2, float eps, AdamScales scales)
{
    m = beta1 * m + (1.0f - beta1) * g;
    v = beta2 * v + (1.0f - beta2) * g * g;
    return {w - m * scales.m / (sqrtf(v) * scales.v + eps), m, v};
}

// the same on parameter i of a state [theta | m | v | t] from its values as fetched earlier: writes all three, returns the new
// weight
__device__ __forceinline__ float adam_one(float *theta, uint64_t P, uint64_t i, float w, float m, float v, float g,
                                          float beta1, float beta2, float eps, AdamScales scales)
{
    const AdamNext next = adam_next(w, m, v, g, beta1, beta2, eps, scales);
    theta[P + i] = next.m;
    theta[2 * P + i] = next.v;
    theta[i] = next.w;
    return next.w;
}

// forward pass of an fp32 model (score_f32.hip); mn: also the minima, or NULL
int32_t score_f32(const eck_model *m, const float *feat, uint64_t ld, uint64_t n, float *out, const MinArgs *mn,
                  hipStream_t stream);
// What a refit's kernels pass on, device memory in the call's workspace
struct RefitScalars {
    float emax;
    uint32_t bad; // data error found in the labels: leave the model alone
    float snr, loss;
};
// The end of costmodel_update in one launch: the SNR of the predictions `pred` made on entry (NULL: already in *sc), the step
// count, the call's results, and the packed weights
int32_t refit_finish(eck_model *m, const float *pred, const float *y, uint64_t n_pairs, int32_t n_steps, const RefitScalars *sc,
                     float *snr_out, float *loss_out, hipStream_t stream);
// How many blocks may be members of a refit's crew (crew.h), and how many of them are taken on at once
struct CrewSize {
    unsigned candidates, at_once;
};
// Adam steps of a BF16 model in two launches per step, or all in one (refit.hip): the bytes it needs in costmodel_update's
// workspace, those of the minibatch's features apart, and the steps themselves (labels y and the data-error flag come from
// the caller's kernels; the last step's mean loss goes to *loss_scalar, device memory; features, ws: 256-byte aligned)
uint64_t refit_features_bytes(const eck_model *m, int minibatch);
uint64_t refit_workspace_bytes(const eck_model *m, int minibatch);
// (refit_begin: labels y from the measured energies, and the weights' copies that the steps multiply with)
int32_t refit_begin(const eck_model *m, const float *energy, uint64_t n_pairs, float *y, RefitScalars *sc, int32_t minibatch, void *ws,
                    hipStream_t st);
int32_t refit_steps(const eck_model *m, const void *feat, int32_t feat_dtype, uint64_t ld, const float *y, uint64_t n_pairs,
                    int32_t n_steps, int32_t minibatch, float lr, float beta1, float beta2, float eps,
                    const uint32_t *bad_flag, float *loss_scalar, void *features, void *ws, CrewSize crew, hipStream_t st);
// the same for fp32 models of any hidden widths and minibatches of any size (refit_f32.hip)
uint64_t refit_f32_workspace_bytes(const eck_model *m, int minibatch);
uint64_t refit_f32_copies_bytes(const eck_model *m); // of the weights, beside the model's state
int32_t refit_f32_begin(const eck_model *m, const float *energy, uint64_t n_pairs, float *y, RefitScalars *sc, int32_t n_steps,
                        int32_t minibatch, void *ws, hipStream_t st);
int32_t refit_f32_steps(const eck_model *m, const float *feat, uint64_t ld, const float *y, uint64_t n_pairs, int32_t n_steps,
                        int32_t minibatch, float lr, float beta1, float beta2, float eps, const uint32_t *bad_flag,
                        float *loss_scalar, void *ws, CrewSize crew, hipStream_t st);
// topk_select on a workspace of the caller's or of the library's; known_min: THRESHOLD mode with the least latency
// of every segment already known (device, one order key per segment), else NULL
int32_t topk_select_impl(const float *energy, const float *latency, const uint8_t *legal, uint64_t n, uint32_t n_segments,
                         uint32_t k, int32_t mode, float alpha, uint32_t m_latency, uint32_t *idx_out, float *energy_out,
                         uint32_t *count_out, void *ws, uint64_t ws_bytes, void *stream, const uint32_t *known_min);
} // namespace eck
