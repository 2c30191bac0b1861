// Dynamic cost-model update: SNR of the current predictions, then minibatch
// Adam on the weighted squared error of Eq. (1)  (Alg. 1: ModelUpdate, SNR;
// Sec. 6.4).  HIP, gfx950.
//
// The steps of fp32 models, and of BF16 models but for the smallest ragged
// minibatches, take two launches each or all run in one (refit_f32.hip,
// refit.hip).  Here are the labels, the SNR, and the steps of those minibatches,
// whose workspace has no room for the others' buffers (some of up to 139 rows that
// are no multiple of 64): a short chain of launches of one strided tile GEMM on the matrix cores (forward, the three
// weight-gradient products with the bias gradient folded in as an extra all-ones
// row, the two back-propagated deltas; bf16 operands, weights, activations and
// back-propagated deltas rounded as they are staged, fp32 accumulation), a
// row-local loss/delta kernel and an element-wise Adam kernel; the width-1
// products of the output layer stay in fp32.  All reductions have a fixed order,
// so a run is reproducible bit for bit.
#include <algorithm>
#include <cmath>

#include "crew.h"
#include "refit_labels.h"

using namespace eck;

namespace {

__device__ __forceinline__ float through_bf16(float x)
{
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7F800000u) == 0x7F800000u) return x;
    u += 0x7FFFu + ((u >> 16) & 1u);
    return __uint_as_float(u & 0xFFFF0000u);
}

struct GemmArgs {
    // C[m][n] = epilogue( sum_k A(m,k) * B(k,n) )
    const void *A;
    int a_is_bf16;      // A holds bf16 bits (feature matrix) instead of fp32
    int64_t sa_m, sa_k; // element strides
    int a_ones_row;     // A(m == a_ones_row, k) reads as 1 (bias-gradient row); -1 = none
    const float *B;
    int64_t sb_k, sb_n;
    float *C;
    int64_t ldc;
    int M, N, K;
    const float *bias; // added per column n, rounded to bf16, or NULL
    int relu;
    const float *mask; // same layout as C: result kept where mask > 0, else 0; or NULL
    int round_c; // pass the result through bf16
};

constexpr int TM = 64, TN = 64;

// The product on the matrix cores for BF16 models: both operands are rounded to bf16 while they
// are staged into LDS, accumulation is fp32 (v_mfma_f32_32x32x16_bf16).  64 x 64 output tile per block,
// one 32 x 32 quadrant per wavefront, 64-deep stages; the next stage's operands are already in
// flight (in registers) while the current one is multiplied.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
constexpr int MK = 64;      // stage depth
constexpr int MLD = MK + 8; // LDS row stride in bf16: 144 bytes keeps the 16-byte fragment reads conflict-free

__device__ __forceinline__ uint16_t to_bf16_bits(float x)
{
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7F800000u) == 0x7F800000u) return (uint16_t)(u >> 16);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// The reduction dimension is also split inside the block: KG groups of four wavefronts take every KG-th
// stage each (these products are latency-bound -- 64 blocks, 8 dependent stages), and their partial tiles
// are added through LDS in group order, so the result does not depend on scheduling.
constexpr int KG = 2;
constexpr size_t GEMM_MFMA_LDS = (size_t)KG * (TM + TN) * MLD * sizeof(uint16_t);
static_assert((KG - 1) * TM * TN * sizeof(float) <= GEMM_MFMA_LDS, "partial tiles reuse the operand buffers");

__global__ __launch_bounds__(256 * KG) void gemm_mfma_kernel(GemmArgs first, GemmArgs second)
{
    // blockIdx.z picks the problem; blocks outside that problem's tile grid leave before any barrier
    const GemmArgs g = blockIdx.z ? second : first;
    if ((int)blockIdx.x * TN >= g.N || (int)blockIdx.y * TM >= g.M) return;
    extern __shared__ __attribute__((aligned(16))) unsigned char gemm_lds[];
    const int group = threadIdx.x >> 8, tid = threadIdx.x & 255, lane = tid & 63, wave = tid >> 6;
    uint16_t *As = reinterpret_cast<uint16_t *>(gemm_lds) + (size_t)group * (TM + TN) * MLD; // [m][k]
    uint16_t *Bs = As + TM * MLD;                                                            // [n][k]
    const int h = lane >> 5, c = lane & 31;
    const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TN;
    const int wm = (wave >> 1) * 32, wn = (wave & 1) * 32; // quadrant of this wavefront
    const bool a_k_fast = g.sa_k == 1, b_k_fast = g.sb_k == 1;
    constexpr int PER = TM * MK / 256; // elements per thread per operand per stage

    // fetch() only loads: every address is clamped into the operand, nothing is decided on what arrives, so the
    // 2 * PER loads of a stage are in flight together (a value that is tested, or loaded under a condition, is
    // waited for on the spot).  stage() then zeroes what lies outside M, N, K, sets the row of ones, converts
    // and stores to the LDS.
    uint32_t ra[PER], rb[PER]; // raw bits as loaded
    int fetched_k0 = 0;
    const int last_a_row = g.a_ones_row == g.M - 1 ? g.M - 2 : g.M - 1; // last row of A that is in memory
    auto fetch = [&](int k0) {
        fetched_k0 = k0;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int e = tid + 256 * q;
            {
                const int m = a_k_fast ? e / MK : e % TM, k = a_k_fast ? e % MK : e / TM;
                const int gm = max(min(m0 + m, last_a_row), 0), gk = min(k0 + k, g.K - 1);
                const int64_t at = (int64_t)gm * g.sa_m + (int64_t)gk * g.sa_k;
                ra[q] = g.a_is_bf16 ? (uint32_t)reinterpret_cast<const uint16_t *>(g.A)[at]
                                    : reinterpret_cast<const uint32_t *>(g.A)[at];
            }
            {
                const int n = b_k_fast ? e / MK : e % TN, k = b_k_fast ? e % MK : e / TN;
                const int gn = min(n0 + n, g.N - 1), gk = min(k0 + k, g.K - 1);
                rb[q] = reinterpret_cast<const uint32_t *>(g.B)[(int64_t)gk * g.sb_k + (int64_t)gn * g.sb_n];
            }
        }
    };
    auto stage = [&]() {
        const int k0 = fetched_k0;
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            const int e = tid + 256 * q;
            const int m = a_k_fast ? e / MK : e % TM, ka = a_k_fast ? e % MK : e / TM;
            const int gm = m0 + m;
            float va = __uint_as_float(g.a_is_bf16 ? ra[q] << 16 : ra[q]);
            if (gm == g.a_ones_row) va = 1.0f;
            if (gm >= g.M || k0 + ka >= g.K) va = 0.0f;
            As[m * MLD + ka] = to_bf16_bits(va);
            const int n = b_k_fast ? e / MK : e % TN, kb = b_k_fast ? e % MK : e / TN;
            float vb = __uint_as_float(rb[q]);
            if (n0 + n >= g.N || k0 + kb >= g.K) vb = 0.0f;
            Bs[n * MLD + kb] = to_bf16_bits(vb);
        }
    };

    f32x16 acc;
#pragma unroll
    for (int j = 0; j < 16; ++j) acc[j] = 0.0f;
    // every group runs the same number of rounds (stages past K read as zero), so the barriers match
    const int n_stages = (g.K + MK - 1) / MK, rounds = (n_stages + KG - 1) / KG;
    fetch(group * MK);
    for (int r = 0; r < rounds; ++r) {
        stage();
        __syncthreads();
        if (r + 1 < rounds) fetch(((r + 1) * KG + group) * MK);
#pragma unroll
        for (int ks = 0; ks < MK / 16; ++ks) {
            const bf16x8 a = *reinterpret_cast<const bf16x8 *>(&As[(wm + c) * MLD + 16 * ks + 8 * h]);
            const bf16x8 b = *reinterpret_cast<const bf16x8 *>(&Bs[(wn + c) * MLD + 16 * ks + 8 * h]);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
        }
        __syncthreads();
    }
    // partial tiles of groups 1 .. KG-1 through LDS, added by group 0 in group order
    float *partial = reinterpret_cast<float *>(gemm_lds); // [KG-1][4 wavefronts][16][64 lanes]
    if (group > 0) {
#pragma unroll
        for (int q = 0; q < 16; ++q) partial[(((group - 1) * 4 + wave) * 16 + q) * 64 + lane] = acc[q];
    }
    __syncthreads();
    if (group > 0) return;
#pragma unroll
    for (int other = 0; other < KG - 1; ++other)
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[q] += partial[((other * 4 + wave) * 16 + q) * 64 + lane];
    // accumulator register q of lane (h, c): row 8*(q/4) + 4h + q%4, column c of the quadrant
#pragma unroll
    for (int q = 0; q < 16; ++q) {
        const int m = m0 + wm + 8 * (q >> 2) + 4 * h + (q & 3), n = n0 + wn + c;
        if (m >= g.M || n >= g.N) continue;
        float v = acc[q];
        if (g.bias) v += through_bf16(g.bias[n]);
        if (g.relu) v = fmaxf(v, 0.0f);
        const int64_t at = (int64_t)m * g.ldc + n;
        if (g.mask && !(g.mask[at] > 0.0f)) v = 0.0f;
        if (g.round_c) v = through_bf16(v);
        g.C[at] = v;
    }
}

__global__ __launch_bounds__(1024) void labels_kernel(const float *__restrict__ e, uint64_t n, float *__restrict__ y, RefitScalars *sc)
{
    make_labels(e, n, y, sc);
}

// SNR = sum y^2 / sum (pred - y)^2 over the whole buffer (one block)
__global__ __launch_bounds__(1024) void snr_kernel(const float *__restrict__ pred, const float *__restrict__ y, uint64_t n, RefitScalars *sc)
{
    const float snr = signal_to_noise(pred, y, n);
    if (threadIdx.x == 0 && !sc->bad) sc->snr = snr;
}

__global__ void adam_kernel(float *__restrict__ state, const float *__restrict__ grad, uint64_t P, int step_in_call,
                            float lr, float beta1, float beta2, float eps, const RefitScalars *sc)
{
    if (sc->bad) return;
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= P) return;
    // (the count itself is advanced once, after the last step)
    const AdamScales scales = adam_scales(lr, beta1, beta2, state[3 * P], step_in_call);
    (void)adam_one(state, P, i, state[i], state[P + i], state[2 * P + i], grad[i], beta1, beta2, eps, scales);
}

// Output layer, forward and backward, fused and row-local: one wavefront per minibatch row computes
//   pred = h2 . w3 + b3,  the row's Eq.-(1) loss term,  dy = 2 (pred - y) / (y * rows),
//   d2[row][j] = dy * w3[j] where h2[row][j] > 0.
// The dot product is a fixed-order tree (per-lane strided partial sums, then a butterfly).
__global__ __launch_bounds__(256) void output_layer_kernel(const float *__restrict__ h2, const float *__restrict__ theta_w3,
                                                           const float *__restrict__ theta_b3, int H2, int rows,
                                                           const float *__restrict__ y,
                                                           float *__restrict__ pred, float *__restrict__ dy,
                                                           float *__restrict__ loss_terms, float *__restrict__ d2)
{
    const int lane = threadIdx.x & 63, r = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (r >= rows) return;
    const float *row = h2 + (int64_t)r * H2;
    float part = 0.0f;
    for (int j = lane; j < H2; j += 64) {
        const float w = through_bf16(theta_w3[j]);
        part = fmaf(row[j], w, part);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) part += __shfl_xor(part, off);
    const float b3 = through_bf16(theta_b3[0]);
    const float p = part + b3, t = y[r], d = p - t;
    const float g = 2.0f * d / (t * (float)rows);
    if (lane == 0) {
        pred[r] = p;
        dy[r] = g;
        loss_terms[r] = d * d / t;
    }
    for (int j = lane; j < H2; j += 64) {
        const float w = through_bf16(theta_w3[j]);
        d2[(int64_t)r * H2 + j] = row[j] > 0.0f ? g * w : 0.0f;
    }
}

// [gW3 ; gb3] = [h2 ; 1]^T dy.  A block owns 64 columns; its 16 wavefronts each sum a contiguous
// range of rows (rows in order, loads batched eight at a time) and the 16 partial sums are added in
// wavefront order, so the result does not depend on scheduling.  Block 0 also reduces the loss terms
// (fixed order, double) when this is the step whose loss is reported.
__global__ __launch_bounds__(1024) void output_grad_kernel(const float *__restrict__ h2, const float *__restrict__ dy,
                                                           int H2, int rows, float *__restrict__ grad_w3b3,
                                                           const float *__restrict__ loss_terms, RefitScalars *sc, int is_last)
{
    __shared__ float partial[16][64];
    const int cg = threadIdx.x & 63, rg = threadIdx.x >> 6;
    const int j = blockIdx.x * 64 + cg;
    const int per = (rows + 15) / 16, r0 = rg * per, r1 = min(rows, r0 + per);
    float acc = 0.0f;
    if (j < H2) {
        int r = r0;
        for (; r + 8 <= r1; r += 8) {
            float v[8], d[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                v[u] = h2[(int64_t)(r + u) * H2 + j];
                d[u] = dy[r + u];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) acc = fmaf(v[u], d[u], acc);
        }
        for (; r < r1; ++r) acc = fmaf(h2[(int64_t)r * H2 + j], dy[r], acc);
    } else if (j == H2) {
        for (int r = r0; r < r1; ++r) acc += dy[r];
    }
    partial[rg][cg] = acc;
    __syncthreads();
    if (rg == 0 && j <= H2) {
        float total = partial[0][cg];
#pragma unroll
        for (int g = 1; g < 16; ++g) total += partial[g][cg];
        grad_w3b3[j] = total;
    }
    if (blockIdx.x == 0 && is_last) {
        __shared__ double scratch[1024];
        double sum = 0.0;
        for (int r = threadIdx.x; r < rows; r += 1024) sum += (double)loss_terms[r];
        sum = block_sum(sum, scratch);
        if (threadIdx.x == 0 && !sc->bad) sc->loss = (float)(sum / rows);
    }
}

struct UpdWs {
    uint64_t scalars, y, pred, h1, h2, dy, lterm, d2, d1, grad, refit, total;
};

UpdWs upd_layout(const eck_model *m, uint64_t n_pairs, int mb)
{
    auto align = [](uint64_t v) { return (v + 255) & ~255ull; };
    UpdWs w;
    uint64_t o = 0;
    w.scalars = o; o = align(o + sizeof(RefitScalars));
    w.y = o;       o = align(o + n_pairs * 4);
    w.pred = o;    o = align(o + n_pairs * 4);
    w.h1 = w.h2 = w.dy = w.lterm = w.d2 = w.d1 = w.grad = o;
    if (m->dtype == ECK_F32) { // its two-launch steps keep all their buffers themselves
        w.refit = o;
        w.total = o + refit_f32_workspace_bytes(m, mb);
        return w;
    }
    w.h1 = o;      o = align(o + (uint64_t)mb * m->widths[1] * 4);
    w.h2 = o;      o = align(o + (uint64_t)mb * m->widths[2] * 4);
    w.dy = o;      o = align(o + (uint64_t)mb * 4);
    w.lterm = o;   o = align(o + (uint64_t)mb * 4);
    w.d2 = o;      o = align(o + (uint64_t)mb * m->widths[2] * 4);
    w.d1 = o;      o = align(o + (uint64_t)mb * m->widths[1] * 4);
    w.grad = o;    o = align(o + m->n_params * 4);
    w.refit = o;   // refit.hip's steps of minibatches of 64s keep their own buffers behind the others
    if (mb % 64 == 0) o += refit_workspace_bytes(m, mb);
    w.total = o;
    return w;
}

struct RefitPlace {
    bool applies;
    uint64_t ws, features;
};

RefitPlace refit_place(const eck_model *m, const UpdWs &w, int mb)
{
    if (m->dtype != ECK_BF16) return {false, 0, 0};
    if (mb % 64 == 0) return {true, w.refit, w.h1};
    const uint64_t features = w.h1 + refit_workspace_bytes(m, mb);
    return {features + refit_features_bytes(m, mb) <= w.total, w.h1, features};
}

// One launch for one product, or for two products that do not depend on each other (grid.z = 2).
void launch_gemm(const GemmArgs &g, hipStream_t st, const GemmArgs *also = nullptr)
{
    const GemmArgs &h = also ? *also : g;
    const dim3 grid((std::max(g.N, h.N) + TN - 1) / TN, (std::max(g.M, h.M) + TM - 1) / TM, also ? 2 : 1);
    // set per call: the attribute belongs to the current device
    (void)hipFuncSetAttribute(reinterpret_cast<const void *>(gemm_mfma_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                              (int)GEMM_MFMA_LDS);
    hipLaunchKernelGGL(gemm_mfma_kernel, grid, dim3(256 * KG), GEMM_MFMA_LDS, st, g, h);
}

} // namespace

extern "C" uint64_t costmodel_update_workspace_bytes(const eck_model *m, uint64_t n_pairs, int32_t minibatch)
{
    if (!m || n_pairs == 0 || minibatch <= 0) return 0;
    return upd_layout(m, n_pairs, minibatch).total;
}

// costmodel_update, its steps by a crew of at most `candidates` blocks, `at_once` of them taken on at a time, where one takes them.
// What a busy chip does to a crew, for the tests: not part of the interface.
extern "C" int32_t eck_update_by_crew(eck_model *m, const void *feat, int32_t feat_dtype, uint64_t ld, const float *energy_measured,
                                      uint64_t n_pairs, int32_t n_steps, int32_t minibatch, float lr, float beta1, float beta2,
                                      float eps, float *snr_out, float *loss_out, void *ws, uint64_t ws_bytes, uint32_t candidates,
                                      uint32_t at_once, void *stream)
{
    if (candidates < 1 || candidates > CREW_MOST || at_once < 1 || at_once > CREW_MOST) return ECK_EINVAL;
    const CrewSize crew = {candidates, at_once};
    if (!m || !feat || !energy_measured || !snr_out || !loss_out) return ECK_EINVAL;
    if (n_pairs == 0 || minibatch <= 0 || n_steps < 0 || n_pairs > (1u << 30)) return ECK_EINVAL;
    if (feat_dtype != ECK_F32 && feat_dtype != ECK_BF16) return ECK_EINVAL;
    if (!(lr > 0.0f) || !(beta1 >= 0.0f && beta1 < 1.0f) || !(beta2 >= 0.0f && beta2 < 1.0f) || !(eps >= 0.0f))
        return ECK_EINVAL;
    if (n_pairs % (uint64_t)minibatch || ld < n_pairs) return ECK_ESHAPE;
    if (m->dtype == ECK_F32 && feat_dtype != ECK_F32) return ECK_EUNSUPPORTED;
    const UpdWs w = upd_layout(m, n_pairs, minibatch);
    if (!ws || ws_bytes < w.total) return ECK_EWORKSPACE;
    if ((uintptr_t)ws & 255) return ECK_EALIGN;

    hipStream_t st = as_stream(stream);
    char *base = static_cast<char *>(ws);
    RefitScalars *sc = reinterpret_cast<RefitScalars *>(base + w.scalars);
    float *y = reinterpret_cast<float *>(base + w.y), *pred = reinterpret_cast<float *>(base + w.pred);
    float *h1 = reinterpret_cast<float *>(base + w.h1), *h2 = reinterpret_cast<float *>(base + w.h2);
    float *dy = reinterpret_cast<float *>(base + w.dy), *d2 = reinterpret_cast<float *>(base + w.d2);
    float *lterm = reinterpret_cast<float *>(base + w.lterm);
    float *d1 = reinterpret_cast<float *>(base + w.d1), *grad = reinterpret_cast<float *>(base + w.grad);
    const int F = m->widths[0], H1 = m->widths[1], H2 = m->widths[2], B = minibatch;
    const uint64_t P = m->n_params;
    float *theta = m->d_state;
    const int elem = feat_dtype == ECK_BF16 ? 2 : 4;

    // Steps by refit.hip: minibatches of 64s have a place for its buffers, the features' where a launch-per-product step would
    // keep the first layer; others where all that such a step keeps is enough, all from 80 rows of 256 units or 140 of 64 on.  8 steps
    // of 250 rows (replayed graphs), product by product and so: 64-256-256 553 and 108.7 us, 32-64-64 460 and 67.0.
    const RefitPlace place = refit_place(m, w, minibatch);
    const bool two_launches = place.applies;
    int32_t rc = ECK_OK;
    if (two_launches) rc = refit_begin(m, energy_measured, n_pairs, y, sc, minibatch, base + place.ws, st);
    else if (m->dtype == ECK_F32) rc = refit_f32_begin(m, energy_measured, n_pairs, y, sc, n_steps, minibatch, base + w.refit, st);
    else hipLaunchKernelGGL(labels_kernel, dim3(1), dim3(1024), 0, st, energy_measured, n_pairs, y, sc);
    if (rc != ECK_OK) return rc;
    // predictions of the model as it stands: the same forward pass that scores candidates
    rc = costmodel_score(m, feat, feat_dtype, ld, n_pairs, pred, nullptr, 0, stream);
    if (rc != ECK_OK) return rc;
    if (two_launches || m->dtype == ECK_F32) {
        rc = two_launches ? refit_steps(m, feat, feat_dtype, ld, y, n_pairs, n_steps, minibatch, lr, beta1, beta2, eps, &sc->bad,
                                        &sc->loss, base + place.features, base + place.ws, crew, st)
                          : refit_f32_steps(m, static_cast<const float *>(feat), ld, y, n_pairs, n_steps, minibatch, lr, beta1, beta2,
                                            eps, &sc->bad, &sc->loss, base + w.refit, crew, st);
        if (rc != ECK_OK) return rc;
        return refit_finish(m, pred, y, n_pairs, n_steps, sc, snr_out, loss_out, st);
    }
    hipLaunchKernelGGL(snr_kernel, dim3(1), dim3(1024), 0, st, pred, y, n_pairs, sc); // (the steps reuse pred)
    const uint64_t nb = n_pairs / (uint64_t)B;
    for (int s = 0; s < n_steps; ++s) {
        const uint64_t row0 = ((uint64_t)s % nb) * (uint64_t)B;
        const void *x = static_cast<const char *>(feat) + row0 * elem; // X(r, f) = feat[f*ld + row0 + r]
        GemmArgs g;
        // h1 = relu(X W1 + b1)
        g = GemmArgs{x, elem == 2, 1, (int64_t)ld, -1, theta + m->off_w[0], H1, 1, h1, H1, B, H1, F,
                     theta + m->off_b[0], 1, nullptr, 1};
        launch_gemm(g, st);
        // h2 = relu(h1 W2 + b2)
        g = GemmArgs{h1, 0, H1, 1, -1, theta + m->off_w[1], H2, 1, h2, H2, B, H2, H1,
                     theta + m->off_b[1], 1, nullptr, 0};
        launch_gemm(g, st);
        // output layer forward + loss + backward into d2, then its weight gradient
        hipLaunchKernelGGL(output_layer_kernel, dim3((B + 3) / 4), dim3(256), 0, st, h2, theta + m->off_w[2],
                           theta + m->off_b[2], H2, B, y + row0, pred, dy, lterm, d2);
        hipLaunchKernelGGL(output_grad_kernel, dim3((H2 + 1 + 63) / 64), dim3(1024), 0, st, h2, dy, H2, B,
                           grad + m->off_w[2], lterm, sc, s == n_steps - 1);
        // [gW2 ; gb2] = [h1 ; 1]^T d2
        g = GemmArgs{h1, 0, 1, H1, H1, d2, H2, 1, grad + m->off_w[1], H2, H1 + 1, H2, B, nullptr, 0, nullptr, 0};
        // d1 = (d2 W2^T) where h1 > 0: needs d2 only, like the product above, so both go in one launch
        const GemmArgs back{d2, 0, H2, 1, -1, theta + m->off_w[1], 1, H2, d1, H1, B, H1, H2, nullptr, 0, h1, 0};
        launch_gemm(g, st, &back);
        // [gW1 ; gb1] = [X ; 1]^T d1
        g = GemmArgs{x, elem == 2, (int64_t)ld, 1, F, d1, H1, 1, grad + m->off_w[0], H1, F + 1, H1, B, nullptr, 0, nullptr, 0};
        launch_gemm(g, st);
        hipLaunchKernelGGL(adam_kernel, dim3((unsigned)((P + 255) / 256)), dim3(256), 0, st, theta, grad, P, s, lr, beta1,
                           beta2, eps, sc);
    }
    ECK_HIP_TRY(hipGetLastError());
    return refit_finish(m, nullptr, y, n_pairs, n_steps, sc, snr_out, loss_out, st);
}

extern "C" int32_t costmodel_update(eck_model *m, const void *feat, int32_t feat_dtype, uint64_t ld,
                                    const float *energy_measured, uint64_t n_pairs, int32_t n_steps, int32_t minibatch,
                                    float lr, float beta1, float beta2, float eps, float *snr_out, float *loss_out,
                                    void *ws, uint64_t ws_bytes, void *stream)
{
    return eck_update_by_crew(m, feat, feat_dtype, ld, energy_measured, n_pairs, n_steps, minibatch, lr, beta1, beta2, eps, snr_out, loss_out,
                              ws, ws_bytes, CREW_MOST, CREW_MOST, stream);
}

extern "C" int32_t eck_k_count(double k, int64_t M, int64_t *count_out)
{
    if (!count_out || M < 0 || !(k >= 0.0 && k <= 1.0)) return ECK_EINVAL;
    *count_out = (int64_t)__builtin_floor(k * (double)M + 0.5);
    return ECK_OK;
}

extern "C" int32_t eck_k_step(double k, double snr, double mu, int64_t M, double *k_out)
{
    if (!k_out || M < 0 || !(k >= 0.0 && k <= 1.0) || mu != mu) return ECK_EINVAL;
    const int64_t measured = (int64_t)__builtin_floor(k * (double)M + 0.5);
    if (measured == 0) {
        *k_out = k;
        return ECK_OK;
    }
    // a NaN ratio (rejected energies) counts as a poor model: measure more
    const bool poor = !(snr >= mu);
    const double next = poor ? k + 0.2 : k - 0.2;
    *k_out = next > 1.0 ? 1.0 : (next < 0.0 ? 0.0 : next);
    return ECK_OK;
}
