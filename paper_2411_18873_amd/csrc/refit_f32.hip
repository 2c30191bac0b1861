// Minibatch Adam steps on the weighted squared error of Eq. (1) for fp32 models of any hidden widths, two launches per
// step (Alg. 1: ModelUpdate; Sec. 6.4).  HIP, gfx950.
//
// The same cut as for BF16 models, with fp32 operands throughout (v_mfma_f32_16x16x4_f32, tiles of f32_tiles.h):
//   rows kernel:     both hidden layers, the output layer, the Eq.-(1) term and its derivative and the deltas of both
//                    hidden layers for 16 minibatch rows per block;
//   weights kernel:  the weight and bias gradients, summed over the minibatch, and the Adam update of each parameter in
//                    the block that completes its gradient.
// A step is a chain of dependent products too small to fill the chip, so it is bound by launches and by the latency of
// each product's loads: weights are requested before the barrier or the product that precedes theirs, several groups of
// sixteen rows of the reduction at a time.  Every sum has a fixed order.
// Measured, 64-128-128-1 on minibatches of 250: 136 us per step launched one product at a time (a vector kernel of two
// blocks for most of them, 30 us each), 15 us in two launches (a block of its own for the bias corrections took 0.85 us a
// step off the rows kernel; the features requested first and the biases' moments with the tile's, 0.6); 64-512-512-1,
// 512 rows: 290 and 70.
#include "f32_tiles.h"

using namespace eck;
using namespace eck::f32;

namespace {

constexpr int ROWS = 16;  // minibatch rows per block of the rows kernel
constexpr int WAVES = 8;  // wavefronts per block, at most (rows kernel), exactly (weights kernel)
constexpr int TILE = 32;  // a block of the weights kernel owns TILE x TILE parameters

struct StepF32 {
    const float *feat; // [F][ld], minibatch row r = column row0 + r
    uint64_t ld, row0;
    int rows, padded;  // minibatch size, and the same rounded up to ROWS
    float *theta;      // [theta | m | v | t], n_params = P
    uint64_t P;
    int F, H1, H2;
    uint64_t off_w1, off_b1, off_w2, off_b2, off_w3, off_b3;
    const float *y;    // labels of the whole buffer
    // what the gradients sum over the minibatch, [padded][width], rows past the minibatch zero
    float *x, *h1, *h2, *d1, *d2, *dy;
    float *lterm;      // [padded] Eq.-(1) terms of the rows
    const uint32_t *bad; // data error found in the labels: leave the model alone
    float *loss_out;   // mean of the Eq.-(1) terms, written in the step with report_loss set
    AdamScales *scales; // of the step (rows kernel -> weights kernel)
    int step_in_call, report_loss;
    float lr, beta1, beta2, eps;
};

// A slice of the way back through a layer: rows = the layer's inputs, reduction = its outputs, so a lane's four steps of
// a group are neighbours in a row of W.  Rows past K re-read the last one and are never used.
template <int J>
struct BackSlice {
    const F32Layer &l;
    int p;
    __amdgpu_buffer_rsrc_t weights;
    uint32_t lane_bytes[J];
    int input[J];

    __device__ BackSlice(const F32Layer &layer, int first, int p_, int c) : l(layer), p(p_)
    {
        weights = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(l.w), 0, l.K * l.H * 4, RSRC_FLAGS);
#pragma unroll
        for (int j = 0; j < J; ++j) {
            input[j] = min(first + J * c + j, l.K - 1);
            lane_bytes[j] = 4u * (uint32_t)(input[j] * l.H + 4 * p);
        }
    }

    __device__ __forceinline__ void group(int g, float (&a)[4][J]) const
    {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const i32x4 f = __builtin_amdgcn_raw_buffer_load_b128(weights, lane_bytes[j], 64 * g, 0);
#pragma unroll
            for (int t = 0; t < 4; ++t) a[t][j] = __int_as_float(f[t]);
        }
    }

    __device__ __forceinline__ void partial_group(int g, float (&a)[4][J]) const
    {
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int k = 16 * g + 4 * p + t;
                const float v = l.w[(int64_t)input[j] * l.H + min(k, l.H - 1)];
                a[t][j] = k < l.H ? v : 0.0f;
            }
    }
};

template <int J>
struct ForwardSlice : Slice<J> {
    using Slice<J>::Slice;
    __device__ __forceinline__ void group(int g, float (&a)[4][J]) const
    {
#pragma unroll
        for (int t = 0; t < 4; ++t) this->row(g, t, a[t]);
    }
};

// The first DEPTH groups of a product's weights, requested ahead (past the end: the last whole group again)
template <int J, int DEPTH, class S>
__device__ __forceinline__ void request(const S &slice, int K, float (&a)[DEPTH][4][J])
{
    const int last = K / 16 - 1;
    if (last < 0) return;
#pragma unroll
    for (int i = 0; i < DEPTH; ++i) slice.group(min(i, last), a[i]);
}

// acc[j] += weights * activations over K, for one tile of 16 columns: DEPTH groups of weights under way at any time
template <int J, int DEPTH, class S>
__device__ __forceinline__ void product(const S &slice, int K, const f32x4 *act, int p, int c, float (&a)[DEPTH][4][J],
                                        f32x4 (&acc)[J])
{
    const int whole = K / 16, last = whole - 1;
    const f32x4 *from = act + p * ROWS + c;
    auto steps = [&](const float (&w)[4][J], const f32x4 &b) {
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int j = 0; j < J; ++j) acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[t][j], b[t], acc[j], 0, 0, 0);
    };
    int g = 0;
    for (; g + DEPTH < whole; g += DEPTH) { // (no branch inside: at one the compiler copies the accumulators)
        f32x4 b[DEPTH];
#pragma unroll
        for (int i = 0; i < DEPTH; ++i) b[i] = from[4 * (g + i) * ROWS];
#pragma unroll
        for (int i = 0; i < DEPTH; ++i) {
            steps(a[i], b[i]);
            slice.group(min(g + DEPTH + i, last), a[i]);
        }
    }
#pragma unroll
    for (int i = 0; i < DEPTH; ++i)
        if (g + i < whole) steps(a[i], from[4 * (g + i) * ROWS]);
    if (K % 16) {
        slice.partial_group(whole, a[0]);
        steps(a[0], from[4 * whole * ROWS]);
    }
}

// ------------------------------------------------------------------------------------------------ rows kernel

// 4 J consecutive units of one minibatch row, unit0 a multiple of four, to a row-major matrix of `width` columns
template <int J>
__device__ __forceinline__ void store_units(float *row, int unit0, int width, const float (&v)[4 * J])
{
    if (width % 4 == 0) {
#pragma unroll
        for (int m = 0; m < J; ++m)
            if (unit0 + 4 * m < width)
                *reinterpret_cast<f32x4 *>(row + unit0 + 4 * m) = f32x4{v[4 * m], v[4 * m + 1], v[4 * m + 2], v[4 * m + 3]};
    } else {
#pragma unroll
        for (int e = 0; e < 4 * J; ++e)
            if (unit0 + e < width) row[unit0 + e] = v[e];
    }
}

// One block = 16 minibatch rows, and one more block for Adam's bias corrections; wavefront w owns units 16 J w .. of both
// hidden layers, J tiles (one or two up to 256 units, so that the products of a layer are spread over as many wavefronts
// as there are).
template <int J>
__global__ __launch_bounds__(64 * WAVES, 2) void step_rows_f32_kernel(StepF32 a)
{
    constexpr int DEPTH = J <= 2 ? 8 : 4, E = 4 * J;
    if (blockIdx.x == gridDim.x - 1) { // the block of Adam's bias corrections
        // (t itself is advanced once, after the last step)
        if (threadIdx.x == 0) *a.scales = adam_scales(a.lr, a.beta1, a.beta2, (uint32_t)a.theta[3 * a.P] + a.step_in_call + 1);
        return;
    }
    extern __shared__ __attribute__((aligned(16))) unsigned char rows_lds[];
    const int F = a.F, H1 = a.H1, H2 = a.H2, r1 = (H1 + 15) / 16 * 4, r2 = (H2 + 15) / 16 * 4;
    f32x4 *x_l = reinterpret_cast<f32x4 *>(rows_lds); // [F / 4][ROWS]
    f32x4 *h1_l = x_l + F / 4 * ROWS;                  // [r1][ROWS]
    f32x4 *d2_l = h1_l + r1 * ROWS;                    // [r2][ROWS]
    float *part_l = reinterpret_cast<float *>(d2_l + r2 * ROWS); // [WAVES][ROWS]
    float *dy_l = part_l + WAVES * ROWS;                         // [ROWS]
    const int tid = threadIdx.x, lane = tid & 63, p = lane >> 4, c = lane & 15, threads = blockDim.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int first = 16 * J * wave, unit0 = first + E * p; // this lane's units: unit0 .. unit0 + E - 1
    const bool has1 = first < H1, has2 = first < H2;
    const int r0 = blockIdx.x * ROWS;
    const bool valid = r0 + c < a.rows;

    const F32Layer l1{a.theta + a.off_w1, a.theta + a.off_b1, F, H1}, l2{a.theta + a.off_w2, a.theta + a.off_b2, H1, H2};
    const ForwardSlice<J> s1(l1, first, p, c), s2(l2, first, p, c);
    const BackSlice<J> back(l2, first, p, c);
    // Everything the first two layers need is requested before anything is waited for, the features, which are needed first, in
    // front
    auto features = [&](int e) {
        const int row = e % ROWS, four = e / ROWS;
        const uint64_t col = a.row0 + min(r0 + row, a.rows - 1);
        f32x4 v;
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = a.feat[(uint64_t)(4 * four + t) * a.ld + col];
        return v;
    };
    auto keep = [&](int e, f32x4 v) {
        const int row = e % ROWS, four = e / ROWS;
        if (r0 + row >= a.rows) v = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        x_l[e] = v;
        *reinterpret_cast<f32x4 *>(a.x + (int64_t)(r0 + row) * F + 4 * four) = v;
    };
    const int items = F / 4 * ROWS;
    const f32x4 first_features = features(min(tid, items - 1));
    float b1[E], b2[E], w3[E], w1f[DEPTH][4][J], w2f[DEPTH][4][J];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        b1[e] = l1.b[min(unit0 + e, H1 - 1)];
        b2[e] = l2.b[min(unit0 + e, H2 - 1)];
        w3[e] = a.theta[a.off_w3 + min(unit0 + e, H2 - 1)];
    }
    float target = a.y[a.row0 + min(r0 + c, a.rows - 1)], bias3 = a.theta[a.off_b3];
    if (has1) request<J, DEPTH>(s1, F, w1f);
    if (has2) request<J, DEPTH>(s2, H1, w2f);
    __builtin_amdgcn_sched_barrier(0);
    if (tid < items) keep(tid, first_features);
    for (int e = tid + threads; e < items; e += threads) keep(e, features(e));
    lds_barrier();
    asm volatile("" : "+v"(target), "+v"(bias3)); // (there by now; left to their use, they wait for all later loads, too)

    // ---- h1 = relu(x W1 + b1)
    float h1[E];
    if (has1) {
        f32x4 acc[J];
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e % J][e / J] = b1[e];
        product<J, DEPTH>(s1, F, x_l, p, c, w1f, acc);
#pragma unroll
        for (int e = 0; e < E; ++e) h1[e] = valid && unit0 + e < H1 ? fmaxf(acc[e % J][e / J], 0.0f) : 0.0f;
#pragma unroll
        for (int m = 0; m < J; ++m)
            if (unit0 / 4 + m < r1) h1_l[(unit0 / 4 + m) * ROWS + c] = f32x4{h1[4 * m], h1[4 * m + 1], h1[4 * m + 2], h1[4 * m + 3]};
        store_units<J>(a.h1 + (int64_t)(r0 + c) * H1, unit0, H1, h1);
    }
    lds_barrier();

    // ---- h2 = relu(h1 W2 + b2), this wavefront's part of the output layer
    float h2[E], y = 0.0f;
    if (has2) {
        f32x4 acc[J];
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e % J][e / J] = b2[e];
        product<J, DEPTH>(s2, H1, h1_l, p, c, w2f, acc);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            h2[e] = valid && unit0 + e < H2 ? fmaxf(acc[e % J][e / J], 0.0f) : 0.0f;
            y = unit0 + e < H2 ? fmaf(h2[e], w3[e], y) : y;
        }
        store_units<J>(a.h2 + (int64_t)(r0 + c) * H2, unit0, H2, h2);
    }
    // W2 for the way back is under way while the output layer is summed
    if (has1) request<J, DEPTH>(back, H2, w1f);
    y += __shfl_xor(y, 16);
    y += __shfl_xor(y, 32);
    if (p == 0) part_l[wave * ROWS + c] = y;
    lds_barrier();
    if (tid < ROWS) {
        float pred = bias3;
        for (int w = 0; w < threads / 64; ++w) pred += part_l[w * ROWS + tid];
        const float d = pred - target;
        const float g = r0 + tid < a.rows ? 2.0f * d / (target * (float)a.rows) : 0.0f;
        a.dy[r0 + tid] = g;
        a.lterm[r0 + tid] = r0 + tid < a.rows ? d * d / target : 0.0f;
        dy_l[tid] = g;
    }
    lds_barrier();

    // ---- d2 = dy w3 where h2 > 0
    if (has2) {
        const float g = dy_l[c];
        float d2[E];
#pragma unroll
        for (int e = 0; e < E; ++e) d2[e] = h2[e] > 0.0f ? g * w3[e] : 0.0f; // (zero past H2 and past the minibatch)
#pragma unroll
        for (int m = 0; m < J; ++m)
            if (unit0 / 4 + m < r2) d2_l[(unit0 / 4 + m) * ROWS + c] = f32x4{d2[4 * m], d2[4 * m + 1], d2[4 * m + 2], d2[4 * m + 3]};
        store_units<J>(a.d2 + (int64_t)(r0 + c) * H2, unit0, H2, d2);
    }
    lds_barrier();

    // ---- d1 = (d2 W2^T) where h1 > 0
    if (has1) {
        f32x4 acc[J];
#pragma unroll
        for (int j = 0; j < J; ++j) acc[j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        product<J, DEPTH>(back, H2, d2_l, p, c, w1f, acc);
        float d1[E];
#pragma unroll
        for (int e = 0; e < E; ++e) d1[e] = h1[e] > 0.0f ? acc[e % J][e / J] : 0.0f;
        store_units<J>(a.d1 + (int64_t)(r0 + c) * H1, unit0, H1, d1);
    }
}

// --------------------------------------------------------------------------------------------- weights kernel

struct Moments {
    float w, m, v;
};

__device__ __forceinline__ Moments load_moments(const StepF32 &a, uint64_t i) { return {a.theta[i], a.theta[a.P + i], a.theta[2 * a.P + i]}; }

__device__ __forceinline__ void adam_one(const StepF32 &a, uint64_t i, Moments s, float g, AdamScales scales)
{
    (void)eck::adam_one(a.theta, a.P, i, s.w, s.m, s.v, g, a.beta1, a.beta2, a.eps, scales);
}

// Blocks, in order: the 32 x 32 tiles of W2, those of W1, then blocks of 16 columns of the output layer.  A tile block:
// G[m][n] = sum_r A[r][m] D[r][n], both row-major over the minibatch rows (A = h1 or x, D = d2 or d1); as two by two
// interleaved matrix-core tiles, so that one 8-byte load per lane and row serves two.  Wavefront w takes every eighth group
// of sixteen rows; the eight partial tiles are added in wavefront order through LDS and every thread updates two
// parameters.  Columns past a matrix's width read what follows (the buffers are padded for it) and are never used.
// The blocks of the first tile row also sum the columns of D: the bias gradient.
__global__ __launch_bounds__(64 * WAVES) void step_weights_f32_kernel(StepF32 a, int blocks2, int blocks1)
{
    __shared__ float part[WAVES][TILE][TILE];
    __shared__ float colsum[WAVES][TILE];
    __shared__ double lsum[64 * WAVES];
    const int tid = threadIdx.x, lane = tid & 63, p = lane >> 4, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool bad = *a.bad != 0;
    const AdamScales scales = *a.scales;
    int block = blockIdx.x;
    if (block < blocks2 + blocks1) {
        const bool second = block < blocks2; // a tile of W2, else of W1
        if (!second) block -= blocks2;
        const int M = second ? a.H1 : a.F, N = second ? a.H2 : a.H1;
        const float *A = second ? a.h1 : a.x, *D = second ? a.d2 : a.d1;
        const uint64_t off_w = second ? a.off_w2 : a.off_w1, off_b = second ? a.off_b2 : a.off_b1;
        const int nt = (N + TILE - 1) / TILE, m0 = block / nt * TILE, n0 = block % nt * TILE;
        // the two parameters this thread updates
        constexpr int PER = TILE * TILE / (64 * WAVES);
        Moments state[PER];
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const int m = m0 + tid / TILE + e * (TILE / PER), n = n0 + tid % TILE;
            state[e] = load_moments(a, off_w + (uint64_t)min(m, M - 1) * N + min(n, N - 1));
        }
        // ... and the bias, in the first tile row
        const uint64_t bias_at = off_b + min(n0 + tid % TILE, N - 1);
        Moments bias_state = {0.0f, 0.0f, 0.0f};
        if (m0 == 0) bias_state = load_moments(a, bias_at);
        const uint32_t a_lane = 4u * (uint32_t)(4 * p * M + m0 + 2 * c), d_lane = 4u * (uint32_t)(4 * p * N + n0 + 2 * c);
        f32x4 acc[2][2];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
        float bsum[2] = {0.0f, 0.0f};
        const int groups = a.padded / 16;
        constexpr int BATCH = 4; // groups requested together
        for (int g0 = wave; g0 < groups; g0 += BATCH * WAVES) {
            i32x2 av[BATCH][4], dv[BATCH][4];
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                const int g = g0 + u * WAVES;
                if (g >= groups) break;
                const __amdgpu_buffer_rsrc_t ar = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(A + (int64_t)16 * g * M), 0, (16 * M + TILE) * 4, RSRC_FLAGS);
                const __amdgpu_buffer_rsrc_t dr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(D + (int64_t)16 * g * N), 0, (16 * N + TILE) * 4, RSRC_FLAGS);
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    av[u][t] = __builtin_amdgcn_raw_buffer_load_b64(ar, a_lane, t * M * 4, 0);
                    dv[u][t] = __builtin_amdgcn_raw_buffer_load_b64(dr, d_lane, t * N * 4, 0);
                }
            }
#pragma unroll
            for (int u = 0; u < BATCH; ++u) {
                if (g0 + u * WAVES >= groups) break;
#pragma unroll
                for (int t = 0; t < 4; ++t) {
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(__int_as_float(av[u][t][i]), __int_as_float(dv[u][t][j]),
                                                                            acc[i][j], 0, 0, 0);
#pragma unroll
                    for (int j = 0; j < 2; ++j) bsum[j] += __int_as_float(dv[u][t][j]);
                }
            }
        }
        // tile (i, j), quarter p, register q: row 2 (4p + q) + i, column 2c + j
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<float2 *>(&part[wave][2 * (4 * p + q) + i][2 * c]) = make_float2(acc[i][0][q], acc[i][1][q]);
        if (m0 == 0) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                bsum[j] += __shfl_xor(bsum[j], 16);
                bsum[j] += __shfl_xor(bsum[j], 32);
                if (p == 0) colsum[wave][2 * c + j] = bsum[j];
            }
        }
        lds_barrier();
        if (bad) return;
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const int lm = tid / TILE + e * (TILE / PER), ln = tid % TILE;
            float g = part[0][lm][ln];
#pragma unroll
            for (int w = 1; w < WAVES; ++w) g += part[w][lm][ln];
            if (m0 + lm < M && n0 + ln < N) adam_one(a, off_w + (uint64_t)(m0 + lm) * N + n0 + ln, state[e], g, scales);
        }
        if (m0 == 0 && tid < TILE && n0 + tid < N) {
            float g = colsum[0][tid];
#pragma unroll
            for (int w = 1; w < WAVES; ++w) g += colsum[w][tid];
            adam_one(a, bias_at, bias_state, g, scales);
        }
        return;
    }
    // ---- output layer: [gW3 ; gb3] = [h2 ; 1]^T dy, 16 columns per block, 32 row groups summed in order
    block -= blocks2 + blocks1;
    float *psum = &part[0][0][0]; // [32 row groups][16 columns]
    constexpr int RG = 64 * WAVES / 16;
    const int cg = tid & 15, rg = tid >> 4, col = block * 16 + cg;
    const int per = (a.padded + RG - 1) / RG, rlo = rg * per, rhi = min(rlo + per, a.padded);
    float sum = 0.0f;
    const uint64_t i_out = col < a.H2 ? a.off_w3 + col : a.off_b3;
    const Moments out_state = load_moments(a, i_out);
    if (col < a.H2) {
        int r = rlo;
        for (; r + 8 <= rhi; r += 8) {
            float v[8], d[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                v[u] = a.h2[(int64_t)(r + u) * a.H2 + col];
                d[u] = a.dy[r + u];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) sum = fmaf(v[u], d[u], sum);
        }
        for (; r < rhi; ++r) sum = fmaf(a.h2[(int64_t)r * a.H2 + col], a.dy[r], sum);
    } else if (col == a.H2) {
        for (int r = rlo; r < rhi; ++r) sum += a.dy[r];
    }
    psum[rg * 16 + cg] = sum;
    const bool report = block == 0 && a.report_loss;
    if (report) {
        double s = 0.0;
        for (int r = tid; r < a.rows; r += 64 * WAVES) s += (double)a.lterm[r];
        lsum[tid] = s;
    }
    __syncthreads();
    if (report) {
        for (int off = 32 * WAVES; off > 0; off >>= 1) {
            if (tid < off) lsum[tid] += lsum[tid + off];
            __syncthreads();
        }
        if (tid == 0 && !bad) *a.loss_out = (float)(lsum[0] / a.rows);
    }
    if (bad) return;
    if (tid < 16 && col <= a.H2) {
        float g = psum[cg];
#pragma unroll
        for (int r = 1; r < RG; ++r) g += psum[r * 16 + cg];
        adam_one(a, i_out, out_state, g, scales);
    }
}

// the buffers behind the others in costmodel_update's workspace; every matrix is padded by one tile width, because a
// weights kernel's lane may read that far past the last row
struct Buffers {
    uint64_t x, h1, h2, d1, d2, dy, lterm, scales, total;
};

Buffers buffers_for(const eck_model *m, int minibatch)
{
    auto align = [](uint64_t v) { return (v + 255) & ~255ull; };
    const uint64_t B = ((uint64_t)minibatch + ROWS - 1) / ROWS * ROWS, F = m->widths[0], H1 = m->widths[1], H2 = m->widths[2];
    Buffers w;
    uint64_t o = 0;
    auto take = [&](uint64_t floats) {
        const uint64_t at = o;
        o = align(o + (floats + TILE) * 4);
        return at;
    };
    w.x = take(B * F);
    w.h1 = take(B * H1);
    w.h2 = take(B * H2);
    w.d1 = take(B * H1);
    w.d2 = take(B * H2);
    w.dy = take(B);
    w.lterm = take(B);
    w.scales = take(2);
    w.total = o;
    return w;
}

} // namespace

uint64_t eck::refit_f32_workspace_bytes(const eck_model *m, int minibatch) { return buffers_for(m, minibatch).total; }

int32_t eck::refit_f32_steps(const eck_model *m, const float *feat, uint64_t ld, const float *y, uint64_t n_pairs,
                             int32_t n_steps, int32_t minibatch, float lr, float beta1, float beta2, float eps,
                             const uint32_t *bad_flag, float *loss_scalar, void *ws, hipStream_t st)
{
    const Buffers w = buffers_for(m, minibatch);
    char *base = static_cast<char *>(ws);
    StepF32 a = {};
    a.feat = feat;
    a.ld = ld;
    a.rows = minibatch;
    a.padded = (minibatch + ROWS - 1) / ROWS * ROWS;
    a.theta = m->d_state;
    a.P = m->n_params;
    a.F = m->widths[0];
    a.H1 = m->widths[1];
    a.H2 = m->widths[2];
    a.off_w1 = m->off_w[0];
    a.off_b1 = m->off_b[0];
    a.off_w2 = m->off_w[1];
    a.off_b2 = m->off_b[1];
    a.off_w3 = m->off_w[2];
    a.off_b3 = m->off_b[2];
    a.y = y;
    a.x = reinterpret_cast<float *>(base + w.x);
    a.h1 = reinterpret_cast<float *>(base + w.h1);
    a.h2 = reinterpret_cast<float *>(base + w.h2);
    a.d1 = reinterpret_cast<float *>(base + w.d1);
    a.d2 = reinterpret_cast<float *>(base + w.d2);
    a.dy = reinterpret_cast<float *>(base + w.dy);
    a.lterm = reinterpret_cast<float *>(base + w.lterm);
    a.scales = reinterpret_cast<AdamScales *>(base + w.scales);
    a.bad = bad_flag;
    a.loss_out = loss_scalar;
    a.lr = lr;
    a.beta1 = beta1;
    a.beta2 = beta2;
    a.eps = eps;
    // the fewest tiles per wavefront that eight wavefronts cover the wider layer with
    const int tiles = ((a.H1 > a.H2 ? a.H1 : a.H2) + 15) / 16, J = (tiles + WAVES - 1) / WAVES, waves = (tiles + J - 1) / J;
    auto rows_kernel = J == 1   ? step_rows_f32_kernel<1>
                       : J == 2 ? step_rows_f32_kernel<2>
                       : J == 3 ? step_rows_f32_kernel<3>
                                : step_rows_f32_kernel<4>;
    const size_t lds = (size_t)ROWS * 16 * (a.F / 4 + (a.H1 + 15) / 16 * 4 + (a.H2 + 15) / 16 * 4) + (WAVES + 1) * ROWS * 4;
    ECK_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(rows_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    auto over = [](int v) { return (v + TILE - 1) / TILE; };
    const int blocks2 = over(a.H1) * over(a.H2), blocks1 = over(a.F) * over(a.H1), out_blocks = (a.H2 + 1 + 15) / 16;
    const uint64_t nb = n_pairs / (uint64_t)minibatch;
    for (int s = 0; s < n_steps; ++s) {
        a.row0 = ((uint64_t)s % nb) * (uint64_t)minibatch;
        a.step_in_call = s;
        a.report_loss = s == n_steps - 1;
        hipLaunchKernelGGL(rows_kernel, dim3(a.padded / ROWS + 1), dim3(64 * waves), lds, st, a);
        hipLaunchKernelGGL(step_weights_f32_kernel, dim3(blocks2 + blocks1 + out_blocks), dim3(64 * WAVES), 0, st, a, blocks2, blocks1);
    }
    ECK_HIP_TRY(hipGetLastError());
    return ECK_OK;
}
