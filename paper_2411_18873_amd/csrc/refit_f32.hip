// Minibatch Adam steps on the weighted squared error of Eq. (1) for fp32 models of any hidden widths, two launches a
// step or, where a step is small enough for one die, all steps in one (Alg. 1: ModelUpdate; Sec. 6.4).  HIP, gfx950.
//
// The same cut as for BF16 models, with fp32 operands throughout (v_mfma_f32_16x16x4_f32, tiles of f32_tiles.h):
//   rows kernel:     both hidden layers, the output layer, the Eq.-(1) term and its derivative and the deltas of both
//                    hidden layers for 16 minibatch rows per block;
//   weights kernel:  the weight and bias gradients, summed over the minibatch, and the Adam update of each parameter in
//                    the block that completes its gradient.
// A step is a chain of dependent products too small to fill the chip, so it is bound by launches and by the latency of
// each product's loads: weights are requested before the barrier or the product that precedes theirs, several groups of
// sixteen rows of the reduction at a time.  Every sum has a fixed order, the same in both forms.
// Measured, 64-128-128-1, 16 steps of 250 rows, a whole call with the state in and out: 252.4 us with two launches a step
// (a block of its own for the bias corrections took 0.85 us a step off the rows kernel; the features requested first and
// the biases' moments with the tile's, 0.6), 195.7 by a crew (crew.h; 192.4 while its number of members was fixed at the start).  One product at a time: 136 us a step.
// 64-512-512-1, 512 rows, two launches: 70 us a step.
#include "crew.h"
#include "f32_tiles.h"
#include "refit_labels.h"

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
    // a crew's copies of the weights (CopySlice): x W1, h1 W2 and d2 W2^T
    float *w1t, *w2t, *w2;
};

// A weight matrix as the products of a crew read it: a tile's weights of a group, four steps a lane, are a contiguous kilobyte.
// n: what the lanes stand for (a unit, or on the way back a layer's input), k: the reduction's index, both padded with zeros to
// sixteens.  One tile a wavefront.
constexpr int CREW_J = 1;
__host__ __device__ inline int copy_groups(int k) { return (k + 15) / 16; }
__host__ __device__ inline uint32_t copy_at(int n, int k, int groups) { return (uint32_t)(((n / 16 * groups + k / 16) * 64 + 16 * (k % 16 / 4) + n % 16) * 4 + k % 4); }

struct CopySlice {
    __amdgpu_buffer_rsrc_t weights;
    uint32_t lane_bytes, first; // of this wavefront's tile

    __device__ CopySlice(const float *copy, int k, int wave, int lane) : weights(crew_buffer(copy)), lane_bytes(16u * lane)
    {
        first = 1024u * (uint32_t)(wave * copy_groups(k));
    }

    __device__ __forceinline__ void group(int g, float (&a)[4][1]) const
    {
        const i32x4 f = __builtin_amdgcn_raw_buffer_load_b128(weights, lane_bytes, first + 1024u * (uint32_t)g, CREW_SC1);
#pragma unroll
        for (int t = 0; t < 4; ++t) a[t][0] = __int_as_float(f[t]);
    }
    __device__ __forceinline__ void partial_group(int g, float (&a)[4][1]) const { group(g, a); } // (padded with zeros)
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
__device__ __forceinline__ void request(const S &slice, int K, float (&a)[DEPTH][4][J], int first = 0, int end = DEPTH)
{
    const int last = K / 16 - 1;
    if (last < 0) return;
#pragma unroll
    for (int i = 0; i < DEPTH; ++i)
        if (i >= first && i < end) slice.group(min(i, last), a[i]);
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

__device__ __forceinline__ AdamScales step_scales(const StepF32 &a, int step_in_call)
{
    return adam_scales(a.lr, a.beta1, a.beta2, a.theta[3 * a.P], step_in_call); // (the count itself is advanced once, after the last step)
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

// The features and labels of ROWS minibatch rows, r0 .. of the minibatch in columns `from` .. of the features: four neighbouring
// features of a row an item, and of the rows past the minibatch zeros.
__device__ __forceinline__ f32x4 row_features(const StepF32 &a, uint64_t row0, int r0, int e)
{
    const int row = e % ROWS, four = e / ROWS;
    const uint64_t col = row0 + min(r0 + row, a.rows - 1);
    f32x4 v;
#pragma unroll
    for (int t = 0; t < 4; ++t) v[t] = a.feat[(uint64_t)(4 * four + t) * a.ld + col];
    return r0 + row < a.rows ? v : f32x4{0.0f, 0.0f, 0.0f, 0.0f};
}
__device__ __forceinline__ void keep_features(const StepF32 &a, int r0, int e, f32x4 v) // for the weights' part
{
    *reinterpret_cast<f32x4 *>(a.x + (int64_t)(r0 + e % ROWS) * a.F + 4 * (e / ROWS)) = v;
}

constexpr int ROWS_BARRIERS = 4; // in step_rows

// ROWS minibatch rows, from r0, by the first `waves` wavefronts; wavefront w owns units 16 J w .. of both hidden layers, J tiles (one
// or two up to 256 units, so that the products of a layer are spread over as many wavefronts as there are).  The rows'
// features lie in x_l; `ready`, called once the first weights are requested, sees to that and returns the label of row c.
template <int J, int DEPTH, bool FRESH, class Ready>
__device__ __forceinline__ void step_rows(const StepF32 &a, const f32x4 *x_l, int r0, unsigned char *rows_lds, int waves, Ready ready)
{
    constexpr int E = 4 * J;
    constexpr int FIRST = 4; // (32 or 64 features: all of their groups)
    const int F = a.F, H1 = a.H1, H2 = a.H2, r1 = (H1 + 15) / 16 * 4, r2 = (H2 + 15) / 16 * 4;
    f32x4 *h1_l = reinterpret_cast<f32x4 *>(rows_lds); // [r1][ROWS]
    f32x4 *d2_l = h1_l + r1 * ROWS;                    // [r2][ROWS]
    float *part_l = reinterpret_cast<float *>(d2_l + r2 * ROWS); // [WAVES][ROWS]
    float *dy_l = part_l + WAVES * ROWS;                         // [ROWS]
    const int tid = FRESH ? crew_thread() : threadIdx.x, lane = tid & 63, p = lane >> 4, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int first = 16 * J * wave, unit0 = first + E * p; // this lane's units: unit0 .. unit0 + E - 1
    const bool has1 = first < H1, has2 = first < H2;
    const bool valid = r0 + c < a.rows;

    const F32Layer l1{a.theta + a.off_w1, a.theta + a.off_b1, F, H1}, l2{a.theta + a.off_w2, a.theta + a.off_b2, H1, H2};
    auto slice = [&](const float *copy, auto ordinary, int K) {
        if constexpr (FRESH) return CopySlice(copy, K, wave, lane);
        else return ordinary;
    };
    const auto s1 = slice(a.w1t, ForwardSlice<J>(l1, first, p, c), F), s2 = slice(a.w2t, ForwardSlice<J>(l2, first, p, c), H1);
    const auto back = slice(a.w2, BackSlice<J>(l2, first, p, c), H2);
    // Everything the first two layers need is requested before anything is waited for (behind the features, by the caller)
    float b1[E], b2[E], w3[E], w1f[FIRST][4][J], w2f[DEPTH][4][J];
    // (units past a layer's end get what follows, the moments at the latest, and are never used)
    auto vector = [&](uint64_t off, float (&v)[E]) {
#pragma unroll
        for (int m = 0; m < J; ++m) {
            const f32x4 four = __builtin_bit_cast(f32x4, fresh_16<FRESH>(a.theta, 4u * (uint32_t)(unit0 + 4 * m), 4u * (uint32_t)off));
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * m + e] = four[e];
        }
    };
    vector(a.off_b1, b1);
    vector(a.off_b2, b2);
    vector(a.off_w3, w3);
    uint32_t nought = 0;
    asm("" : "+v"(nought)); // (a load of one address for all lanes would be waited for where it stands, to become a scalar)
    float bias3 = fresh_float<FRESH>(a.theta, nought, 4 * (uint32_t)a.off_b3);
    if (has1) request<J, FIRST>(s1, F, w1f);
    // (A wavefront stands still until its loads have started, 16 cycles a kilobyte and unit: with the weights at hand in the L2,
    // most of the second layer's are requested behind the first one's product, and those of the way back behind the second's.)
    constexpr int AT_ONCE = FRESH ? 2 : DEPTH;
    if (has2) request<J, DEPTH>(s2, H1, w2f, 0, AT_ONCE);
    __builtin_amdgcn_sched_barrier(0);
    float target = ready(tid);
    asm volatile("" : "+v"(target), "+v"(bias3)); // (there by now; left to their use, they wait for all later loads, too)

    // ---- h1 = relu(x W1 + b1)
    float h1[E];
    if (has1) {
        f32x4 acc[J];
#pragma unroll
        for (int e = 0; e < E; ++e) acc[e % J][e / J] = b1[e];
        product<J, FIRST>(s1, F, x_l, p, c, w1f, acc);
        if (FRESH) {
            __builtin_amdgcn_sched_barrier(0);
            if (has2) request<J, DEPTH>(s2, H1, w2f, AT_ONCE);
            __builtin_amdgcn_sched_barrier(0);
        }
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
    float wbf[DEPTH][4][J];
    if (!FRESH && has1) request<J, DEPTH>(back, H2, wbf);
    y += __shfl_xor(y, 16);
    y += __shfl_xor(y, 32);
    if (p == 0) part_l[wave * ROWS + c] = y;
    lds_barrier();
    if (tid < ROWS) {
        float pred = bias3;
        for (int w = 0; w < waves; ++w) pred += part_l[w * ROWS + tid];
        const float d = pred - target;
        const float g = r0 + tid < a.rows ? 2.0f * d / (target * (float)a.rows) : 0.0f;
        a.dy[r0 + tid] = g;
        a.lterm[r0 + tid] = r0 + tid < a.rows ? d * d / target : 0.0f;
        dy_l[tid] = g;
    }
    if (FRESH && has1) request<J, DEPTH>(back, H2, wbf);
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
        product<J, DEPTH>(back, H2, d2_l, p, c, wbf, acc);
        float d1[E];
#pragma unroll
        for (int e = 0; e < E; ++e) d1[e] = h1[e] > 0.0f ? acc[e % J][e / J] : 0.0f;
        store_units<J>(a.d1 + (int64_t)(r0 + c) * H1, unit0, H1, d1);
    }
}

template <int J>
constexpr int rows_depth() { return J <= 2 ? 8 : 4; } // groups of weights requested together

// One more block works out Adam's scales
template <int J>
__global__ __launch_bounds__(64 * WAVES, 2) void step_rows_f32_kernel(StepF32 a)
{
    if (blockIdx.x == gridDim.x - 1) {
        if (threadIdx.x == 0) *a.scales = step_scales(a, a.step_in_call);
        return;
    }
    extern __shared__ __attribute__((aligned(16))) unsigned char rows_lds[];
    f32x4 *x_l = reinterpret_cast<f32x4 *>(rows_lds); // [F / 4][ROWS]
    const int r0 = blockIdx.x * ROWS, threads = blockDim.x, items = a.F / 4 * ROWS, tid = threadIdx.x;
    const f32x4 first_features = row_features(a, a.row0, r0, min(tid, items - 1));
    const float target = a.y[a.row0 + min(r0 + (tid & 15), a.rows - 1)];
    step_rows<J, rows_depth<J>(), false>(a, x_l, r0, rows_lds + items * sizeof(f32x4), threads / 64, [&](int) {
        auto keep = [&](int e, f32x4 v) {
            x_l[e] = v;
            keep_features(a, r0, e, v);
        };
        if (tid < items) keep(tid, first_features);
        for (int e = tid + threads; e < items; e += threads) keep(e, row_features(a, a.row0, r0, e));
        lds_barrier();
        return target;
    });
}

// --------------------------------------------------------------------------------------------- weights kernel

// Blocks of work, in order: the TILE x TILE tiles of W2, those of W1, then 16 columns of the output layer.

// One of WAVES parts of a tile's sums, by a wavefront: G[m][n] = sum_r A[r][m] D[r][n], both row-major over the minibatch rows
// (A = h1 or x, D = d2 or d1); as two by two interleaved matrix-core tiles, so that one 8-byte load per lane and row serves
// two.  Part w takes every eighth group of sixteen rows.  Columns past a matrix's width read what follows (the buffers are
// padded for it) and are never used.  The first tile row also sums the columns of D: the bias gradient.
template <bool FRESH>
__device__ __forceinline__ void tile_part(const float *A, const float *D, int M, int N, int m0, int n0, int groups, int w, int lane,
                                          float (*part)[TILE], float *colsum)
{
    constexpr int POLICY = FRESH ? CREW_SC1 : 0;
    const int p = lane >> 4, c = lane & 15;
    const uint32_t a_lane = 4u * (uint32_t)(4 * p * M + m0 + 2 * c), d_lane = 4u * (uint32_t)(4 * p * N + n0 + 2 * c);
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    float bsum[2] = {0.0f, 0.0f};
    // A group of sixteen rows: at an offset where the rows are a crew's few, else by a descriptor of its own, which ends with the
    // columns that it may read (2^21 rows of 512 units are 2^32 bytes)
    auto rows_of = [](const float *matrix, int width, int g) {
        if (FRESH) return crew_buffer(matrix);
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<float *>(matrix + (int64_t)16 * g * width), 0, (16 * width + TILE) * 4, RSRC_FLAGS);
    };
    constexpr int BATCH = 4; // groups requested together
    for (int g0 = w; g0 < groups; g0 += BATCH * WAVES) {
        i32x2 av[BATCH][4], dv[BATCH][4];
#pragma unroll
        for (int u = 0; u < BATCH; ++u) {
            const int g = g0 + u * WAVES;
            if (g >= groups) break;
            const __amdgpu_buffer_rsrc_t ar = rows_of(A, M, g), dr = rows_of(D, N, g);
            const int row = FRESH ? 16 * g : 0;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                av[u][t] = __builtin_amdgcn_raw_buffer_load_b64(ar, a_lane, (row + t) * M * 4, POLICY);
                dv[u][t] = __builtin_amdgcn_raw_buffer_load_b64(dr, d_lane, (row + t) * N * 4, POLICY);
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
            *reinterpret_cast<float2 *>(&part[2 * (4 * p + q) + i][2 * c]) = make_float2(acc[i][0][q], acc[i][1][q]);
    if (m0 == 0) {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            bsum[j] += __shfl_xor(bsum[j], 16);
            bsum[j] += __shfl_xor(bsum[j], 32);
            if (p == 0) colsum[2 * c + j] = bsum[j];
        }
    }
}

// The update of a tile's parameters by THREADS threads: the parts of its sums added in order, then Adam
template <int THREADS, bool FRESH>
struct TileUpdate {
    static constexpr int PER = TILE * TILE / THREADS; // parameters of a thread, TILE / PER rows apart
    const StepF32 &a;
    int tid, M, N, m0, n0;
    uint32_t off, bias_at;
    AdamNext state[PER], bias_state; // as they were

    __device__ __forceinline__ TileUpdate(const StepF32 &args, bool second, int m0_, int n0_, int tid_)
        : a(args), tid(tid_), M(second ? args.H1 : args.F), N(second ? args.H2 : args.H1), m0(m0_), n0(n0_)
    {
        off = (uint32_t)(second ? a.off_w2 : a.off_w1);
        bias_at = (uint32_t)(second ? a.off_b2 : a.off_b1) + min(n0 + tid % TILE, N - 1);
    }

    __device__ __forceinline__ AdamNext load(uint32_t i) const // (past the L1: as a crew grows, a tile passes from member to member)
    {
        const __amdgpu_buffer_rsrc_t theta = crew_buffer(a.theta);
        auto get = [&](uint32_t moment) { return __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(theta, 4 * i, 4 * moment * (uint32_t)a.P, FRESH ? CREW_SC1 : 0)); };
        return {get(0), get(1), get(2)};
    }

    __device__ __forceinline__ float store(uint32_t i, AdamNext s, float g, AdamScales scales) const
    {
        const __amdgpu_buffer_rsrc_t theta = crew_buffer(a.theta);
        auto put = [&](uint32_t moment, float v) { __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(v), theta, 4 * i, 4 * moment * (uint32_t)a.P, 0); };
        const AdamNext next = adam_next(s.w, s.m, s.v, g, a.beta1, a.beta2, a.eps, scales);
        put(0, next.w);
        put(1, next.m);
        put(2, next.v);
        return next.w;
    }

    __device__ __forceinline__ void request()
    {
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const int m = m0 + tid / TILE + e * (TILE / PER), n = n0 + tid % TILE;
            state[e] = load(off + (uint32_t)(min(m, M - 1) * N + min(n, N - 1)));
        }
        if (m0 == 0) bias_state = load(bias_at);
    }

    // copy(m, n, w): what else becomes of a new weight
    template <class Copy>
    __device__ __forceinline__ void update(const float (*part)[TILE][TILE], const float (*colsum)[TILE], AdamScales scales, Copy copy) const
    {
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const int lm = tid / TILE + e * (TILE / PER), ln = tid % TILE;
            float g = part[0][lm][ln];
#pragma unroll
            for (int w = 1; w < WAVES; ++w) g += part[w][lm][ln];
            if (m0 + lm < M && n0 + ln < N) copy(m0 + lm, n0 + ln, store(off + (uint32_t)((m0 + lm) * N + n0 + ln), state[e], g, scales));
        }
        if (m0 == 0 && tid < TILE && n0 + tid < N) {
            float g = colsum[0][tid];
#pragma unroll
            for (int w = 1; w < WAVES; ++w) g += colsum[w][tid];
            (void)store(bias_at, bias_state, g, scales);
        }
    }
};

// The output layer: [gW3 ; gb3] = [h2 ; 1]^T dy, 16 columns by THREADS threads: 32 row groups, rows in order, four groups' sums then
// along the wavefront and the eight fours in order.
constexpr int OUT_GROUPS = 32;
template <int THREADS, bool FRESH>
struct OutputBlock {
    static constexpr int SETS = OUT_GROUPS * 16 / THREADS; // row groups of a thread
    const StepF32 &a;
    int tid, col;
    float w, m, v;

    __device__ __forceinline__ OutputBlock(const StepF32 &args, int block, int tid_) : a(args), tid(tid_), col(block * 16 + (tid_ & 15)) {}
    __device__ __forceinline__ uint64_t parameter() const { return col < a.H2 ? a.off_w3 + col : a.off_b3; }

    __device__ __forceinline__ void request()
    {
        const uint32_t at = 4u * (uint32_t)parameter(), P4 = 4u * (uint32_t)a.P;
        w = fresh_float<FRESH>(a.theta, at, 0);
        m = fresh_float<FRESH>(a.theta, at, P4);
        v = fresh_float<FRESH>(a.theta, at, 2 * P4);
    }

    __device__ __forceinline__ void sum(float *psum) const // [OUT_GROUPS / 4][16]
    {
        constexpr int AHEAD = 8;
        const int per = (a.padded + OUT_GROUPS - 1) / OUT_GROUPS;
        // (a group's first row in the offset where the rows are a crew's few, else in the base; a 32nd of what fits the memory is
        // less than 2^32 bytes)
        const float *h2[SETS], *dy[SETS];
        uint32_t at[SETS], dy_at[SETS];
        int rows[SETS]; // none for groups behind the minibatch, whose loads, and a last group's, end in the buffers behind h2 and dy
        float sum[SETS];
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
            const int group = (tid >> 4) + s * (THREADS / 16), first = min(group * per, a.padded - 1);
            rows[s] = a.padded - group * per;
            const int in_offset = FRESH ? first : 0, in_base = first - in_offset;
            h2[s] = a.h2 + (int64_t)in_base * a.H2;
            dy[s] = a.dy + in_base;
            at[s] = 4u * (uint32_t)(in_offset * a.H2 + min(col, a.H2 - 1));
            dy_at[s] = 4u * (uint32_t)in_offset;
            sum[s] = 0.0f;
        }
        for (int r = 0; r < per; r += AHEAD) {
            float h[SETS][AHEAD], d[SETS][AHEAD];
#pragma unroll
            for (int s = 0; s < SETS; ++s)
#pragma unroll
                for (int u = 0; u < AHEAD; ++u) {
                    const uint32_t row = min(r + u, per - 1);
                    h[s][u] = fresh_float<FRESH>(h2[s], at[s], 4u * row * (uint32_t)a.H2);
                    d[s][u] = fresh_float<FRESH>(dy[s], dy_at[s], 4u * row);
                }
#pragma unroll
            for (int s = 0; s < SETS; ++s)
#pragma unroll
                for (int u = 0; u < AHEAD; ++u) {
                    const float next = col < a.H2 ? fmaf(h[s][u], d[s][u], sum[s]) : sum[s] + d[s][u];
                    sum[s] = r + u < min(per, rows[s]) ? next : sum[s];
                }
        }
#pragma unroll
        for (int s = 0; s < SETS; ++s) {
            sum[s] += __uint_as_float(lane_exchange(__float_as_uint(sum[s]), 16));
            sum[s] += __uint_as_float(lane_exchange(__float_as_uint(sum[s]), 32));
            if ((tid & 63) < 16) psum[((tid >> 6) + s * (THREADS / 64)) * 16 + tid % 16] = sum[s];
        }
    }

    __device__ __forceinline__ void update(const float *psum, AdamScales scales) const
    {
        if (tid >= 16 || col > a.H2) return;
        float g = psum[tid];
#pragma unroll
        for (int four = 1; four < OUT_GROUPS / 4; ++four) g += psum[four * 16 + tid];
        (void)eck::adam_one(a.theta, a.P, parameter(), w, m, v, g, a.beta1, a.beta2, a.eps, scales);
    }
};

__global__ __launch_bounds__(64 * WAVES) void step_weights_f32_kernel(StepF32 a, int blocks2, int blocks1)
{
    __shared__ float part[WAVES][TILE][TILE];
    __shared__ float colsum[WAVES][TILE];
    __shared__ double loss[WAVES];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool bad = *a.bad != 0;
    const AdamScales scales = *a.scales;
    int block = blockIdx.x;
    if (block < blocks2 + blocks1) {
        const bool second = block < blocks2; // a tile of W2, else of W1
        if (!second) block -= blocks2;
        const int M = second ? a.H1 : a.F, N = second ? a.H2 : a.H1;
        const int nt = (N + TILE - 1) / TILE, m0 = block / nt * TILE, n0 = block % nt * TILE;
        TileUpdate<64 * WAVES, false> tile(a, second, m0, n0, tid);
        tile.request();
        tile_part<false>(second ? a.h1 : a.x, second ? a.d2 : a.d1, M, N, m0, n0, a.padded / 16, wave, lane, part[wave], colsum[wave]);
        lds_barrier();
        if (!bad) tile.update(part, colsum, scales, [](int, int, float) {});
        return;
    }
    block -= blocks2 + blocks1;
    OutputBlock<64 * WAVES, false> out(a, block, tid);
    out.request();
    out.sum(&part[0][0][0]);
    const bool report = a.report_loss && block == 0;
    if (report) {
        const double s = loss_part<WAVES>(a.lterm, a.rows, wave, lane);
        if (lane == 0) loss[wave] = s;
    }
    lds_barrier();
    if (bad) return;
    out.update(&part[0][0][0], scales);
    if (report && tid == 64) {
        double s = loss[0];
#pragma unroll
        for (int w = 1; w < WAVES; ++w) s += loss[w];
        *a.loss_out = (float)(s / a.rows);
    }
}

// ------------------------------------------------------------------------------------- all steps in one launch
//
// The same steps by a crew (crew.h): rows, a barrier, weights, a barrier, twelve wavefronts a member (so that a lane has 168
// registers).  Eight take a tile of W2 or W1, the other four 16 columns of the output layer.  All sums are those of
// the two launches, in their order: the same bits.
constexpr int CREW_THREADS = 768, CREW_MAIN = 64 * WAVES, CREW_SIDE = CREW_THREADS - CREW_MAIN;

struct CrewLds { // byte offsets: either part's buffers from 0, behind them what outlives a part
    uint32_t out, x, y, scales, total;
    __host__ __device__ explicit CrewLds(int F, int H1, int H2)
    {
        const uint32_t rows = ROWS * 16 * ((H1 + 15) / 16 * 4 + (H2 + 15) / 16 * 4) + (WAVES + 1) * ROWS * 4;
        out = (WAVES * TILE * TILE + WAVES * TILE) * 4;
        const uint32_t weights = out + OUT_GROUPS / 4 * 16 * 4;
        x = rows > weights ? rows : weights;
        y = x + 2 * ROWS * F * 4;
        scales = y + 2 * ROWS * 4;
        total = scales + (uint32_t)sizeof(AdamScales);
    }
};

// FULL: all members have been there from the start, as in most calls (one code for all, and so a number of members that varies,
// takes 0.1 to 0.25 us a step more)
template <bool FULL>
__device__ __forceinline__ void crew_steps(const StepF32 &a, Crew crew, int first_step, int n_steps, uint64_t n_pairs, unsigned char *crew_lds)
{
    if (FULL) {
        crew.size = CREW_MOST;
        crew.barriers = 0;
        first_step = 0;
    }
    const CrewLds at(a.F, a.H1, a.H2);
    const int rank = (int)crew.rank, row_blocks = a.padded / ROWS, items = a.F / 4 * ROWS;
    const int widest = a.H1 > a.H2 ? a.H1 : a.H2, row_waves = (widest + 15) / 16;
    const int groups1 = copy_groups(a.H1), groups2 = copy_groups(a.H2);
    auto over = [](int v) { return (v + TILE - 1) / TILE; };
    const int across2 = over(a.H2), across1 = over(a.H1), tiles2 = across1 * across2, tiles1 = over(a.F) * across1;
    const int tiles = tiles2 + tiles1, out_blocks = (a.H2 + 1 + 15) / 16, items_most = tiles > out_blocks ? tiles : out_blocks;
    auto x_of = [&](int step) { return reinterpret_cast<f32x4 *>(crew_lds + at.x) + (step & 1) * items; };
    auto y_of = [&](int step) { return reinterpret_cast<float *>(crew_lds + at.y) + (step & 1) * ROWS; };
    AdamScales *scales_of = reinterpret_cast<AdamScales *>(crew_lds + at.scales); // of the step, in its weights' phase
    // The features and labels come from memory, some 2 us: the wavefronts that have no units fetch those of a member's first rows
    // of a step during the step before.
    auto stage = [&](int step, uint64_t row0, int r0, int t) { // by threads t = 0 .. CREW_SIDE - 1
        const float y = a.y[row0 + min(r0 + (t & 15), a.rows - 1)];
        for (int e = t; e < items; e += CREW_SIDE) x_of(step)[e] = row_features(a, row0, r0, e);
        if (t < ROWS) y_of(step)[t] = y;
    };
    uint64_t row0 = first_step == 0 ? 0 : (uint32_t)first_step % ((uint32_t)n_pairs / (uint32_t)a.rows) * (uint32_t)a.rows;
    if (rank < row_blocks) {
        const int t = crew_thread() - CREW_MAIN;
        if (t >= 0) stage(first_step, row0, ROWS * rank, t);
        lds_barrier();
    }
    int step = first_step, members = FULL ? (int)CREW_MOST : (int)crew.size;
    auto one_step = [&] __attribute__((always_inline)) {
        const bool last = step + 1 == n_steps;
        uint64_t next_row0 = row0 + a.rows;
        if (next_row0 == n_pairs) next_row0 = 0;
        for (int i = rank; i < row_blocks; i += members) {
            const int tid = crew_thread(), wave = __builtin_amdgcn_readfirstlane(tid >> 6), r0 = ROWS * i;
            if (i != rank) {
                lds_barrier();
                if (wave >= WAVES) stage(step, row0, r0, tid - CREW_MAIN);
                lds_barrier();
            }
            if (wave < row_waves) {
                step_rows<CREW_J, 8, true>(a, x_of(step), r0, crew_lds, row_waves, [&](int tid) { return y_of(step)[tid & 15]; });
            } else {
                if (wave >= WAVES) {
                    for (int e = tid - CREW_MAIN; e < items; e += CREW_SIDE) keep_features(a, r0, e, x_of(step)[e]);
                    if (i == rank && !last) stage(step + 1, next_row0, r0, tid - CREW_MAIN);
                }
                for (int barrier = 0; barrier < ROWS_BARRIERS; ++barrier) lds_barrier();
            }
        }
        if (crew_thread() == CREW_MAIN) *scales_of = step_scales(a, step);
        row0 = next_row0;
        // (what a member updates is requested in front of the barrier)
        auto together = [&](int base) {
            if (base == 0) {
                crew.arrive();
                crew.meet();
            }
        };
        for (int base = 0; base < items_most; base += members) {
            const int tid = crew_thread(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
            if (wave < WAVES) {
                using Parts = float(*)[TILE][TILE];
                const Parts part = reinterpret_cast<Parts>(crew_lds);
                float(*colsum)[TILE] = reinterpret_cast<float(*)[TILE]>(part + WAVES);
                const int item = base + rank;
                const bool mine = item < tiles, second = item < tiles2;
                const int block = second ? item : item - tiles2, across = second ? across2 : across1;
                const int m0 = block / across * TILE, n0 = block % across * TILE;
                TileUpdate<CREW_MAIN, true> tile(a, second, m0, n0, tid);
                if (mine) tile.request();
                together(base);
                if (mine) tile_part<true>(second ? a.h1 : a.x, second ? a.d2 : a.d1, tile.M, tile.N, m0, n0, a.padded / 16, wave, lane, part[wave], colsum[wave]);
                lds_barrier();
                if (mine) {
                    tile.update(part, colsum, *scales_of, [&](int m, int n, float w) {
                        if (second) {
                            a.w2t[copy_at(n, m, groups1)] = w;
                            a.w2[copy_at(m, n, groups2)] = w;
                        } else {
                            a.w1t[copy_at(n, m, a.F / 16)] = w;
                        }
                    });
                }
            } else {
                const int item = base + members - 1 - rank; // (the first ones to members that have no tile, if there are any)
                const bool mine = item < out_blocks;
                OutputBlock<CREW_SIDE, true> out(a, item, tid - CREW_MAIN);
                float *psum = reinterpret_cast<float *>(crew_lds + at.out);
                if (mine) out.request();
                together(base);
                if (mine) out.sum(psum);
                lds_barrier();
                if (mine) {
                    out.update(psum, *scales_of);
                    if (last && item == 0 && wave == CREW_THREADS / 64 - 1) {
                        const double s = loss_sum_fresh<WAVES>(a.lterm, a.rows, lane);
                        if (lane == 0) *a.loss_out = (float)(s / a.rows);
                    }
                }
            }
            if (members < items_most) lds_barrier(); // (the LDS is free again)
        }
        if (!last) {
            if (!FULL) crew.summon(step + 1);
            crew.arrive();
            crew.meet();
        }
    };
    for (; step < n_steps; ++step) {
        one_step();
        if (!FULL && step + 1 < n_steps && crew.grown()) members = (int)crew.size;
    }
    if (!FULL) crew.dismiss();
}

__global__ __launch_bounds__(CREW_THREADS) void steps_f32_crew_kernel(StepF32 a, CrewState *state, unsigned pick, int n_steps, uint64_t n_pairs,
                                                                      unsigned at_once)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char crew_lds[];
    if (blockIdx.x % CREW_DIES != pick || *a.bad != 0) return;
    Crew crew;
    const int first_step = crew.join(state, at_once, reinterpret_cast<uint32_t *>(crew_lds));
    if (first_step < 0) return;
    __syncthreads(); // (the words are read)
    if (first_step == 0 && crew.size == CREW_MOST) crew_steps<true>(a, crew, 0, n_steps, n_pairs, crew_lds);
    else crew_steps<false>(a, crew, first_step, n_steps, n_pairs, crew_lds);
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
    w.scales = take(sizeof(CrewState) / 4 - TILE);
    w.total = o;
    return w;
}

// the fewest tiles per wavefront that eight wavefronts cover the wider layer with
int tiles_a_wave(const eck_model *m)
{
    const int tiles = ((m->widths[1] > m->widths[2] ? m->widths[1] : m->widths[2]) + 15) / 16;
    return (tiles + WAVES - 1) / WAVES;
}

// Up to 128 units (copies are kept for those) and 32 blocks of rows, one a member; a crew's launch and roll take as long as two
// steps gain.  us a call (replayed graphs), two launches a step / crew:
//   64-128-128, 250 rows: 2 steps 38.6 / 40.1, 3 steps 59.0 / 56.5, 8 steps 126 / 110; 512: 141 / 126, 1000: 159 / 218
//   32-64-64, 8 steps of 16 rows 89 / 77, 512: 111 / 103; 64-16-16, 8 steps of 64 rows 85.3 / 73.4
//   64-256-256, 8 steps of 128 rows 211 / 205, 250: 219 / 227 (its weights, 0.6 MB a block of rows, are what a unit is slow with)
bool crew_takes(const eck_model *m, int minibatch, int n_steps) { return m->d_copies && n_steps >= 3 && minibatch <= 512; }

// a crew's words lie where the two launches leave Adam's scales
CrewState *crew_state(const eck_model *m, int minibatch, void *ws)
{
    return reinterpret_cast<CrewState *>(static_cast<char *>(ws) + buffers_for(m, minibatch).scales);
}

// a crew's copies, in floats
struct Copies {
    uint32_t w2t, w2, total; // w1t first
};
__host__ __device__ inline Copies copies_of(int F, int H1, int H2)
{
    Copies c;
    c.w2t = (uint32_t)(16 * copy_groups(H1) * F);
    c.w2 = c.w2t + (uint32_t)(16 * copy_groups(H2) * 16 * copy_groups(H1));
    c.total = c.w2 + (uint32_t)(16 * copy_groups(H1) * 16 * copy_groups(H2));
    return c;
}

// The last block: labels, and the crew's words; the others: its copies of the weights, four of a lane a thread
__global__ __launch_bounds__(1024) void refit_f32_prepare_kernel(const float *theta, uint32_t off_w1, uint32_t off_w2, int F, int H1, int H2,
                                                                 float *copies, const float *energy, uint64_t n_pairs, float *y, RefitScalars *sc,
                                                                 CrewState *crew)
{
    if (blockIdx.x == gridDim.x - 1) {
        crew_clear(crew);
        make_labels(energy, n_pairs, y, sc);
        return;
    }
    const Copies at = copies_of(F, H1, H2);
    const uint32_t four = (blockIdx.x * 1024 + threadIdx.x) * 4;
    if (four >= at.total) return;
    const bool first = four < at.w2t, back = four >= at.w2;
    const uint32_t i = (four - (first ? 0 : back ? at.w2 : at.w2t)) / 4;
    const int groups = first ? F / 16 : copy_groups(back ? H2 : H1);
    const int lane = i % 64, group = i / 64 % groups, tile = i / 64 / groups;
    const int n = 16 * tile + (lane & 15), k = 16 * group + 4 * (lane >> 4);
    f32x4 w;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        if (first) w[t] = n < H1 ? theta[off_w1 + (k + t) * H1 + n] : 0.0f;
        else if (back) w[t] = n < H1 && k + t < H2 ? theta[off_w2 + n * H2 + k + t] : 0.0f;
        else w[t] = n < H2 && k + t < H1 ? theta[off_w2 + (k + t) * H2 + n] : 0.0f;
    }
    *reinterpret_cast<f32x4 *>(copies + four) = w;
}

} // namespace

uint64_t eck::refit_f32_copies_bytes(const eck_model *m)
{
    if (m->dtype != ECK_F32 || tiles_a_wave(m) != CREW_J) return 0;
    return 4ull * copies_of(m->widths[0], m->widths[1], m->widths[2]).total;
}

int32_t eck::refit_f32_begin(const eck_model *m, const float *energy, uint64_t n_pairs, float *y, RefitScalars *sc, int32_t n_steps,
                             int32_t minibatch, void *ws, hipStream_t st)
{
    const int F = m->widths[0], H1 = m->widths[1], H2 = m->widths[2];
    const unsigned copies = crew_takes(m, minibatch, n_steps) ? (copies_of(F, H1, H2).total / 4 + 1023) / 1024 : 0;
    hipLaunchKernelGGL(refit_f32_prepare_kernel, dim3(copies + 1), dim3(1024), 0, st, m->d_state, (uint32_t)m->off_w[0], (uint32_t)m->off_w[1], F, H1,
                       H2, m->d_copies, energy, n_pairs, y, sc, crew_state(m, minibatch, ws));
    ECK_HIP_TRY(hipGetLastError());
    return ECK_OK;
}

uint64_t eck::refit_f32_workspace_bytes(const eck_model *m, int minibatch) { return buffers_for(m, minibatch).total; }

int32_t eck::refit_f32_steps(const eck_model *m, const float *feat, uint64_t ld, const float *y, uint64_t n_pairs,
                             int32_t n_steps, int32_t minibatch, float lr, float beta1, float beta2, float eps,
                             const uint32_t *bad_flag, float *loss_scalar, void *ws, CrewSize crew, hipStream_t st)
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
    const int J = tiles_a_wave(m), waves = ((a.H1 > a.H2 ? a.H1 : a.H2) + 16 * J - 1) / (16 * J);
    auto rows_kernel = J == 1   ? step_rows_f32_kernel<1>
                       : J == 2 ? step_rows_f32_kernel<2>
                       : J == 3 ? step_rows_f32_kernel<3>
                                : step_rows_f32_kernel<4>;
    if (crew_takes(m, minibatch, n_steps)) {
        const Copies copies = copies_of(a.F, a.H1, a.H2);
        a.w1t = m->d_copies;
        a.w2t = m->d_copies + copies.w2t;
        a.w2 = m->d_copies + copies.w2;
        const CrewLds at(a.F, a.H1, a.H2);
        ECK_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(steps_f32_crew_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)at.total));
        CrewState *state = crew_state(m, minibatch, ws);
        hipLaunchKernelGGL(steps_f32_crew_kernel, dim3(CREW_DIES * crew.candidates), dim3(CREW_THREADS), at.total, st, a, state, crew_pick(state), n_steps,
                           n_pairs, crew.at_once);
        ECK_HIP_TRY(hipGetLastError());
        return ECK_OK;
    }
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
