// Minibatch Adam steps on the weighted squared error of Eq. (1) for BF16 models (Alg. 1: ModelUpdate; Sec. 6.4).  HIP, gfx950.
//
// A step of the refit is a chain of small dependent products; launched one by one it is bound by launch latency.
// Here it is cut where the data dependencies allow no less:
//   rows:     everything that is local to a minibatch row, for 32 rows per block -- both hidden layers, the output layer,
//             the Eq.-(1) loss term and its derivative, and the deltas of both hidden layers (the back-propagation through
//             W2 included).  Activations pass from layer to layer through LDS.
//   weights:  everything that sums over the rows of the minibatch -- the three weight gradients and the bias gradients --
//             one 32 x 32 tile of a weight matrix by four wavefronts, a quarter of the rows each, added in wavefront order;
//             the Adam update of the tile's parameters follows at once in the same block (each parameter's gradient is
//             complete there), together with the bf16 copies the next step's rows multiply with.
// Two launches a step, or, where the steps are small enough for one die, all steps in one launch by the blocks of a crew
// (crew.h): the same blocks of work and the same bits.
// All large products run on the matrix cores (v_mfma_f32_32x32x16_bf16, fp32 accumulation) with the same operand
// roundings as the launch-per-product path: features, weights, first hidden activations and both deltas in bf16,
// biases and the output weights rounded through bf16, the second hidden layer and the output layer in fp32.
// Every reduction has a fixed order, so a run is reproducible bit for bit.
// What bounds a step is the latency of loads right after a launch or a barrier and the chain of dependent phases, so both
// parts request all that they can name before they wait for any of it, and values become bfloat16 two at a time by the
// hardware's conversion.  Measured, 64-256-256-1, 8 steps of 512 rows, a whole call with the state in and out: 145.0 us with
// two launches a step, 115.5 by a crew (114.9 while its number of members was fixed at the start).  Of a crew's step of some 10 us the rows take 5.3 (the weights of a block of rows,
// 288 KB through one unit's 130 GB/s, 2.2), the weights 3.5, the two barriers what is left.
#include "crew.h"
#include "refit_labels.h"

using namespace eck;

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ uint16_t bf16_bits(float x)
{
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7F800000u) == 0x7F800000u) return (uint16_t)(u >> 16);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// two values as bfloat16, rounded to nearest, in a word (one instruction; by the integer steps above, twelve)
__device__ __forceinline__ uint32_t bf16_two(float a, float b)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const bf16x2 two = {(__bf16)a, (__bf16)b};
    return __builtin_bit_cast(uint32_t, two);
}

__device__ __forceinline__ float through_bf16(float x) { return __uint_as_float((uint32_t)bf16_bits(x) << 16); }

// Matrix-core tile (v_mfma_f32_32x32x16_bf16, D = A * B + C, one wavefront, lane = 32 h + c):
//   A (32 rows x 16 k): lane (h, r = c) holds A[r][8h .. 8h+7]      -> 16 contiguous bytes of a k-major row
//   B (16 k x 32 cols): lane (h, c) holds B[8h .. 8h+7][c]           -> 16 contiguous bytes of a k-major column
//   D (32 x 32):        lane (h, c) register q holds D[8 (q / 4) + 4h + q % 4][c]
__device__ __forceinline__ int d_row(int q, int h) { return 8 * (q >> 2) + 4 * h + (q & 3); }

// Operands of the matrix instructions live in memory in fragment order, so that the 64 lanes of a load read one
// contiguous kilobyte: element (n, k) of a matrix whose k index is the reduction index and whose n index picks the
// row (A) or column (B) of the tile sits at
//   ((n / 32 * (K / 16) + place(n / 32, k / 16)) * 64 + 32 * (k % 16 / 8) + n % 32) * 8 + k % 8    (K = length of the reduction)
// The wavefronts of a block, and the blocks of a launch, walk through tiles at strides of many kilobytes in step, so their
// requests would meet in the same few channels of the L2; place() turns every group of four fragments by the tile's and the
// group's number.
__device__ __forceinline__ int place(int tile, int ks, int K) { return ks ^ ((tile + (ks >> 2)) & (K >= 64 ? 3 : (K >> 4) - 1)); }

__device__ __forceinline__ int64_t frag_at(int n, int k, int K)
{
    return ((int64_t)((n >> 5) * (K >> 4) + place(n >> 5, k >> 4, K)) * 64 + 32 * ((k >> 3) & 1) + (n & 31)) * 8 + (k & 7);
}

struct StepArgs {
    const void *feat;   // [F][ld] bf16 or fp32, minibatch row r = column row0 + r
    uint64_t ld, row0;
    int rows, padded;   // minibatch size B, and the same rounded up to 64: the rows behind it are zeros
    bool aligned;       // no such rows, and the features of four neighbouring ones are whole 8 or 16 bytes
    float *theta;       // fp32 master [theta | m | v | t], n_params = P
    uint64_t P;
    uint64_t off_w1, off_b1, off_w2, off_b2, off_w3, off_b3;
    // bf16 copies of the weights, in fragment order:
    uint16_t *w1t;      // n = unit of layer 1, k = feature       (x W1)
    uint16_t *w2t;      // n = unit of layer 2, k = unit of layer 1   (h1 W2)
    uint16_t *w2;       // n = unit of layer 1, k = unit of layer 2   (d2 W2^T)
    const float *y;     // labels of the whole buffer
    // what the weight gradients sum over the minibatch, bf16 in fragment order with n = unit, k = minibatch row:
    uint16_t *h1t;      // first hidden layer
    uint16_t *d2t;      // delta of the second hidden layer
    uint16_t *d1t;      // delta of the first hidden layer
    uint16_t *xt;       // features
    float *h2;          // fp32 [B][H2]
    float *dy;          // fp32 [B]
    float *lterm;       // fp32 [B]  Eq.-(1) terms of the rows
    const uint32_t *bad; // data error found in the labels: leave the model alone
    float *loss_out;    // mean of the Eq.-(1) terms, written in the step with report_loss set
    AdamScales *scales; // of the step (rows kernel -> weights kernel); a crew: its words
    int step_in_call, report_loss;
    float lr, beta1, beta2, eps;
};

// ------------------------------------------------------------------------------------------------ rows kernel

// Weight fragments of one 32-column tile (k-major columns starting at b_col) are fetched up to 16 k-steps at a time,
// so that one round trip to the L2 covers that much of the reduction; the first batch is requested long before
// its product starts (EARLY k-steps), the rest -- reductions deeper than 256 -- inside the product.
template <int K>
struct Fragments {
    static constexpr int EARLY = K / 16 < 16 ? K / 16 : 16;
    bf16x8 b[EARLY];
};

// fragment ks of tile `tile` of a matrix: the K / 16 fragments of a 32-column tile are 512 elements each
template <int K, bool FRESH>
__device__ __forceinline__ bf16x8 fragment(const uint16_t *matrix, int tile, int ks, int lane)
{
    return __builtin_bit_cast(bf16x8, fresh_16<FRESH>(matrix, 16u * lane, 2u * (uint32_t)(tile * 32 * K + 512 * place(tile, ks, K))));
}

template <int K, bool FRESH>
__device__ __forceinline__ void fetch_fragments(const uint16_t *matrix, int tile, int lane, Fragments<K> &f, int first = 0,
                                                int end = Fragments<K>::EARLY)
{
#pragma unroll
    for (int ks = 0; ks < Fragments<K>::EARLY; ++ks)
        if (ks >= first && ks < end) f.b[ks] = fragment<K, FRESH>(matrix, tile, ks, lane);
}

// A (32 x K, bf16, in LDS with row stride LDA) * B (K x 32, tile `tile` of a matrix, first batch of fragments in f)
template <int K, int LDA, bool FRESH>
__device__ __forceinline__ f32x16 row_tile_product(const uint16_t *a_lds, const uint16_t *matrix, int tile, const Fragments<K> &f, int lane)
{
    constexpr int EARLY = Fragments<K>::EARLY;
    const uint16_t *ap = a_lds + (lane & 31) * LDA + 8 * (lane >> 5);
    f32x16 acc;
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[q] = 0.0f;
    bf16x8 later[K / 16 > EARLY ? EARLY : 1];
    if (K / 16 > EARLY) {
#pragma unroll
        for (int ks = 0; ks < EARLY; ++ks) later[ks] = fragment<K, FRESH>(matrix, tile, EARLY + ks, lane);
    }
#pragma unroll
    for (int ks = 0; ks < EARLY; ++ks)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8 *>(ap + 16 * ks), f.b[ks], acc, 0, 0, 0);
    if (K / 16 > EARLY) {
        static_assert(K / 16 <= 2 * EARLY, "reductions of at most 512");
#pragma unroll
        for (int ks = 0; ks < K / 16 - EARLY; ++ks)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8 *>(ap + 16 * (EARLY + ks)), later[ks], acc,
                                                          0, 0, 0);
    }
    return acc;
}

// Registers 4g .. 4g+3 of a D tile -- rows 8g + 4h .. +3 of column c -- as bf16 into a fragment-ordered matrix with
// n = column (unit), k = minibatch row: four consecutive k of one lane's fragment, one 8-byte store.
__device__ __forceinline__ void store_rows4(uint16_t *t, int unit, int rows_total, int row, uint32_t lo, uint32_t hi)
{
    *reinterpret_cast<uint2 *>(t + frag_at(unit, row, rows_total)) = make_uint2(lo, hi);
}

// the same four values into a row-major LDS matrix: rows row .. row + 3 of column col
__device__ __forceinline__ void put_rows4(uint16_t *lds, int ld, int row, int col, uint32_t lo, uint32_t hi)
{
    uint16_t *at = lds + row * ld + col;
    at[0] = (uint16_t)lo;
    at[ld] = (uint16_t)(lo >> 16);
    at[2 * ld] = (uint16_t)hi;
    at[3 * ld] = (uint16_t)(hi >> 16);
}

__device__ __forceinline__ AdamScales step_scales(const StepArgs &a, int step_in_call)
{
    return adam_scales(a.lr, a.beta1, a.beta2, a.theta[3 * a.P], step_in_call); // (the count itself is advanced once, after the last step)
}

// LDS of a block that takes 32 rows, and of their features
template <int F, int H1, int H2>
constexpr size_t rows_lds_bytes()
{
    constexpr int NW = (H1 > H2 ? H1 : H2) / 32;
    return (size_t)32 * ((H1 + 8) + (H2 + 8)) * sizeof(uint16_t) + (NW * 32 + 32 + NW * 32 * 33) * sizeof(float);
}

// The features and labels of 32 minibatch rows, from row r0, by NT threads: four neighbouring rows of a feature each.
template <int F, bool FEAT_BF16, int NT>
struct RowInputs {
    static constexpr int FOURS = 32 * F / 4, PER = (FOURS + NT - 1) / NT, LDX = F + 8; // LDS row stride: no conflicts
    uint2 x2[FEAT_BF16 ? PER : 1];
    float4 x4[FEAT_BF16 ? 1 : PER];
    float y;

    static __device__ __forceinline__ int item(int t, int k) { return min(t + k * NT, FOURS - 1); }

    __device__ __forceinline__ void request(const StepArgs &a, uint64_t row0, int r0, int t) // row0: the minibatch's first column
    {
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int e = item(t, k), row = r0 + 4 * (e & 7);
            const uint64_t at = (uint64_t)(e >> 3) * a.ld + row0;
            const uint16_t *f2 = reinterpret_cast<const uint16_t *>(a.feat) + at;
            const float *f4 = reinterpret_cast<const float *>(a.feat) + at;
            if (a.aligned) {
                if constexpr (FEAT_BF16) x2[k] = *reinterpret_cast<const uint2 *>(f2 + row);
                else x4[k] = *reinterpret_cast<const float4 *>(f4 + row);
            } else { // one by one, the rows behind the minibatch from its last
                const int last = a.rows - 1;
                if constexpr (FEAT_BF16) {
                    uint32_t v[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) v[u] = f2[min(row + u, last)];
#pragma unroll
                    for (int u = 0; u < 4; ++u) v[u] = row + u <= last ? v[u] : 0;
                    x2[k] = make_uint2(v[0] | v[1] << 16, v[2] | v[3] << 16);
                } else {
                    float v[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) v[u] = f4[min(row + u, last)];
#pragma unroll
                    for (int u = 0; u < 4; ++u) v[u] = row + u <= last ? v[u] : 0.0f;
                    x4[k] = make_float4(v[0], v[1], v[2], v[3]);
                }
            }
        }
        y = a.y[row0 + min(r0 + (t & 31), a.rows - 1)];
    }

    // x: [32][LDX], the rows as bf16; xt: the minibatch's features in fragment order, its rows from r0
    __device__ __forceinline__ void keep(const StepArgs &a, int t, uint16_t *x, uint16_t *xt, int r0) const
    {
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int e = item(t, k);
            uint2 two;
            if constexpr (FEAT_BF16) two = x2[k];
            else two = make_uint2(bf16_two(x4[k].x, x4[k].y), bf16_two(x4[k].z, x4[k].w));
            put_rows4(x, LDX, 4 * (e & 7), e >> 3, two.x, two.y);
            store_rows4(xt, e >> 3, a.padded, r0 + 4 * (e & 7), two.x, two.y);
        }
    }
};

constexpr int ROWS_BARRIERS = 4; // in step_rows

// 32 minibatch rows, row r0 of the minibatch on, by H / 32 wavefronts of the widest layer, one per 32-column tile, so every
// layer is one tile product per wavefront.  A wavefront fetches the weight fragments of its next product before it waits for
// anything else: those of the first two layers at the very start, those of the back-propagation while the output layer is
// being reduced.  The rows' features lie in x_l; `ready`, called once the first weights are requested, sees to that and
// returns the label of row tid % 32.
template <int F, int H1, int H2, bool FRESH, class Ready>
__device__ __forceinline__ void step_rows(const StepArgs &a, const uint16_t *x_l, int r0, unsigned char *rows_lds, Ready ready)
{
    constexpr int NW = (H1 > H2 ? H1 : H2) / 32;
    constexpr int LDX = F + 8, LD1 = H1 + 8, LD2 = H2 + 8; // LDS row strides in bf16: 16-byte fragment reads without conflicts
    static_assert(H1 % 32 == 0 && H2 % 32 == 0 && F % 16 == 0 && NW <= 16, "tile shapes");
    uint16_t *h1_l = reinterpret_cast<uint16_t *>(rows_lds);     // [32][LD1]
    uint16_t *d2_l = h1_l + 32 * LD1;                            // [32][LD2]
    float *part_l = reinterpret_cast<float *>(d2_l + 32 * LD2);  // [NW][32] per-wavefront partial dot products
    float *dy_l = part_l + NW * 32;                              // [32]
    float *tile_l = dy_l + 32;                                   // [NW][32][33] output-layer terms
    const int tid = FRESH ? crew_thread() : threadIdx.x, lane = tid & 63, h = lane >> 5, c = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // this wavefront owns a tile of the first / second layer
    const bool has1 = H1 == 32 * NW || wave < H1 / 32, has2 = H2 == 32 * NW || wave < H2 / 32;
    const int col = 32 * wave + c;

    // Everything the first two layers need is requested before anything is waited for, the features (by the caller), which are
    // needed first, in front: a load at the start of a launch goes past the L2 and takes more than a microsecond, and a bias
    // rounded where it arrived held the features back by as much again.
    Fragments<F> w1f;
    Fragments<H1> w2f;
    uint32_t nought = 0;
    asm("" : "+v"(nought)); // (a load of one address for all lanes would be waited for where it stands, to become a scalar)
    const int col1 = min(col, H1 - 1), col2 = min(col, H2 - 1);
    const float bias1_raw = fresh_float<FRESH>(a.theta, 4 * col1, 4 * (uint32_t)a.off_b1), bias2_raw = fresh_float<FRESH>(a.theta, 4 * col2, 4 * (uint32_t)a.off_b2);
    const float w3_raw = fresh_float<FRESH>(a.theta, 4 * col2, 4 * (uint32_t)a.off_w3), bias3_raw = fresh_float<FRESH>(a.theta, nought, 4 * (uint32_t)a.off_b3);
    if (has1) fetch_fragments<F, FRESH>(a.w1t, wave, lane, w1f);
    // (A compute unit's loads start one after the other, 16 cycles a kilobyte, and a wavefront stands still until its own have:
    // with the loads at hand in the L2, most of the second layer's are requested behind the first one's product.)
    constexpr int AT_ONCE = FRESH ? 4 : Fragments<H1>::EARLY;
    if (has2) fetch_fragments<H1, FRESH>(a.w2t, wave, lane, w2f, 0, AT_ONCE);
    __builtin_amdgcn_sched_barrier(0);
    const float target = ready(tid);
    const float bias1 = through_bf16(bias1_raw), bias2 = through_bf16(bias2_raw), w3 = through_bf16(w3_raw), bias3 = through_bf16(bias3_raw);

    // ---- h1 = relu(x W1 + b1), bf16
    if (has1) {
        const f32x16 acc = row_tile_product<F, LDX, FRESH>(x_l, a.w1t, wave, w1f, lane);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = fmaxf(acc[4 * g + e] + bias1, 0.0f);
            const uint32_t lo = bf16_two(v[0], v[1]), hi = bf16_two(v[2], v[3]);
            put_rows4(h1_l, LD1, d_row(4 * g, h), col, lo, hi);
            store_rows4(a.h1t, col, a.padded, r0 + d_row(4 * g, h), lo, hi);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (has2) fetch_fragments<H1, FRESH>(a.w2t, wave, lane, w2f, AT_ONCE);
    lds_barrier();

    // ---- h2 = relu(h1 W2 + b2), fp32; the partial output-layer products of this wavefront's columns
    float h2v[16], dot[16];
#pragma unroll
    for (int q = 0; q < 16; ++q) h2v[q] = dot[q] = 0.0f;
    if (has2) {
        const f32x16 acc = row_tile_product<H1, LD1, FRESH>(h1_l, a.w2t, wave, w2f, lane);
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            h2v[q] = fmaxf(acc[q] + bias2, 0.0f);
            a.h2[(int64_t)(r0 + d_row(q, h)) * H2 + col] = h2v[q];
            dot[q] = h2v[q] * w3;
        }
    }
    // the fragments of W2 for the way back are under way while the output layer is summed
    Fragments<H2> wbf;
    if (!FRESH && has1) fetch_fragments<H2, FRESH>(a.w2, wave, lane, wbf);
    // Output layer: every lane holds 16 row-terms of one column.  The wavefront's 32 x 32 terms go through LDS so
    // that a lane can add up 16 columns of one row (fixed order); the two halves of the row meet in one exchange.
    {
        float *terms = tile_l + wave * (32 * 33); // [32 rows][33]: rows a bank apart
#pragma unroll
        for (int q = 0; q < 16; ++q) terms[d_row(q, h) * 33 + c] = dot[q];
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // the wavefront reads back what its own lanes wrote
        float sum = 0.0f;
#pragma unroll
        for (int j = 0; j < 16; ++j) sum += terms[c * 33 + 16 * h + j];
        sum += __shfl_xor(sum, 32);
        if (h == 0) part_l[wave * 32 + c] = sum;
    }
    lds_barrier();
    if (tid < 32) {
        float pred = part_l[tid];
#pragma unroll
        for (int w = 1; w < H2 / 32; ++w) pred += part_l[w * 32 + tid];
        pred += bias3;
        const float d = pred - target;
        const bool counts = r0 + tid < a.rows;
        const float g = counts ? 2.0f * d / (target * (float)a.rows) : 0.0f;
        a.dy[r0 + tid] = g;
        a.lterm[r0 + tid] = counts ? d * d / target : 0.0f;
        dy_l[tid] = g;
    }
    if (FRESH && has1) fetch_fragments<H2, FRESH>(a.w2, wave, lane, wbf, 0, Fragments<H2>::EARLY / 2);
    lds_barrier();
    // ---- d2 = dy w3 where h2 > 0, bf16
    if (has2) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const float4 dy = *reinterpret_cast<const float4 *>(dy_l + d_row(4 * g, h)); // four neighbouring rows
            const float row_dy[4] = {dy.x, dy.y, dy.z, dy.w};
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = h2v[4 * g + e] > 0.0f ? row_dy[e] * w3 : 0.0f;
            const uint32_t lo = bf16_two(v[0], v[1]), hi = bf16_two(v[2], v[3]);
            put_rows4(d2_l, LD2, d_row(4 * g, h), col, lo, hi);
            store_rows4(a.d2t, col, a.padded, r0 + d_row(4 * g, h), lo, hi);
        }
    }
    __builtin_amdgcn_sched_barrier(0);
    if (FRESH && has1) fetch_fragments<H2, FRESH>(a.w2, wave, lane, wbf, Fragments<H2>::EARLY / 2);
    lds_barrier();
    // ---- d1 = (d2 W2^T) where h1 > 0, bf16
    if (has1) {
        const f32x16 acc = row_tile_product<H2, LD2, FRESH>(d2_l, a.w2, wave, wbf, lane);
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            float v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) // a ReLU output: positive unless its bits are zero
                v[e] = h1_l[d_row(4 * g + e, h) * LD1 + col] != 0 ? acc[4 * g + e] : 0.0f;
            store_rows4(a.d1t, col, a.padded, r0 + d_row(4 * g, h), bf16_two(v[0], v[1]), bf16_two(v[2], v[3]));
        }
    }
}

template <int F, int H1, int H2, bool FEAT_BF16>
__global__ __launch_bounds__((H1 > H2 ? H1 : H2) * 2) void step_rows_kernel(StepArgs a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char rows_lds[];
    const int r0 = blockIdx.x * 32; // first minibatch row of this block
    constexpr int NT = (H1 > H2 ? H1 : H2) * 2;
    if (blockIdx.x == gridDim.x - 1) {
        if (threadIdx.x == 0) *a.scales = step_scales(a, a.step_in_call);
        return;
    }
    uint16_t *x_l = reinterpret_cast<uint16_t *>(rows_lds + rows_lds_bytes<F, H1, H2>());
    RowInputs<F, FEAT_BF16, NT> inputs;
    inputs.request(a, a.row0, r0, threadIdx.x);
    step_rows<F, H1, H2, false>(a, x_l, r0, rows_lds, [&](int tid) {
        inputs.keep(a, tid, x_l, a.xt, r0);
        lds_barrier();
        return inputs.y;
    });
}

// --------------------------------------------------------------------------------------------- weights kernel

// The output layer: [gW3 ; gb3] = [h2 ; 1]^T dy by 256 threads a block, 16 columns: four neighbouring ones and every 64th row a
// thread, rows in order, the threads' sums then along the wavefront and over the four of them.  The first block also takes b3.
// (With a 64th of the rows together, a wavefront's loads lay hundreds of kilobytes apart and met in a few channels: the longest blocks
// of the weights kernel, 60 us against 39.7 at 16384 rows of 256 units, 402 against 344 at 65536 of 512.)
template <int H2, bool FRESH>
struct OutputBlock {
    static constexpr int BLOCKS = H2 / 16, ROW_SETS = 64;
    const StepArgs &a;
    int tid, block;
    float w, m, v; // of column tid % 32; behind the columns, b3

    __device__ __forceinline__ OutputBlock(const StepArgs &args, int block_, int tid_) : a(args), tid(tid_), block(block_) {}

    __device__ __forceinline__ bool updates() const { return tid < 16 + (block == 0); }
    __device__ __forceinline__ uint64_t parameter() const { return (tid & 31) < 16 ? a.off_w3 + block * 16 + (tid & 31) : a.off_b3; }

    __device__ __forceinline__ void request()
    {
        const uint32_t at = 4u * (uint32_t)parameter(), P4 = 4u * (uint32_t)a.P;
        w = fresh_float<FRESH>(a.theta, at, 0);
        m = fresh_float<FRESH>(a.theta, at, P4);
        v = fresh_float<FRESH>(a.theta, at, 2 * P4);
    }

    __device__ __forceinline__ void sum(float *psum) // [4 wavefronts][17]
    {
        constexpr int AHEAD = FRESH ? 8 : 16; // rows under way together
        const int lane = tid & 63, per = a.padded / ROW_SETS;
        const uint32_t first = (uint32_t)(tid >> 2), at = 4u * (first * H2 + (uint32_t)(block * 16 + 4 * (lane & 3)));
        float sums[5] = {0.0f, 0.0f, 0.0f, 0.0f, 0.0f};
        for (int r = 0; r < per; r += AHEAD) {
            float4 h[AHEAD];
            float d[AHEAD];
            // (2^21 rows of 512 units are 2^32 bytes: the base is 64 bits wide)
            const float *h2 = a.h2 + (uint64_t)r * (ROW_SETS * H2), *dy = a.dy + (uint64_t)r * ROW_SETS;
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                const uint32_t row = 4u * ROW_SETS * (uint32_t)min(u, per - 1 - r);
                h[u] = __builtin_bit_cast(float4, fresh_16<FRESH>(h2, at, H2 * row));
                d[u] = fresh_float<FRESH>(dy, 4u * first, row);
            }
#pragma unroll
            for (int u = 0; u < AHEAD; ++u) {
                if (r + u < per) {
                    sums[0] = fmaf(h[u].x, d[u], sums[0]);
                    sums[1] = fmaf(h[u].y, d[u], sums[1]);
                    sums[2] = fmaf(h[u].z, d[u], sums[2]);
                    sums[3] = fmaf(h[u].w, d[u], sums[3]);
                    sums[4] += d[u];
                }
            }
        }
#pragma unroll
        for (int e = 0; e < 5; ++e) {
#pragma unroll
            for (uint32_t off = 4; off < 64; off <<= 1) sums[e] += __uint_as_float(lane_exchange(__float_as_uint(sums[e]), off));
        }
        if (lane < 4) {
#pragma unroll
            for (int e = 0; e < 4; ++e) psum[(tid >> 6) * 17 + 4 * lane + e] = sums[e];
            if (lane == 0) psum[(tid >> 6) * 17 + 16] = sums[4];
        }
    }

    __device__ __forceinline__ void update(const float *psum, AdamScales scales) const
    {
        if (!updates()) return;
        const float g = (psum[tid] + psum[17 + tid]) + (psum[34 + tid] + psum[51 + tid]);
        (void)adam_one(a.theta, a.P, parameter(), w, m, v, g, a.beta1, a.beta2, a.eps, scales);
    }
};

constexpr int LOSS_PARTS = 4; // the loss's sum, as many as a block of the weights kernel has wavefronts

// Blocks, in order: the 32 x 32 tiles of W2 (H1/32 x H2/32), the tiles of W1 (F/32 x H1/32), then blocks of 16
// columns of the output layer.  A tile block: C[m][n] = sum_r A[m][r] B[r][n] with both operands stored row-index
// fastest (A = h1^T or x^T, B = d2^T or d1^T); wavefront w sums rows [w B/4, (w+1) B/4) -- its fragments fetched
// eight k-steps at a time, and the Adam state of the four parameters each thread will update fetched before that --
// the four partial tiles are added in wavefront order through LDS, then 256 threads update four parameters each.
// The blocks of the first tile row also sum the columns of B: the bias gradient.
template <int F, int H1, int H2>
__global__ __launch_bounds__(256) void step_weights_kernel(StepArgs a)
{
    __shared__ float part[4][16][64];   // partial tiles of the four wavefronts
    __shared__ float colsum[4][32];     // partial bias gradients
    __shared__ double loss[LOSS_PARTS];
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, c = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int TILES_W2 = (H1 / 32) * (H2 / 32), TILES_W1 = (F / 32) * (H1 / 32);
    const int B = a.padded;
    const bool bad = *a.bad != 0;
    const AdamScales scales = *a.scales;
    int block = blockIdx.x;
    if (block < TILES_W2 + TILES_W1) {
        const bool second = block < TILES_W2; // a tile of W2, else of W1
        if (!second) block -= TILES_W2;
        const int nt = second ? H2 / 32 : H1 / 32;
        const int mt = block / nt, ntile = block % nt;
        // the parameters this thread updates: tile elements (q = 4 wave + e, lane) -> row d_row(q, h), column c
        uint64_t at[4];
        float w_old[4], m_old[4], v_old[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int m = 32 * mt + d_row(4 * wave + e, h), n = 32 * ntile + c;
            at[e] = second ? a.off_w2 + (uint64_t)m * H2 + n : a.off_w1 + (uint64_t)m * H1 + n;
            w_old[e] = a.theta[at[e]];
            m_old[e] = a.theta[a.P + at[e]];
            v_old[e] = a.theta[2 * a.P + at[e]];
        }
        // ... and the bias that it updates, in the first tile row
        const uint64_t bias_at = (second ? a.off_b2 : a.off_b1) + 32 * ntile + (tid & 31);
        float bias_w = 0.0f, bias_m = 0.0f, bias_v = 0.0f;
        if (mt == 0) {
            bias_w = a.theta[bias_at];
            bias_m = a.theta[a.P + bias_at];
            bias_v = a.theta[2 * a.P + bias_at];
        }
        // A rows: hidden unit (W2) or feature (W1) 32 mt + m; B columns: unit 32 ntile + n
        const uint16_t *bsrc = (second ? a.d2t : a.d1t) + (int64_t)ntile * 32 * B + lane * 8; // fragments of tile ntile
        const uint16_t *asrc = (second ? a.h1t : a.xt) + (int64_t)mt * 32 * B + lane * 8;
        const int k0 = wave * (B / 64), k1 = k0 + B / 64; // k-steps of 16 rows
        f32x16 acc;
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[q] = 0.0f;
        float bsum = 0.0f;
        for (int kb = k0; kb < k1; kb += 8) {
            bf16x8 av[8], bv[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int ks = kb + u < k1 ? kb + u : k1 - 1; // clamped: every load stays inside the operands
                bv[u] = *reinterpret_cast<const bf16x8 *>(bsrc + (int64_t)512 * place(ntile, ks, B));
                av[u] = *reinterpret_cast<const bf16x8 *>(asrc + (int64_t)512 * place(mt, ks, B));
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                if (kb + u < k1) {
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[u], bv[u], acc, 0, 0, 0);
                    if (mt == 0) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) bsum += (float)bv[u][e];
                    }
                }
            }
        }
#pragma unroll
        for (int q = 0; q < 16; ++q) part[wave][q][lane] = acc[q];
        if (mt == 0) {
            bsum += __shfl_xor(bsum, 32); // the two halves of a wavefront hold different rows of the same column
            if (h == 0) colsum[wave][c] = bsum;
        }
        lds_barrier();
        if (bad) return;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int q = 4 * wave + e;
            const float g = ((part[0][q][lane] + part[1][q][lane]) + part[2][q][lane]) + part[3][q][lane];
            const int m = 32 * mt + d_row(q, h), n = 32 * ntile + c;
            const float w = adam_one(a.theta, a.P, at[e], w_old[e], m_old[e], v_old[e], g, a.beta1, a.beta2, a.eps, scales);
            const uint16_t wb = (uint16_t)bf16_two(w, w);
            if (second) {
                a.w2[frag_at(m, n, H2)] = wb;
                a.w2t[frag_at(n, m, H1)] = wb;
            } else {
                a.w1t[frag_at(n, m, F)] = wb;
            }
        }
        if (mt == 0 && tid < 32) {
            const float g = ((colsum[0][tid] + colsum[1][tid]) + colsum[2][tid]) + colsum[3][tid];
            (void)adam_one(a.theta, a.P, bias_at, bias_w, bias_m, bias_v, g, a.beta1, a.beta2, a.eps, scales);
        }
        return;
    }
    // ---- output layer
    OutputBlock<H2, false> out(a, block - (TILES_W2 + TILES_W1), tid);
    out.request();
    out.sum(&part[0][0][0]);
    const bool report = a.report_loss && out.block == 0;
    if (report) {
        const double s = loss_part<LOSS_PARTS>(a.lterm, a.rows, wave, lane);
        if (lane == 0) loss[wave] = s;
    }
    lds_barrier();
    if (bad) return;
    out.update(&part[0][0][0], scales);
    if (report && tid == 64) *a.loss_out = (float)((((loss[0] + loss[1]) + loss[2]) + loss[3]) / a.rows);
}

// ------------------------------------------------------------------------------------- all steps in one launch
//
// The same steps by a crew: rows, a barrier, weights, a barrier, twelve wavefronts a member (so that a lane has 168 registers).
// Blocks of 32 rows as above.  Of the weights, eight wavefronts take 32 x 64 parameters of W2, four to a tile of 32 x 32; the other four a
// tile of W1, or 16 columns of the output layer.  All sums are those of the two launches, in their order: the same bits.
constexpr int CREW_THREADS = 768, CREW_MAIN = 512;

template <int F, int H1, int H2>
struct CrewCut {
    static constexpr int MAIN = (H1 / 32) * (H2 / 64), TILES_W1 = (F / 32) * (H1 / 32), SIDE = TILES_W1 + OutputBlock<H2, true>::BLOCKS;
    static constexpr int ITEMS = MAIN > SIDE ? MAIN : SIDE;
    // LDS of the weights' phase, in floats: partial tiles and column sums, behind them the turned copies' wavefronts
    static constexpr int PARTS = 4 * 16 * 64, SUMS = 4 * 32, TURN = 3 * (PARTS + SUMS); // of three tiles
    static constexpr size_t WEIGHTS_LDS = TURN * sizeof(float) + CREW_THREADS / 64 * 8 * 34 * sizeof(uint16_t);
    static_assert(WEIGHTS_LDS % 16 == 0 && rows_lds_bytes<F, H1, H2>() % 16 == 0, "aligned");
    static constexpr size_t PHASE_LDS = rows_lds_bytes<F, H1, H2>() > WEIGHTS_LDS ? rows_lds_bytes<F, H1, H2>() : WEIGHTS_LDS;
    static constexpr size_t LDS = PHASE_LDS + 2 * (32 * (F + 8) * sizeof(uint16_t) + 32 * sizeof(float)) + sizeof(AdamScales); // and two minibatches' rows
    static constexpr int ROW_WAVES = (H1 > H2 ? H1 : H2) / 32;
    static_assert(H1 % 32 == 0 && H2 % 64 == 0 && F % 32 == 0, "whole tiles");
};

// The sums over the minibatch of a tile of 32 x 32 parameters, (mt, nt), by four wavefronts, a quarter of the rows each.
// inputs, deltas: both in fragment order.  parts: [4][16][64], sums: [4][32]
__device__ __forceinline__ void crew_sums(const StepArgs &a, const uint16_t *inputs, const uint16_t *deltas, int mt, int nt, int quarter, int lane,
                                          float *parts, float *sums)
{
    constexpr int AHEAD = 8; // k-steps of 16 rows under way together
    const int B = a.padded, k0 = quarter * (B / 64), k1 = k0 + B / 64;
    f32x16 acc;
    float bsum = 0.0f;
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[q] = 0.0f;
    for (int kb = k0; kb < k1; kb += AHEAD) {
        crew_i32x4 av[AHEAD], bv[AHEAD];
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            const int ks = min(kb + u, k1 - 1); // clamped: every load stays inside the operands
            av[u] = fresh_16<true>(inputs, 16u * lane, 2u * (uint32_t)(mt * 32 * B + 512 * place(mt, ks, B)));
            bv[u] = fresh_16<true>(deltas, 16u * lane, 2u * (uint32_t)(nt * 32 * B + 512 * place(nt, ks, B)));
        }
#pragma unroll
        for (int u = 0; u < AHEAD; ++u) {
            if (kb + u < k1) {
                const bf16x8 b = __builtin_bit_cast(bf16x8, bv[u]);
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, av[u]), b, acc, 0, 0, 0);
                if (mt == 0) {
#pragma unroll
                    for (int e = 0; e < 8; ++e) bsum += (float)b[e];
                }
            }
        }
    }
#pragma unroll
    for (int q = 0; q < 16; ++q) parts[(quarter * 16 + q) * 64 + lane] = acc[q];
    if (mt == 0) {
        bsum += __shfl_xor(bsum, 32); // the two halves of a wavefront hold different rows of the same column
        if (lane < 32) sums[quarter * 32 + lane] = bsum;
    }
}

// The update of a tile of 32 x 32 parameters of a layer with N outputs by four wavefronts, eight rows each, a lane four
// neighbours in a row.
template <int N>
struct CrewTile {
    const StepArgs &a;
    int lane, eight, mt, nt;
    uint32_t mine, bias_mine; // byte offset in theta of this thread's parameters, of its bias
    float4 w, m, v;
    float bias_w, bias_m, bias_v;

    __device__ __forceinline__ CrewTile(const StepArgs &args, uint64_t off_w, uint64_t off_b, int mt_, int nt_, int eight_, int lane_)
        : a(args), lane(lane_), eight(eight_), mt(mt_), nt(nt_)
    {
        mine = 4u * ((uint32_t)off_w + (uint32_t)(row() * N + col()));
        bias_mine = 4u * ((uint32_t)off_b + (uint32_t)(32 * nt + (lane & 31)));
    }

    __device__ __forceinline__ int row() const { return 32 * mt + 8 * eight + (lane >> 3); }
    __device__ __forceinline__ int col() const { return 32 * nt + 4 * (lane & 7); }
    __device__ __forceinline__ bool has_bias() const { return mt == 0 && eight == 0; }

    __device__ __forceinline__ void request() // (past the L1: as the crew grows, a tile passes from member to member)
    {
        const uint32_t P4 = 4u * (uint32_t)a.P;
        const __amdgpu_buffer_rsrc_t theta = crew_buffer(a.theta);
        w = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(theta, mine, 0, CREW_SC1));
        m = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(theta, mine, P4, CREW_SC1));
        v = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(theta, mine, 2 * P4, CREW_SC1));
        if (has_bias()) {
            bias_w = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(theta, bias_mine, 0, CREW_SC1));
            bias_m = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(theta, bias_mine, P4, CREW_SC1));
            bias_v = __int_as_float(__builtin_amdgcn_raw_buffer_load_b32(theta, bias_mine, 2 * P4, CREW_SC1));
        }
    }

    // parts, sums: the tile's from crew_sums.  Returns the new weights of this thread as bf16.
    __device__ __forceinline__ uint2 update(const float *parts, const float *sums, AdamScales scales) const
    {
        const uint32_t P4 = 4u * (uint32_t)a.P;
        const __amdgpu_buffer_rsrc_t theta = crew_buffer(a.theta);
        const float *at = parts + (4 * eight + (lane >> 3 & 3)) * 64 + (lane & 32) + 4 * (lane & 7);
        float4 g = *reinterpret_cast<const float4 *>(at);
#pragma unroll
        for (int p = 1; p < 4; ++p) {
            const float4 more = *reinterpret_cast<const float4 *>(at + p * 16 * 64);
            g = make_float4(g.x + more.x, g.y + more.y, g.z + more.z, g.w + more.w);
        }
        const AdamNext n[4] = {adam_next(w.x, m.x, v.x, g.x, a.beta1, a.beta2, a.eps, scales), adam_next(w.y, m.y, v.y, g.y, a.beta1, a.beta2, a.eps, scales),
                               adam_next(w.z, m.z, v.z, g.z, a.beta1, a.beta2, a.eps, scales), adam_next(w.w, m.w, v.w, g.w, a.beta1, a.beta2, a.eps, scales)};
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(crew_i32x4, make_float4(n[0].w, n[1].w, n[2].w, n[3].w)), theta, mine, 0, 0);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(crew_i32x4, make_float4(n[0].m, n[1].m, n[2].m, n[3].m)), theta, mine, P4, 0);
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(crew_i32x4, make_float4(n[0].v, n[1].v, n[2].v, n[3].v)), theta, mine, 2 * P4, 0);
        if (has_bias() && lane < 32) {
            float sum = sums[lane];
#pragma unroll
            for (int p = 1; p < 4; ++p) sum += sums[p * 32 + lane];
            const AdamNext b = adam_next(bias_w, bias_m, bias_v, sum, a.beta1, a.beta2, a.eps, scales);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(b.w), theta, bias_mine, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(b.m), theta, bias_mine, P4, 0);
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_int(b.v), theta, bias_mine, 2 * P4, 0);
        }
        return make_uint2(bf16_two(n[0].w, n[1].w), bf16_two(n[2].w, n[3].w));
    }

    // ... and into the copy whose reduction runs over the rows: eight of them together, in `turn`, 8 x 34 values of this
    // wavefront's (stores of two bytes each took a microsecond to arrive)
    __device__ __forceinline__ void store_turned(uint16_t *matrix, int rows, uint2 next, uint16_t *turn) const
    {
        uint32_t *at = reinterpret_cast<uint32_t *>(turn + (lane >> 3) * 34 + 4 * (lane & 7));
        at[0] = next.x;
        at[1] = next.y;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); // the wavefront reads back what its own lanes wrote
        const uint16_t *from = turn + (lane >> 5) * 4 * 34 + (lane & 31);
        const uint32_t lo = from[0] | (uint32_t)from[34] << 16, hi = from[68] | (uint32_t)from[102] << 16;
        store_rows4(matrix, 32 * nt + (lane & 31), rows, 32 * mt + 8 * eight + 4 * (lane >> 5), lo, hi);
    }
};

template <int F, int H1, int H2, bool FEAT_BF16>
__global__ __launch_bounds__(CREW_THREADS) void steps_crew_kernel(StepArgs a, CrewState *state, unsigned pick, int n_steps, uint64_t n_pairs, unsigned at_once)
{
    using Cut = CrewCut<F, H1, H2>;
    extern __shared__ __attribute__((aligned(16))) unsigned char crew_lds[];
    if (blockIdx.x % CREW_DIES != pick || *a.bad != 0) return;
    Crew crew;
    const int first_step = crew.join(state, at_once, reinterpret_cast<uint32_t *>(crew_lds));
    if (first_step < 0) return;
    __syncthreads(); // (the words are read)
    const int rank = (int)crew.rank, row_blocks = a.padded / 32;
    // The rows' features and labels come from memory, some 2 us: the wavefronts that have no tile of a layer fetch those of a
    // member's first rows of a step during the step before, into the other half of the buffers.
    constexpr int STAGERS = CREW_THREADS - CREW_MAIN;
    using Inputs = RowInputs<F, FEAT_BF16, STAGERS>;
    auto x_of = [&](int step) { return reinterpret_cast<uint16_t *>(crew_lds + Cut::PHASE_LDS) + (step & 1) * (32 * Inputs::LDX); };
    AdamScales *scales_of = reinterpret_cast<AdamScales *>(crew_lds + Cut::LDS - sizeof(AdamScales)); // of the step, in its weights' phase
    auto y_of = [&](int step) { return reinterpret_cast<float *>(crew_lds + Cut::PHASE_LDS + 2 * 32 * Inputs::LDX * sizeof(uint16_t)) + (step & 1) * 32; };
    auto xt_of = [&](int step) { return a.xt + (step & 1) * ((uint64_t)F * a.padded); };
    auto stage = [&](int step, uint64_t row0, int r0, int t) { // by threads t = 0 .. STAGERS - 1
        Inputs inputs;
        inputs.request(a, row0, r0, t);
        inputs.keep(a, t, x_of(step), xt_of(step), r0);
        if (t < 32) y_of(step)[t] = inputs.y;
    };
    uint64_t row0 = first_step == 0 ? 0 : (uint32_t)first_step % ((uint32_t)n_pairs / (uint32_t)a.rows) * (uint32_t)a.rows;
    if (rank < row_blocks) {
        const int t = crew_thread() - CREW_MAIN;
        if (t >= 0) stage(first_step, row0, 32 * rank, t);
        lds_barrier();
    }
    int step = first_step, members = (int)crew.size;
    auto one_step = [&] __attribute__((always_inline)) {
        uint64_t next_row0 = row0 + a.rows;
        if (next_row0 == n_pairs) next_row0 = 0;
        for (int i = rank; i < row_blocks; i += members) {
            const int tid = crew_thread(), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
            if (i != rank) { // (a small crew)
                lds_barrier();
                if (wave >= CREW_MAIN / 64) stage(step, row0, 32 * i, tid - CREW_MAIN);
                lds_barrier();
            }
            if (wave < Cut::ROW_WAVES) {
                step_rows<F, H1, H2, true>(a, x_of(step), 32 * i, crew_lds, [&](int tid) { return y_of(step)[tid & 31]; });
            } else {
                if (wave >= CREW_MAIN / 64 && i == rank && step + 1 < n_steps) stage(step + 1, next_row0, 32 * i, tid - CREW_MAIN);
                for (int barrier = 0; barrier < ROWS_BARRIERS; ++barrier) lds_barrier();
            }
        }
        if (crew_thread() == CREW_MAIN) *scales_of = step_scales(a, step);
        row0 = next_row0;
        const bool last = step + 1 == n_steps;
        auto adam = [&] { return *scales_of; };
        // (what a member updates is requested in front of the barrier)
        auto together = [&](int base) {
            if (base == 0) {
                crew.arrive();
                crew.meet();
            }
        };
        for (int base = 0; base < Cut::ITEMS; base += members) {
            const int tid = crew_thread(), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
            const int main_item = base + rank, side_item = base + members - 1 - rank; // (the side's first members have no rows)
            const int third = wave >> 2, quarter = wave & 3; // the tiles of W2, then the side
            float *parts = reinterpret_cast<float *>(crew_lds) + third * (Cut::PARTS + Cut::SUMS), *sums = parts + Cut::PARTS;
            uint16_t *turn = reinterpret_cast<uint16_t *>(reinterpret_cast<float *>(crew_lds) + Cut::TURN) + wave * (8 * 34);
            if (third < 2) {
                const int mt = main_item / (H2 / 64), nt = main_item % (H2 / 64) * 2 + third;
                CrewTile<H2> tile(a, a.off_w2, a.off_b2, mt, nt, quarter, lane);
                const bool mine = main_item < Cut::MAIN;
                if (mine) tile.request();
                together(base);
                if (mine) crew_sums(a, a.h1t, a.d2t, mt, nt, quarter, lane, parts, sums);
                lds_barrier();
                if (mine) {
                    const uint2 next = tile.update(parts, sums, adam());
                    *reinterpret_cast<uint2 *>(a.w2 + frag_at(tile.row(), tile.col(), H2)) = next;
                    tile.store_turned(a.w2t, H1, next, turn);
                }
            } else if (side_item < Cut::TILES_W1) {
                const int mt = side_item / (H1 / 32), nt = side_item % (H1 / 32);
                CrewTile<H1> tile(a, a.off_w1, a.off_b1, mt, nt, quarter, lane);
                tile.request();
                together(base);
                crew_sums(a, xt_of(step), a.d1t, mt, nt, quarter, lane, parts, sums);
                lds_barrier();
                tile.store_turned(a.w1t, F, tile.update(parts, sums, adam()), turn);
            } else {
                OutputBlock<H2, true> out(a, side_item - Cut::TILES_W1, tid - CREW_MAIN);
                const bool mine = side_item < Cut::SIDE;
                if (mine) out.request();
                together(base);
                if (mine) out.sum(parts);
                lds_barrier();
                if (mine) {
                    out.update(parts, adam());
                    if (last && out.block == 0 && wave == CREW_THREADS / 64 - 1) {
                        const double s = loss_sum_fresh<LOSS_PARTS>(a.lterm, a.rows, lane);
                        if (lane == 0) *a.loss_out = (float)(s / a.rows);
                    }
                }
            }
            if (members < Cut::ITEMS) lds_barrier(); // (the LDS is free again)
        }
        if (!last) {
            crew.summon(step + 1);
            crew.arrive();
            crew.meet();
        }
    };
    // (two loops, so that what follows from the number of members is worked out where it changes, not in every step)
    for (; step < n_steps; members = (int)crew.size)
        do one_step();
        while (++step < n_steps && !crew.grown());
    crew.dismiss();
}

// The last block: labels; the others: bf16 copies of W1 and W2 in the fragment order the rows kernel multiplies with
__global__ __launch_bounds__(1024) void step_prepare_kernel(const float *theta, uint64_t off_w1, uint64_t off_w2, int F, int H1, int H2,
                                                            uint16_t *w1t, uint16_t *w2t, uint16_t *w2, const float *energy,
                                                            uint64_t n_pairs, float *y, RefitScalars *sc, CrewState *crew)
{
    if (blockIdx.x == gridDim.x - 1) {
        crew_clear(crew);
        make_labels(energy, n_pairs, y, sc);
        return;
    }
    const int n1 = F * H1, n2 = H1 * H2;
    for (int e = blockIdx.x * 1024 + threadIdx.x; e < n1 + n2; e += (gridDim.x - 1) * 1024) {
        if (e < n1) {
            const int f = e / H1, i = e % H1;
            w1t[frag_at(i, f, F)] = bf16_bits(theta[off_w1 + e]);
        } else {
            const int x = e - n1, i = x / H2, j = x % H2;
            const uint16_t b = bf16_bits(theta[off_w2 + x]);
            w2[frag_at(i, j, H2)] = b;
            w2t[frag_at(j, i, H1)] = b;
        }
    }
}

// A crew's launch and roll take as long as three steps gain; with more blocks of rows than members the chip's other dies are missed.
// us a call (replayed graphs), two launches a step / crew:
//   64-256-256, 512 rows: 2 steps 44.0 / 45.6, 3 steps 56.8 / 56.8, 4 steps 75.7 / 72.7, 8 steps 127 / 114; 1024 rows: 84.1 / 83.8, 144 / 138
//   64-128-128, 64 rows: 3 steps 36.2 / 37.9, 4 steps 52.4 / 50.5, 8 steps 86.5 / 78.1; 1024: 63.2 / 58.8, 107 / 92; 1536: 71 / 76, 123 / 126; 2048: 77 / 81, 135 / 135
//   32-64-64, 64 rows: 4 steps 47.8 / 44.5, 8 steps 78.8 / 68.8; 1024: 55.0 / 53.5, 93 / 84; 2048: 66.6 / 73.1, 116 / 122
bool crew_takes(int minibatch, int n_steps) { return n_steps >= 4 && minibatch <= 32 * (int)CREW_MOST; }

template <int F, int H1, int H2>
int32_t launch_steps(const eck_model *m, StepArgs a, int32_t feat_dtype, int32_t n_steps, uint64_t n_pairs, float *loss_scalar,
                     CrewSize crew, hipStream_t st)
{
    constexpr int NW = (H1 > H2 ? H1 : H2) / 32;
    constexpr size_t lds = rows_lds_bytes<F, H1, H2>() + 32 * (F + 8) * sizeof(uint16_t);
    auto rows_kernel = feat_dtype == ECK_BF16 ? step_rows_kernel<F, H1, H2, true> : step_rows_kernel<F, H1, H2, false>;
    auto weights_kernel = step_weights_kernel<F, H1, H2>;
    ECK_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(rows_kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)lds));
    const int B = a.rows;
    if constexpr (H1 <= 256 && H2 <= 256) {
        if (crew_takes(a.padded, n_steps)) {
            constexpr size_t crew_lds = CrewCut<F, H1, H2>::LDS;
            auto crew_kernel = feat_dtype == ECK_BF16 ? steps_crew_kernel<F, H1, H2, true> : steps_crew_kernel<F, H1, H2, false>;
            ECK_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(crew_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)crew_lds));
            CrewState *state = reinterpret_cast<CrewState *>(a.scales);
            a.loss_out = loss_scalar;
            hipLaunchKernelGGL(crew_kernel, dim3(CREW_DIES * crew.candidates), dim3(CREW_THREADS), crew_lds, st, a, state, crew_pick(state), n_steps, n_pairs,
                               crew.at_once);
            ECK_HIP_TRY(hipGetLastError());
            return ECK_OK;
        }
    }
    const uint64_t nb = n_pairs / (uint64_t)B;
    const unsigned weight_blocks = (H1 / 32) * (H2 / 32) + (F / 32) * (H1 / 32) + OutputBlock<H2, false>::BLOCKS;
    for (int s = 0; s < n_steps; ++s) {
        a.row0 = ((uint64_t)s % nb) * (uint64_t)B;
        a.step_in_call = s;
        a.report_loss = s == n_steps - 1;
        a.loss_out = loss_scalar;
        hipLaunchKernelGGL(rows_kernel, dim3(a.padded / 32 + 1), dim3(NW * 64), lds, st, a);
        hipLaunchKernelGGL(weights_kernel, dim3(weight_blocks), dim3(256), 0, st, a);
    }
    (void)m;
    ECK_HIP_TRY(hipGetLastError());
    return ECK_OK;
}

} // namespace

static int padded_rows(int minibatch) { return (minibatch + 63) / 64 * 64; }

uint64_t eck::refit_features_bytes(const eck_model *m, int minibatch) { return 4ull * m->widths[0] * padded_rows(minibatch); }

uint64_t eck::refit_workspace_bytes(const eck_model *m, int minibatch)
{
    auto align = [](uint64_t v) { return (v + 255) & ~255ull; };
    const uint64_t F = m->widths[0], H1 = m->widths[1], H2 = m->widths[2], B = (uint64_t)padded_rows(minibatch);
    return align(F * H1 * 2) + align(H1 * H2 * 2) * 2 + align(H1 * B * 2) * 2 + align(H2 * B * 2) + align(B * H2 * 4) +
           align(B * 4) * 2 + 256;
}

// the buffers of a call's steps in its workspace, and the model's own
static StepArgs step_buffers(const eck_model *m, int32_t minibatch, void *ws)
{
    auto align = [](uint64_t v) { return (v + 255) & ~255ull; };
    const uint64_t F = m->widths[0], H1 = m->widths[1], H2 = m->widths[2], B = (uint64_t)padded_rows(minibatch);
    char *p = static_cast<char *>(ws);
    auto take = [&](uint64_t bytes) {
        char *at = p;
        p += align(bytes);
        return at;
    };
    StepArgs a = {};
    a.rows = minibatch;
    a.padded = padded_rows(minibatch);
    a.theta = m->d_state;
    a.P = m->n_params;
    a.off_w1 = m->off_w[0];
    a.off_b1 = m->off_b[0];
    a.off_w2 = m->off_w[1];
    a.off_b2 = m->off_b[1];
    a.off_w3 = m->off_w[2];
    a.off_b3 = m->off_b[2];
    a.w1t = reinterpret_cast<uint16_t *>(take(F * H1 * 2));
    a.w2t = reinterpret_cast<uint16_t *>(take(H1 * H2 * 2));
    a.w2 = reinterpret_cast<uint16_t *>(take(H1 * H2 * 2));
    a.h1t = reinterpret_cast<uint16_t *>(take(H1 * B * 2));
    a.d1t = reinterpret_cast<uint16_t *>(take(H1 * B * 2));
    a.d2t = reinterpret_cast<uint16_t *>(take(H2 * B * 2));
    a.h2 = reinterpret_cast<float *>(take(B * H2 * 4));
    a.dy = reinterpret_cast<float *>(take(B * 4));
    a.lterm = reinterpret_cast<float *>(take(B * 4));
    a.scales = reinterpret_cast<AdamScales *>(take(sizeof(CrewState)));
    return a;
}

// a crew's words lie where the two launches leave Adam's scales
static CrewState *crew_state(const StepArgs &a) { return reinterpret_cast<CrewState *>(a.scales); }

int32_t eck::refit_begin(const eck_model *m, const float *energy, uint64_t n_pairs, float *y, RefitScalars *sc, int32_t minibatch, void *ws,
                         hipStream_t st)
{
    const StepArgs a = step_buffers(m, minibatch, ws);
    const int F = m->widths[0], H1 = m->widths[1], H2 = m->widths[2], blocks = (F * H1 + H1 * H2 + 1023) / 1024;
    hipLaunchKernelGGL(step_prepare_kernel, dim3((blocks < 256 ? blocks : 256) + 1), dim3(1024), 0, st, a.theta, a.off_w1, a.off_w2, F, H1, H2,
                       a.w1t, a.w2t, a.w2, energy, n_pairs, y, sc, crew_state(a));
    ECK_HIP_TRY(hipGetLastError());
    return ECK_OK;
}

int32_t eck::refit_steps(const eck_model *m, const void *feat, int32_t feat_dtype, uint64_t ld, const float *y, uint64_t n_pairs,
                         int32_t n_steps, int32_t minibatch, float lr, float beta1, float beta2, float eps,
                         const uint32_t *bad_flag, float *loss_scalar, void *features, void *ws, CrewSize crew, hipStream_t st)
{
    const int F = m->widths[0], H1 = m->widths[1], H2 = m->widths[2];
    StepArgs a = step_buffers(m, minibatch, ws);
    a.xt = static_cast<uint16_t *>(features);
    const uint64_t elem = feat_dtype == ECK_BF16 ? 2 : 4;
    a.aligned = a.padded == minibatch && ld * elem % 16 == 0 && ((uintptr_t)feat & 15) == 0;
    a.feat = feat;
    a.ld = ld;
    a.y = y;
    a.bad = bad_flag;
    a.lr = lr;
    a.beta1 = beta1;
    a.beta2 = beta2;
    a.eps = eps;
    if (F == 64 && H1 == 512 && H2 == 512) return launch_steps<64, 512, 512>(m, a, feat_dtype, n_steps, n_pairs, loss_scalar, crew, st);
    if (F == 64 && H1 == 256 && H2 == 256) return launch_steps<64, 256, 256>(m, a, feat_dtype, n_steps, n_pairs, loss_scalar, crew, st);
    if (F == 64 && H1 == 128 && H2 == 128) return launch_steps<64, 128, 128>(m, a, feat_dtype, n_steps, n_pairs, loss_scalar, crew, st);
    if (F == 32 && H1 == 64 && H2 == 64) return launch_steps<32, 64, 64>(m, a, feat_dtype, n_steps, n_pairs, loss_scalar, crew, st);
    return ECK_EUNSUPPORTED;
}
