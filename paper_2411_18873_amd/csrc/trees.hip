// The cost model in the form the paper itself uses (Sec. 5.4 "Approach"): an ensemble of regression trees
// built one after another by gradient boosting on the weighted squared error of Eq. (1); the prediction is
// the sum of the trees' outputs.  HIP, gfx950.
//
// Trees are complete binary trees of a fixed depth d stored level by level: node j tests
// "x[feature_j] < threshold_j"; true -> node 2j+1, false (also NaN) -> node 2j+2; after d tests the walk stands
// on node (2^d - 1) + leaf.  A node that does not split has threshold +inf.
//
// Scoring: one candidate per lane.  A block stages the features of its candidates and a chunk of trees in LDS
// and walks eight trees at a time per lane (eight independent chains of dependent LDS reads); leaf values are
// added in fp32 in tree order, so the result does not depend on how trees are chunked, shared or interleaved.
//
// Boosting: gradient statistics are rounded to integers of resolution 2^-20 and summed with integer atomics,
// so every histogram, and with it every split decision, is independent of the order of execution; gains are
// evaluated in fp64 from those integers.
#include "eck_internal.h"
#include "lanes.h"
#include "refit_labels.h"

#include <atomic>
#include <new>
#include <type_traits>

using namespace eck;

struct eck_trees {
    int32_t n_feat, depth, capacity, n_trees;
    float base;
    uint8_t *d_feat = nullptr; // [capacity][2^d - 1]
    float *d_thr = nullptr;    // [capacity][2^d - 1]
    float *d_leaf = nullptr;   // [capacity][2^d]
    uint32_t *d_word = nullptr; // [capacity][2^d] the nodes as the scoring kernel reads them for bfloat16 features, from 1 on
    int device = -1;
};

namespace {

constexpr int BLOCK = 256;
constexpr int BINS = 256;
constexpr int WALKS = 8; // trees walked at the same time by one lane
constexpr double FIX = 1048576.0; // 2^20

__device__ __forceinline__ float feature_value(const void *feat, int is_bf16, uint64_t at)
{
    if (is_bf16) return __uint_as_float((uint32_t)reinterpret_cast<const uint16_t *>(feat)[at] << 16);
    return reinterpret_cast<const float *>(feat)[at];
}

// ------------------------------------------------------------------------------------------------ scoring

// A node as it sits in LDS.  With fp32 features: the threshold's bits and the byte offset of the feature's row.  With
// bfloat16 features one word, which halves the node reads and puts the nodes of a tree of depth six in different banks:
// the feature's number plus one in the lower half, and above it sixteen bits chosen such that the word, read as a float,
// is a threshold of the same comparison: for every bfloat16 x (infinities, both zeros and NaN included)
//   x < t  <=>  x < word.
// The lower half is never zero, so a positive word lies strictly between two neighbouring bfloat16 values, above the one
// in its upper half, and a negative one below it; hence the largest bfloat16 below a positive t, and the truncation of a
// negative one; +inf becomes the largest finite value (all but +inf and NaN are below the word), a zero of either sign
// becomes -0 (the negative values, denormals too, are below it), and -inf and NaN give a negative NaN (nothing is;
// x minus it is a positive one: the subtraction negates its second operand).
__device__ __forceinline__ uint32_t bf16_node(float t, uint32_t feature)
{
    const uint32_t u = __float_as_uint(t);
    uint32_t upper;
    if (t != t || u == 0xFF800000u) upper = 0xFF80u;
    else if ((u << 1) == 0) upper = 0x8000u;
    else if (u >> 31) upper = u >> 16;
    else upper = (u - 1) >> 16; // the largest bfloat16 below t: truncation unless t is one itself
    return upper << 16 | (feature + 1);
}

__host__ __device__ inline uint32_t tree_lds_bytes(int depth, bool feat_bf16)
{
    return (feat_bf16 ? (1u << depth) * 4u : ((1u << depth) - 1u) * 8u) + (1u << depth) * 4u;
}

// The scoring kernel's numbering for bfloat16 features: children of i are 2i + 1 when x < t and 2i when not, the other
// way round than the arrays', so that the sign of x - t is the step.  Node i (numbered from 1) of the arrays sits at
__device__ __forceinline__ uint32_t mirrored(uint32_t i) { return i ? (3u << (31 - __clz((int)i))) - 1u - i : 0u; }

// An ensemble handed over: the arrays, and the words of its nodes (one launch instead of a copy per array).  Also, with the
// arrays in place already, just the words.
__global__ void tree_set_kernel(const uint8_t *nf, const float *nt, const float *leaf, int n_feat, int depth, int n_trees,
                                uint8_t *nf_out, float *nt_out, float *leaf_out, uint32_t *words)
{
    const uint32_t nodes = (1u << depth) - 1u, e = blockIdx.x * blockDim.x + threadIdx.x, t = e >> depth, i = e & nodes;
    if (t >= (uint32_t)n_trees) return;
    const uint64_t from = (uint64_t)t * nodes + (i ? i - 1 : 0); // word 0 is not read
    const uint8_t f = nf[from];
    const float thr = nt[from];
    words[(t << depth) + mirrored(i)] = bf16_node(thr, min((uint32_t)f, (uint32_t)n_feat - 1u));
    if (nf_out && i) {
        nf_out[from] = f;
        nt_out[from] = thr;
    }
    if (leaf_out) leaf_out[e] = leaf[e];
}

// An ensemble handed back: n_nodes nodes and n_leaves leaves, of which there are more
__global__ __launch_bounds__(256) void tree_get_kernel(const uint8_t *nf, const float *nt, const float *leaf, uint64_t n_nodes, uint64_t n_leaves,
                                                       uint8_t *nf_out, float *nt_out, float *leaf_out)
{
    const uint64_t step = (uint64_t)gridDim.x * 256;
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < n_leaves; i += step) {
        leaf_out[i] = leaf[i];
        if (i >= n_nodes) continue;
        nf_out[i] = nf[i];
        nt_out[i] = nt[i];
    }
}

// C candidates per block, its trees shared between S groups of C threads.
//   S == 1: every thread walks all trees of its candidate.  bfloat16 features stay that: a wavefront takes every second
//     of 128 candidates, so that its lanes read different words, hence banks, of whatever rows they are at.
//   S > 1, for few candidates: group s walks every S-th set of eight trees, the leaves meet in LDS and the first group
//     adds them up.  Features are kept as floats.
// What bounds it: vector instructions, then the two dependent LDS reads of a visit (node, feature value).  A visit takes
// four: the node's address, the feature value's (mask and join), the difference to the threshold, and the step, which
// shifts the difference's sign into the node's number.  Measured, 100 trees of depth 6 on 2^20 candidates: 136-138 us (62 %
// of the cycles issue vector instructions, 69 % of those a unit is busy, two fifths move LDS data; no bank conflicts); with eight-byte nodes, a
// compare into a mask and an add with carry 156 us.  Without effect: more wavefronts (trees shared by two groups over
// 256 or 384 candidates, 158-165 us), the first two levels' nodes through the scalar cache; nodes gathered from the L1
// instead of the LDS: 184 us for a quarter of them.
template <bool FEAT_BF16, int C, int S>
__global__ __launch_bounds__(C *S) void tree_score_kernel(const uint8_t *__restrict__ node_feat,
                                                          const float *__restrict__ node_thr,
                                                          const float *__restrict__ leaf,
                                                          const uint32_t *__restrict__ words, int n_feat, int depth,
                                                          int n_trees, int chunk_trees, float base,
                                                          const void *__restrict__ feat, uint64_t ld, uint64_t n,
                                                          float *__restrict__ out, uint32_t n_tiles)
{
    constexpr int T = C * S;
    constexpr bool HALF = FEAT_BF16 && S == 1;
    using Elem = typename std::conditional<FEAT_BF16, uint16_t, float>::type; // in memory
    using Cell = typename std::conditional<HALF, uint16_t, float>::type;      // in LDS
    using Node = typename std::conditional<FEAT_BF16, uint32_t, uint2>::type;
    constexpr uint32_t ROW = C * sizeof(Cell); // bytes from one feature's row to the next
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const uint32_t nodes = (1u << depth) - 1u, leaves = 1u << depth;
    // Nodes from one tree to the next in LDS.  With bfloat16 features a tree's leaves follow its words, so that after the
    // last level i is the leaf's place, too.
    const uint32_t stride = FEAT_BF16 ? 2 * leaves : nodes;
    Cell *x_lds = reinterpret_cast<Cell *>(lds);                                   // [n_feat][C]
    Node *node_lds = reinterpret_cast<Node *>(lds + (size_t)n_feat * ROW);         // [chunk][nodes]
    float *leaf_lds = reinterpret_cast<float *>(node_lds + (size_t)chunk_trees * stride); // fp32: [chunk][leaves]
    float *val_lds = leaf_lds + (FEAT_BF16 ? 0 : (size_t)chunk_trees * leaves);    // S > 1: [chunk][C] leaves reached
    // (the compiler cannot tell that a wavefront has one slot: left to itself it works a walk's tree addresses out per lane)
    const int tid = threadIdx.x, within = tid % C, slot = S == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid / C);
    // this thread's candidate in the tile
    const int mine = HALF ? 2 * ((within >> 7) * 64 + (within & 63)) + ((within >> 6) & 1) : within;
    // where the dynamic LDS starts within the workgroup's allocation (the hand-written loads below take raw LDS
    // addresses)
    const uint32_t lds_base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)lds;
    const uint32_t lane_at = lds_base + (uint32_t)mine * sizeof(Cell); // of this candidate in row 0
    // HALF: where a word's feature value is: the row's offset bits of the word, joined by the lane's place, in one
    // instruction -- right as long as the dynamic part starts at zero, which the launcher makes sure of; else the row's
    // number times ROW plus that
    constexpr uint32_t ROW_BITS = 0xFFFFu & ~(ROW - 1u);
    auto place_of = [&](uint32_t word) {
        uint32_t at;
        if constexpr (HALF) asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(at) : "v"(word), "s"(ROW_BITS), "v"(lane_at));
        else asm("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(at) : "v"(word), "s"(ROW), "v"(lane_at - ROW));
        return at;
    };
    const Elem *feat_e = reinterpret_cast<const Elem *>(feat);
    auto cell_of = [](Elem v) {
        if constexpr (FEAT_BF16 && !HALF) return __uint_as_float((uint32_t)v << 16);
        else return (Cell)v;
    };

    typedef uint32_t u32x4 __attribute__((ext_vector_type(4), aligned(2))); // (rows of odd length start anywhere)
    typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
    // HALF: a NaN counts as not below any threshold, but a negative one would look negative to the walks: it is staged as a
    // positive one.  Features hardly ever hold one, so whole rows are only looked at, and rewritten when there is one.
    constexpr uint32_t BF16_INF = 0x7F80u;
    auto positive_nans = [](uint32_t two) {
        if ((two & 0x7FFFu) > BF16_INF) two &= ~0x8000u;
        if ((two & 0x7FFF0000u) > BF16_INF << 16) two &= ~0x80000000u;
        return two;
    };

    // sixteen bytes moved towards the first by 1 to 127 bits
    auto shifted = [](u32x4 v, uint32_t bits) {
        uint64_t lo = (uint64_t)v[1] << 32 | v[0], hi = (uint64_t)v[3] << 32 | v[2];
        if (bits >= 64) lo = hi >> (bits - 64), hi = 0;
        else lo = lo >> bits | hi << (64 - bits), hi >>= bits;
        return u32x4{(uint32_t)lo, (uint32_t)(lo >> 32), (uint32_t)hi, (uint32_t)(hi >> 32)};
    };

    uint32_t upper[WALKS]; // HALF: feature values as they arrive, in the upper halves
#pragma unroll
    for (int w = 0; w < WALKS; ++w) upper[w] = 0;

    for (uint32_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
        const uint64_t first_cand = (uint64_t)tile * C;
        __syncthreads(); // the previous tile's walks are over
        if (n >= 16 / sizeof(Elem)) {
            // Sixteen bytes of a row per load; up to eight loads of a thread under way together, fewer for the last ones.
            // Columns past n are not read: in the last tile a piece that would reach past them is read from further left and
            // shifted.
            constexpr int PER = 16 / sizeof(Elem), LOADS = C / PER; // elements per load, loads per row
            const bool inside = first_cand + C <= n;
            const uint64_t last = n - PER;
            const int pieces = n_feat * LOADS;
            auto stage = [&](auto loads, auto whole, int e0) {
                constexpr int N = decltype(loads)::value;
                constexpr bool WHOLE = decltype(whole)::value; // every piece of the tile lies inside
                u32x4 v[N];
#pragma unroll
                for (int k = 0; k < N; ++k) {
                    const int e = min(e0 + k * T + tid, pieces - 1);
                    const uint64_t col = first_cand + (e % LOADS) * PER;
                    v[k] = *reinterpret_cast<const u32x4 *>(feat_e + (uint64_t)(e / LOADS) * ld + (WHOLE || col < last ? col : last));
                }
                if constexpr (!WHOLE) {
#pragma unroll
                    for (int k = 0; k < N; ++k) {
                        const uint64_t col = first_cand + min(e0 + k * T + tid, pieces - 1) % LOADS * PER;
                        if (col > last && col < last + PER) v[k] = shifted(v[k], (uint32_t)(col - last) * (8 * sizeof(Elem)));
                    }
                }
                if constexpr (HALF) {
                    u16x2 most = {0, 0};
#pragma unroll
                    for (int k = 0; k < N; ++k)
#pragma unroll
                        for (int q = 0; q < 4; ++q) most = __builtin_elementwise_max(most, __builtin_bit_cast(u16x2, v[k][q] & 0x7FFF7FFFu));
                    if (__any(most[0] > BF16_INF || most[1] > BF16_INF)) {
#pragma unroll
                        for (int k = 0; k < N; ++k)
#pragma unroll
                            for (int q = 0; q < 4; ++q) v[k][q] = positive_nans(v[k][q]);
                    }
                }
#pragma unroll
                for (int k = 0; k < N; ++k) { // (past the end: the last piece again, where it already is)
                    const int e = min(e0 + k * T + tid, pieces - 1);
                    Cell *to = x_lds + e * PER;
                    if constexpr (sizeof(Cell) == sizeof(Elem)) {
                        *reinterpret_cast<uint4 *>(to) = make_uint4(v[k][0], v[k][1], v[k][2], v[k][3]);
                    } else {
                        float4 *f = reinterpret_cast<float4 *>(to);
                        f[0] = make_float4(__uint_as_float(v[k][0] << 16), __uint_as_float(v[k][0] & 0xFFFF0000u),
                                           __uint_as_float(v[k][1] << 16), __uint_as_float(v[k][1] & 0xFFFF0000u));
                        f[1] = make_float4(__uint_as_float(v[k][2] << 16), __uint_as_float(v[k][2] & 0xFFFF0000u),
                                           __uint_as_float(v[k][3] << 16), __uint_as_float(v[k][3] & 0xFFFF0000u));
                    }
                }
            };
            auto stage_all = [&](auto whole) {
                int e0 = 0;
                for (; pieces - e0 > 2 * T; e0 += 8 * T) stage(std::integral_constant<int, 8>(), whole, e0);
                for (; e0 < pieces; e0 += T) stage(std::integral_constant<int, 1>(), whole, e0);
            };
            if (inside) stage_all(std::true_type());
            else stage_all(std::false_type());
        } else { // rows of less than sixteen bytes
            // Sixteen rows at a time, every load and store unconditional (a lane beyond n re-reads the last candidate,
            // a row beyond n_feat the last row, and stores that same value where it already is): with a condition on
            // either side the compiler waits for each load right before its store, one round trip per feature.
            const uint64_t col = first_cand + within < n ? first_cand + within : n - 1;
            for (int f0 = slot * 16; f0 < n_feat; f0 += 16 * S) {
                Elem v[16];
#pragma unroll
                for (int k = 0; k < 16; ++k) v[k] = feat_e[(uint64_t)min(f0 + k, n_feat - 1) * ld + col];
                if constexpr (HALF) {
#pragma unroll
                    for (int k = 0; k < 16; ++k) v[k] = (uint16_t)positive_nans(v[k]);
                }
#pragma unroll
                for (int k = 0; k < 16; ++k) x_lds[min(f0 + k, n_feat - 1) * C + within] = cell_of(v[k]);
            }
        }
        float acc = base;
        for (int t0 = 0; t0 < n_trees; t0 += chunk_trees) {
            const int in_chunk = min(chunk_trees, n_trees - t0);
            __syncthreads(); // features staged / previous chunk consumed
            // Four loads of a thread and array under way together (past the end: the last element again, where it already
            // is): with one at a time a chunk takes a round trip to memory per T elements.
            constexpr int AHEAD = 4;
            if constexpr (FEAT_BF16) {
                const uint32_t count = (uint32_t)in_chunk * leaves;
                for (uint32_t e0 = tid; e0 < count; e0 += AHEAD * T) {
                    float value[AHEAD];
                    uint32_t word[AHEAD];
#pragma unroll
                    for (int k = 0; k < AHEAD; ++k) {
                        const uint64_t from = (uint64_t)t0 * leaves + min(e0 + k * T, count - 1);
                        value[k] = leaf[from];
                        word[k] = words[from];
                    }
#pragma unroll
                    for (int k = 0; k < AHEAD; ++k) {
                        const uint32_t e = min(e0 + k * T, count - 1), to = (e >> depth) * stride, i = e & nodes;
                        // HALF: the row's byte offset in place of its number; below it, outside the mask, a one that keeps
                        // the lower half from being zero
                        if (HALF) word[k] = (word[k] & 0xFFFF0000u) | (((word[k] & 0xFFFFu) - 1u) * ROW + 1u);
                        node_lds[to + i] = word[k];
                        node_lds[to + leaves + (nodes - i)] = __float_as_uint(value[k]); // (mirrored, like the nodes)
                    }
                }
            } else {
                const uint32_t n_leaves = (uint32_t)in_chunk * leaves, n_nodes = (uint32_t)in_chunk * nodes;
                for (uint32_t e0 = tid; e0 < n_leaves; e0 += AHEAD * T) {
                    float value[AHEAD], thr[AHEAD];
                    uint8_t f[AHEAD];
#pragma unroll
                    for (int k = 0; k < AHEAD; ++k) { // (a tree has one leaf more than nodes)
                        const uint64_t node = (uint64_t)t0 * nodes + min(e0 + k * T, n_nodes - 1);
                        value[k] = leaf[(uint64_t)t0 * leaves + min(e0 + k * T, n_leaves - 1)];
                        thr[k] = node_thr[node];
                        f[k] = node_feat[node];
                    }
#pragma unroll
                    for (int k = 0; k < AHEAD; ++k) {
                        leaf_lds[min(e0 + k * T, n_leaves - 1)] = value[k];
                        node_lds[min(e0 + k * T, n_nodes - 1)] =
                            make_uint2(__float_as_uint(thr[k]), min((uint32_t)f[k], (uint32_t)n_feat - 1u) * ROW);
                    }
                }
            }
            __syncthreads();
            // One set of walks, from tree t of the chunk on.  Nodes are numbered from 1 here, children of i: 2i and 2i + 1.
            // Bytes from the nodes (and with fp32 features, the leaves) of the set's first tree to those of each walk's: past
            // the chunk's end the last tree is walked again.
            uint32_t node_off[WALKS], leaf_off[WALKS];
#pragma unroll
            for (int w = 0; w < WALKS; ++w) {
                node_off[w] = w * stride * sizeof(Node);
                leaf_off[w] = w * leaves * 4;
            }
            auto walk = [&](auto walks, int t) {
                constexpr int W = decltype(walks)::value;
                if (t + W > in_chunk) {
#pragma unroll
                    for (int w = 0; w < W; ++w) {
                        node_off[w] = min(w, in_chunk - 1 - t) * stride * sizeof(Node);
                        leaf_off[w] = min(w, in_chunk - 1 - t) * leaves * 4;
                    }
                }
                uint32_t i[W];
#pragma unroll
                for (int w = 0; w < W; ++w) i[w] = 1;
                const unsigned char *first_node = reinterpret_cast<const unsigned char *>(node_lds + (size_t)t * stride - (FEAT_BF16 ? 0 : 1));
                const unsigned char *first_leaf = reinterpret_cast<const unsigned char *>(leaf_lds + (size_t)t * leaves - leaves);
                auto node_at = [&](int w) { return reinterpret_cast<const Node *>(first_node + node_off[w])[i[w]]; };
                // feature values at `at`, and one step of every walk
                auto read_x = [&](const uint32_t(&at)[W], float(&x)[W]) {
                    if constexpr (HALF && W == 8) {
                        // A bfloat16 is the upper half of the float of the same value.  The load below writes
                        // only the upper half of its destination, whose lower half is zero from the start and
                        // stays so: the float arrives ready, without a shift.  The compiler has no such load, so
                        // it is issued here, and waited for in the same statement: the compiler takes the eight
                        // registers for written when it ends.
                        asm volatile("ds_read_u16_d16_hi %0, %8\n\t"
                                     "ds_read_u16_d16_hi %1, %9\n\t"
                                     "ds_read_u16_d16_hi %2, %10\n\t"
                                     "ds_read_u16_d16_hi %3, %11\n\t"
                                     "ds_read_u16_d16_hi %4, %12\n\t"
                                     "ds_read_u16_d16_hi %5, %13\n\t"
                                     "ds_read_u16_d16_hi %6, %14\n\t"
                                     "ds_read_u16_d16_hi %7, %15\n\t"
                                     "s_waitcnt lgkmcnt(0)"
                                     : "+&v"(upper[0]), "+&v"(upper[1]), "+&v"(upper[2]), "+&v"(upper[3]), "+&v"(upper[4]),
                                       "+&v"(upper[5]), "+&v"(upper[6]), "+&v"(upper[7])
                                     : "v"(at[0]), "v"(at[1]), "v"(at[2]), "v"(at[3]), "v"(at[4]), "v"(at[5]), "v"(at[6]),
                                       "v"(at[7]));
#pragma unroll
                        for (int w = 0; w < W; ++w) x[w] = __uint_as_float(upper[w]);
                    } else {
#pragma unroll
                        for (int w = 0; w < W; ++w) {
                            const Cell v = *reinterpret_cast<const Cell *>(lds + (at[w] - lds_base));
                            if constexpr (HALF) x[w] = __uint_as_float((uint32_t)v << 16);
                            else x[w] = v;
                        }
                    }
                };
                auto step = [&](const float(&x)[W], const float(&thr)[W]) {
                    if constexpr (HALF) {
                        // i <- 2i + sign(x - t): x < t exactly when the difference is negative (denormals are kept, no
                        // NaN here is negative)
#pragma unroll
                        for (int w = 0; w < W; ++w) i[w] = __builtin_amdgcn_alignbit(i[w], __float_as_uint(x[w] - thr[w]), 31u);
                    } else if constexpr (W == 8) {
                        // i <- i + i + (outcome of the comparison): a compare into a scalar mask and an add with that
                        // mask as carry-in, written out because the compiler makes three instructions of it.  Four walks
                        // per statement keep the compares four instructions ahead of the adds that read their masks.
#define ECK_STEP(CMP)                                                                                                          \
    asm(CMP " %4, %8, %12\n\t" CMP " %5, %9, %13\n\t" CMP " %6, %10, %14\n\t" CMP " %7, %11, %15\n\t"                            \
            "v_addc_co_u32_e64 %0, %4, %0, %0, %4\n\t"                                                                         \
            "v_addc_co_u32_e64 %1, %5, %1, %1, %5\n\t"                                                                         \
            "v_addc_co_u32_e64 %2, %6, %2, %2, %6\n\t"                                                                         \
            "v_addc_co_u32_e64 %3, %7, %3, %3, %7"                                                                             \
        : "+v"(i[w]), "+v"(i[w + 1]), "+v"(i[w + 2]), "+v"(i[w + 3]), "=&s"(m0), "=&s"(m1), "=&s"(m2), "=&s"(m3)               \
        : "v"(x[w]), "v"(x[w + 1]), "v"(x[w + 2]), "v"(x[w + 3]), "v"(thr[w]), "v"(thr[w + 1]), "v"(thr[w + 2]), "v"(thr[w + 3]))
#pragma unroll
                        for (int w = 0; w < W; w += 4) {
                            unsigned long long m0, m1, m2, m3;
                            if constexpr (FEAT_BF16) ECK_STEP("v_cmp_lt_f32_e64"); // (mirrored)
                            else ECK_STEP("v_cmp_nlt_f32_e64");
                        }
#undef ECK_STEP
                    } else {
#pragma unroll
                        for (int w = 0; w < W; ++w) i[w] = 2 * i[w] + ((x[w] < thr[w]) == FEAT_BF16 ? 1u : 0u);
                    }
                };
                float x[W], thr[W];
                uint32_t at[W];
                for (int l = 0; l < depth; ++l) {
                    Node nd[W];
#pragma unroll
                    for (int w = 0; w < W; ++w) nd[w] = node_at(w);
#pragma unroll
                    for (int w = 0; w < W; ++w) {
                        if constexpr (FEAT_BF16) {
                            thr[w] = __uint_as_float(nd[w]);
                            at[w] = place_of(nd[w]);
                        } else {
                            thr[w] = __uint_as_float(nd[w].x);
                            at[w] = lane_at + nd[w].y;
                        }
                    }
                    read_x(at, x);
                    step(x, thr);
                }
                float v[W]; // i in [2^d, 2^(d+1))
#pragma unroll
                for (int w = 0; w < W; ++w) {
                    if constexpr (FEAT_BF16) v[w] = __uint_as_float(node_at(w));
                    else v[w] = reinterpret_cast<const float *>(first_leaf + leaf_off[w])[i[w]];
                }
                if constexpr (S == 1) {
                    if (t + W <= in_chunk) {
#pragma unroll
                        for (int w = 0; w < W; ++w) acc = acc + v[w]; // tree order
                    } else {
#pragma unroll
                        for (int w = 0; w < W; ++w) acc = t + w < in_chunk ? acc + v[w] : acc;
                    }
                } else {
#pragma unroll
                    for (int w = 0; w < W; ++w) val_lds[(size_t)(t + w) * C + within] = v[w];
                }
            };
            for (int t = slot * WALKS; t < in_chunk; t += S * WALKS) {
                // (the last one or two trees of a chunk alone: six walks of eight would be for nothing)
                if (in_chunk - t > 2) walk(std::integral_constant<int, WALKS>(), t);
                else walk(std::integral_constant<int, 2>(), t);
            }
            if constexpr (S > 1) {
                __syncthreads();
                if (slot == 0) {
                    int t = 0;
                    for (; t + WALKS <= in_chunk; t += WALKS) {
                        float v[WALKS];
#pragma unroll
                        for (int w = 0; w < WALKS; ++w) v[w] = val_lds[(size_t)(t + w) * C + within];
#pragma unroll
                        for (int w = 0; w < WALKS; ++w) acc = acc + v[w]; // tree order
                    }
                    for (; t < in_chunk; ++t) acc = acc + val_lds[(size_t)t * C + within];
                }
            }
        }
        if (slot == 0 && first_cand + mine < n) out[first_cand + mine] = acc;
    }
}

template <bool FEAT_BF16, int C, int S>
int32_t launch_score_as(const eck_trees *m, int n_trees, const void *feat, uint64_t ld, uint64_t n, float *out, hipStream_t st)
{
    const size_t per_tree = tree_lds_bytes(m->depth, FEAT_BF16) + (S > 1 ? C * 4 : 0);
    const size_t x_bytes = (size_t)m->n_feat * C * (FEAT_BF16 && S == 1 ? 2 : 4), lds_cu = 156 * 1024;
    const uint64_t tiles64 = (n + C - 1) / C;
    if (tiles64 > 0xFFFFFFFFull) return ECK_EUNSUPPORTED;
    // Trees per chunk.  The walks are chains of dependent LDS reads, so what counts is how many wavefronts a
    // compute unit holds: the smallest chunk (one group of simultaneous walks) beside the feature tile lets
    // the most blocks share the 160 KB; blocks per unit = what fits, chunk = what is left of a block's share.
    const size_t floor_bytes = x_bytes + S * WALKS * per_tree;
    if (floor_bytes > lds_cu) return ECK_EUNSUPPORTED;
    size_t blocks_cu = lds_cu / floor_bytes;
    if (blocks_cu > (size_t)(2048 / (C * S))) blocks_cu = 2048 / (C * S); // 2048 threads per unit
    const size_t share = lds_cu / blocks_cu;
    int chunk = (int)((share - x_bytes) / per_tree);
    chunk -= chunk % (S * WALKS);
    const int rounded = (n_trees + WALKS - 1) / WALKS * WALKS;
    if (n_trees > 0 && chunk > rounded) chunk = rounded;
    if (chunk < WALKS) chunk = WALKS;
    const size_t lds = x_bytes + (size_t)chunk * per_tree;
    int cus = 256;
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, m->device);
    const uint32_t n_tiles = (uint32_t)tiles64;
    const uint32_t want = (uint32_t)cus * (uint32_t)blocks_cu;
    const uint32_t grid = n_tiles < want ? n_tiles : want;
    auto kern = tree_score_kernel<FEAT_BF16, C, S>;
    if (FEAT_BF16 && S == 1) {
        // The walks' joined addresses need the dynamic LDS at zero, where it starts unless the kernel declares a
        // __shared__ variable; a build in which it does is refused (asked of the runtime once per kernel).
        static std::atomic<bool> starts_at_zero{false};
        if (!starts_at_zero.load(std::memory_order_relaxed)) {
            hipFuncAttributes attr;
            ECK_HIP_TRY(hipFuncGetAttributes(&attr, reinterpret_cast<const void *>(kern)));
            if (attr.sharedSizeBytes != 0) return ECK_EDEVICE;
            starts_at_zero.store(true, std::memory_order_relaxed);
        }
    }
    ECK_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize,
                                    (int)lds));
    hipLaunchKernelGGL(kern, dim3(grid), dim3(C * S), lds, st, m->d_feat, m->d_thr, m->d_leaf, m->d_word, m->n_feat, m->depth,
                       n_trees, chunk, m->base, feat, ld, n, out, n_tiles);
    ECK_HIP_TRY(hipGetLastError());
    return ECK_OK;
}

// For few candidates a block takes 64 or 128 of them and shares the trees between eight or four groups of threads: blocks of
// 512 would leave compute units idle, and every tree would wait for the one before.  Up to two such blocks per compute unit;
// with sixteen trees or fewer, where six of eight groups have none, one of 64 candidates.  Deep trees and many features leave
// no room in the LDS (depth 8 with 64 features): one group then.  us per call on 256 units, eight groups / four / one, 64
// features, depth 6, bfloat16 unless said:
//   100 trees: 1000 candidates 7.7 / 10.9 / 22, 32768 10.2 / 11.3 / 23, 65536 17.7 / 14.9 / 23, 131072 32 / 27 / 23
//   16 trees: 32768 6.3 / 6.3 / 6.5, fp32 6.8 / 6.2 / 6.2; depth 8 with 8 features 7.7 / - / 7.3, 8 trees 7.0 / - / 6.3
template <bool FEAT_BF16>
int32_t launch_score_of(const eck_trees *m, int n_trees, const void *feat, uint64_t ld, uint64_t n, float *out, hipStream_t st)
{
    // refused as ever: 256 candidates' features and eight trees with eight-byte nodes have to fit a compute unit
    const size_t lds_cu = 156 * 1024, elem = FEAT_BF16 ? 2 : 4, eight = WALKS * tree_lds_bytes(m->depth, false);
    if ((size_t)m->n_feat * 256 * elem + eight > lds_cu) return ECK_EUNSUPPORTED;
    const size_t small_tree = tree_lds_bytes(m->depth, FEAT_BF16);
    int cus = 256;
    (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, m->device);
    const uint64_t units = (uint64_t)cus;
    if (n <= (n_trees > 2 * WALKS ? 2 : 1) * 64 * units && (size_t)m->n_feat * 64 * 4 + 64 * (small_tree + 64 * 4) <= lds_cu)
        return launch_score_as<FEAT_BF16, 64, 8>(m, n_trees, feat, ld, n, out, st);
    if (n <= 2 * 128 * units && 2 * ((size_t)m->n_feat * 128 * 4 + 32 * (small_tree + 128 * 4)) <= lds_cu)
        return launch_score_as<FEAT_BF16, 128, 4>(m, n_trees, feat, ld, n, out, st);
    if constexpr (FEAT_BF16) {
        // a row's offset has to fit a word's lower half
        if (m->n_feat <= 64) return launch_score_as<true, 512, 1>(m, n_trees, feat, ld, n, out, st);
        if (m->n_feat <= 128) return launch_score_as<true, 256, 1>(m, n_trees, feat, ld, n, out, st);
        return launch_score_as<true, 128, 1>(m, n_trees, feat, ld, n, out, st);
    } else {
        // 512 candidates per block when two such blocks fit a compute unit (a staged chunk of trees then serves twice as
        // many candidates), else 256
        if (2 * ((size_t)m->n_feat * 512 * 4 + WALKS * small_tree) <= lds_cu)
            return launch_score_as<false, 512, 1>(m, n_trees, feat, ld, n, out, st);
        return launch_score_as<false, 256, 1>(m, n_trees, feat, ld, n, out, st);
    }
}

int32_t launch_score(const eck_trees *m, int n_trees, const void *feat, int32_t feat_dtype, uint64_t ld, uint64_t n,
                     float *out, hipStream_t st)
{
    return feat_dtype == ECK_BF16 ? launch_score_of<true>(m, n_trees, feat, ld, n, out, st)
                                  : launch_score_of<false>(m, n_trees, feat, ld, n, out, st);
}

// ----------------------------------------------------------------------------------------------- boosting

// feature value -> histogram bin: 256 bins of width 1/4 on [0, 64); "bin(x) <= b" is "x < (b + 1) / 4"
__device__ __forceinline__ uint32_t bin_of(float x)
{
    if (!(x >= 0.0f)) return x != x ? 255u : 0u;
    const float s = x * 4.0f;
    return s >= 255.0f ? 255u : (uint32_t)(int)s;
}

__device__ __forceinline__ long long quantise(double v)
{
    if (v > FIX) v = FIX; // |g| and h are clamped to 2^20: 2^20 samples cannot overflow 63 bits
    if (v < -FIX) v = -FIX;
    return __double2ll_rn(v * FIX);
}

// The last row of blocks: labels (its first block); the others: bins of every (feature, pair), computed once per call; row
// n_feat of the bins is 1 where feature 0 is not below +inf (the pairs that go right at a node without a split, whose test
// is "feature 0 < +inf").
__global__ __launch_bounds__(1024) void tree_prepare_kernel(const void *__restrict__ feat, int is_bf16, uint64_t ld, uint64_t n_pairs, int n_feat,
                                                            uint8_t *__restrict__ bins, const float *__restrict__ energy,
                                                            float *__restrict__ y, RefitScalars *sc)
{
    const uint64_t i = (uint64_t)blockIdx.x * 1024 + threadIdx.x;
    const int f = blockIdx.y;
    if (f == n_feat) {
        if (blockIdx.x == 0) make_labels(energy, n_pairs, y, sc);
        return;
    }
    if (i >= n_pairs) return;
    const float x = feature_value(feat, is_bf16, (uint64_t)f * ld + i);
    bins[(uint64_t)f * n_pairs + i] = (uint8_t)bin_of(x);
    if (f == 0) bins[(uint64_t)n_feat * n_pairs + i] = x < __builtin_inff() ? 0 : 1;
}

// SNR = sum y^2 / sum (p - y)^2 (the ensemble on entry)
__device__ __forceinline__ void entry_quality(const float *__restrict__ p, const float *__restrict__ y, uint64_t n, RefitScalars *sc)
{
    const float snr = signal_to_noise(p, y, n);
    if (threadIdx.x == 0 && !sc->bad) sc->snr = snr;
}

// the same, or the mean Eq.-(1) loss (which == 1)
__global__ __launch_bounds__(1024) void tree_quality_kernel(const float *__restrict__ p, const float *__restrict__ y,
                                                            uint64_t n, int which, RefitScalars *sc)
{
    if (which == 0) {
        entry_quality(p, y, n, sc);
        return;
    }
    __shared__ double scratch[512];
    double loss = 0.0;
    for (uint64_t i = threadIdx.x; i < n; i += 1024) {
        const double yi = y[i], d = (double)p[i] - yi;
        loss += d * d / yi;
    }
    loss = block_sum(loss, scratch);
    if (threadIdx.x == 0 && !sc->bad) sc->loss = (float)(loss / (double)n);
}

// first and second derivative of Eq. (1) in the prediction, as integers of resolution 2^-20
// (also: every node of the tree about to be built starts as "does not split"; the grid is at least 256 threads,
// a tree at most 255 nodes)
__global__ void tree_grad_kernel(const float *__restrict__ p, const float *__restrict__ y, uint64_t n,
                                 long long *__restrict__ gq, long long *__restrict__ hq, uint32_t *__restrict__ at,
                                 uint8_t *__restrict__ nf, float *__restrict__ nt, uint32_t nodes)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < nodes) {
        nf[i] = 0;
        nt[i] = __builtin_inff();
    }
    if (i >= n) return;
    const double yi = (double)y[i], d = (double)p[i] - yi;
    gq[i] = quantise(2.0 * d / yi);
    hq[i] = quantise(2.0 / yi);
    at[i] = 0;
}

__global__ void tree_zero_kernel(unsigned long long *ptr, uint64_t words)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < words) ptr[i] = 0;
}

// Histograms of one level: hist[node in level][feature][bin] = (sum g, sum h, count) over the pairs that
// stand on that node.  Every pair of a level hits the few cells of one feature, and device-wide atomics on
// them serialise, so a block takes one feature, a group of 8 nodes and a slice of the pairs, accumulates in
// LDS (integer atomics) and merges its non-empty cells once.
constexpr uint32_t LDS_HIST_NODES = 8;
__global__ __launch_bounds__(BLOCK) void tree_hist_lds_kernel(const uint8_t *__restrict__ bins,
                                                             const long long *__restrict__ gq,
                                                             const long long *__restrict__ hq,
                                                             const uint32_t *__restrict__ at, uint64_t n_pairs,
                                                             int n_feat, uint32_t first_node, uint32_t level_nodes,
                                                             unsigned long long *__restrict__ hist)
{
    __shared__ unsigned long long cells[LDS_HIST_NODES * BINS * 3];
    const uint32_t group0 = blockIdx.z * LDS_HIST_NODES; // first node (within the level) of this block's group
    const uint32_t in_group = min(LDS_HIST_NODES, level_nodes - group0);
    const uint32_t n_cells = in_group * BINS * 3;
    for (uint32_t c = threadIdx.x; c < n_cells; c += BLOCK) cells[c] = 0;
    __syncthreads();
    const int f = blockIdx.y;
    for (uint64_t i = (uint64_t)blockIdx.x * BLOCK + threadIdx.x; i < n_pairs; i += (uint64_t)gridDim.x * BLOCK) {
        const uint32_t r = at[i] - first_node - group0; // wraps for nodes below the group
        if (r >= in_group) continue;
        const uint32_t b = bins[(uint64_t)f * n_pairs + i];
        unsigned long long *cell = cells + ((uint64_t)r * BINS + b) * 3;
        atomicAdd(cell, (unsigned long long)gq[i]);
        atomicAdd(cell + 1, (unsigned long long)hq[i]);
        atomicAdd(cell + 2, 1ull);
    }
    __syncthreads();
    for (uint32_t c = threadIdx.x; c < n_cells; c += BLOCK) {
        const unsigned long long v = cells[c];
        if (!v) continue;
        const uint32_t r = group0 + c / (BINS * 3), rest = c % (BINS * 3);
        atomicAdd(hist + ((uint64_t)r * n_feat + f) * BINS * 3 + rest, v);
    }
}

// The split of largest gain, in two parts.  tree_split_kernel: one block per (node of the level, group of four
// features), a wavefront per feature, a lane per four consecutive bins; prefix sums over the bins by data-parallel moves.
// gain(f, b) = GL^2/(HL+lam) + GR^2/(HR+lam) - G^2/(H+lam) in fp64; the largest gain > 0 wins, ties to the
// lower feature, then the lower bin (the candidate's rank f * 256 + b breaks ties in every comparison).  The
// block leaves its best (gain, rank) in `partial`; the kernel that moves the pairs to their children compares
// the groups' results.  The fp64 divisions of a node are thus spread over up to 64 compute units instead of
// one.  Every cell read is set back to zero, so that the histogram buffer is clear again for the next level
// without a pass of its own.
struct SplitRecord { // the best split of one node on one feature, or on a group of features
    double gain;
    uint32_t rank, pad;
};
constexpr int SPLIT_FEATS = 4; // features, and wavefronts, per block

__device__ __forceinline__ bool better_split(double og, uint32_t orank, double g, uint32_t rank)
{
    return og > g || (og == g && orank < rank);
}

// The best split of a wavefront's, in every lane: the largest gain, and the lowest rank of those that have it (ranks are
// distinct but for the one of no split).  (Exchanging gain and rank together: a hundred instructions for forty.)
__device__ __forceinline__ void best_of_wave(double &gain, uint32_t &rank)
{
    const double most = wave_most(gain);
    const uint64_t have = __ballot(gain == most);
    if (__popcll(have) == 1) rank = (uint32_t)__builtin_amdgcn_readlane((int)rank, (int)__ffsll((unsigned long long)have) - 1);
    else rank = wave_least(gain == most ? rank : 0xFFFFFFFFu);
    gain = most;
}

__global__ __launch_bounds__(SPLIT_FEATS * 64) void tree_split_kernel(unsigned long long *__restrict__ hist, int n_feat,
                                                                      double lam, SplitRecord *__restrict__ partial)
{
    const uint32_t r = blockIdx.x; // node within the level
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int f = blockIdx.y * SPLIT_FEATS + wave;
    double best = 0.0;
    uint32_t best_rank = 0xFFFFFFFFu;
    if (f < n_feat) { // wave-uniform
        unsigned long long *cells = hist + (((uint64_t)r * n_feat + f) * BINS + 4 * lane) * 3;
        long long g[4], hh[4], c[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            g[q] = (long long)cells[3 * q];
            hh[q] = (long long)cells[3 * q + 1];
            c[q] = (long long)cells[3 * q + 2];
        }
#pragma unroll
        for (int q = 0; q < 12; ++q) cells[q] = 0;
#pragma unroll
        for (int q = 1; q < 4; ++q) {
            g[q] += g[q - 1];
            hh[q] += hh[q - 1];
            c[q] += c[q - 1];
        }
        // inclusive prefix of the lanes' totals; its last lane holds the node's totals (every pair of the node is
        // in exactly one bin of every feature, so each feature's histogram sums to the same G, H, N)
        long long pg = wave_prefix_sum((int64_t)g[3]), ph = wave_prefix_sum((int64_t)hh[3]), pc = wave_prefix_sum((int64_t)c[3]);
        const long long G = last_lane(pg), H = last_lane(ph), N = last_lane(pc);
        if (N > 1) {
            const double parent = (double)G * (double)G / ((double)H + lam);
            pg -= g[3];
            ph -= hh[3];
            pc -= c[3];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int b = 4 * lane + q;
                const long long GL = pg + g[q], HL = ph + hh[q], NL = pc + c[q];
                if (b >= 255 || NL == 0 || NL == N) continue;
                const long long GR = G - GL, HR = H - HL;
                const double gain = (double)GL * (double)GL / ((double)HL + lam) +
                                    (double)GR * (double)GR / ((double)HR + lam) - parent;
                const uint32_t rank = (uint32_t)f * BINS + (uint32_t)b;
                if (gain > best || (gain == best && gain > 0.0 && rank < best_rank)) {
                    best = gain;
                    best_rank = rank;
                }
            }
        }
    }
    best_of_wave(best, best_rank);
    __shared__ double s_gain[SPLIT_FEATS];
    __shared__ uint32_t s_rank[SPLIT_FEATS];
    if (lane == 0) {
        s_gain[wave] = best;
        s_rank[wave] = best_rank;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
#pragma unroll
        for (int w = 1; w < SPLIT_FEATS; ++w)
            if (better_split(s_gain[w], s_rank[w], best, best_rank)) {
                best = s_gain[w];
                best_rank = s_rank[w];
            }
        SplitRecord out;
        out.gain = best;
        out.rank = best_rank;
        out.pad = 0;
        partial[(uint64_t)r * gridDim.y + blockIdx.y] = out;
    }
}

// Move every pair to the child its node's test sends it to.  The node's test is settled here, from the feature
// groups' partial results: every pair standing on a node arrives at the same (feature, threshold) and writes it
// (equal values, so the order does not matter); nodes no pair stands on keep "does not split".
__global__ void tree_partition_kernel(const void *__restrict__ feat, int is_bf16, uint64_t ld, uint64_t n_pairs,
                                      const SplitRecord *__restrict__ partial, uint32_t groups, uint32_t first_node,
                                      const RefitScalars *sc, uint8_t *__restrict__ nf, float *__restrict__ nt,
                                      uint32_t *__restrict__ at)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_pairs) return;
    const uint32_t j = at[i];
    const SplitRecord *mine = partial + (uint64_t)(j - first_node) * groups;
    double best = 0.0;
    uint32_t best_rank = 0xFFFFFFFFu;
    for (uint32_t g = 0; g < groups; ++g) {
        const SplitRecord o = mine[g];
        if (better_split(o.gain, o.rank, best, best_rank)) {
            best = o.gain;
            best_rank = o.rank;
        }
    }
    uint32_t f = 0;
    float thr = __builtin_inff();
    if (!sc->bad && best_rank != 0xFFFFFFFFu && best > 0.0) {
        f = best_rank / BINS;
        thr = (float)((best_rank % BINS) + 1) * 0.25f;
    }
    nf[j] = (uint8_t)f;
    nt[j] = thr;
    const float x = feature_value(feat, is_bf16, (uint64_t)f * ld + i);
    at[i] = 2 * j + (x < thr ? 1u : 2u);
}

// one block: statistics of every leaf by integer atomics in LDS, then w = -eta G / (H + lam) (fp64 -> fp32)
__global__ __launch_bounds__(1024) void tree_leaf_kernel(const long long *__restrict__ gq, const long long *__restrict__ hq,
                                                         const uint32_t *__restrict__ at, uint64_t n_pairs,
                                                         uint32_t nodes, uint32_t leaves, double eta, double lam,
                                                         float *__restrict__ leaf_out, const RefitScalars *sc)
{
    __shared__ unsigned long long sg[256], sh[256], sn[256];
    for (uint32_t l = threadIdx.x; l < leaves; l += 1024) sg[l] = sh[l] = sn[l] = 0;
    __syncthreads();
    for (uint64_t i = threadIdx.x; i < n_pairs; i += 1024) {
        const uint32_t l = at[i] - nodes;
        atomicAdd(&sg[l], (unsigned long long)gq[i]);
        atomicAdd(&sh[l], (unsigned long long)hq[i]);
        atomicAdd(&sn[l], 1ull);
    }
    __syncthreads();
    for (uint32_t l = threadIdx.x; l < leaves; l += 1024) {
        const long long G = (long long)sg[l], H = (long long)sh[l];
        float w = 0.0f;
        if (sn[l] && !sc->bad) w = (float)(-eta * (double)G / ((double)H + lam));
        leaf_out[l] = w;
    }
}

__global__ void tree_advance_kernel(float *__restrict__ p, const uint32_t *__restrict__ at, const float *__restrict__ lw,
                                    uint32_t nodes, uint64_t n_pairs)
{
    const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_pairs) p[i] = p[i] + lw[at[i] - nodes];
}

__global__ void tree_finish_kernel(const RefitScalars *sc, float *snr_out, float *loss_out)
{
    if (threadIdx.x || blockIdx.x) return;
    *snr_out = sc->snr;
    *loss_out = sc->loss;
}

// ------------------------------------------------------------------- boosting, one launch per level
//
// With the few thousand pairs a search measures, a level is too little work for three launches (histograms, splits, moving
// the pairs: 7.3 + 5.6 + 4.9 us at depth 6 with 1536 pairs).  Here a level is one: a block takes one feature and up to
// sixteen nodes, first settles the level before -- reads the features' best splits of every node and works out
// where each pair stands now, the same in every block, block (0, 0) writing it down -- then builds its histograms in LDS
// and finds its best splits.  At level 0 the level before is the last one of the tree before: the pairs get their leaf's
// value, from the split's left and right sums, and their new derivatives.  So a round of depth d takes d launches.
// Every sum is an integer sum and every decision the one the three-launch path takes, so the trees are the same bits.
// What bounds it: the loads right after a launch, the LDS atomics and the scan, one after the other.  A level of 2048 pairs of 64
// features at depth 6 takes 7.0 us, a root 8.8 (9.8 and 12.4 where the pairs were requested after settling, every scan went over
// all bins and a split's sums were reduced along with its gain); eight rounds on 1536 pairs 490 and 324.

// The pairs' counts are not needed: h = 2 / y is at least 2 for every valid label, so a side is empty exactly when its
// sum of h is zero (and with an invalid label nothing splits).

constexpr int LEVEL_THREADS = 1024;
constexpr int LEVEL_SLOTS = 16;         // histograms of a block: one feature of up to sixteen nodes, a wavefront each
constexpr int LEVEL_STRIDE = BINS + 1;  // cells from one histogram to the next: equal bins of neighbours in different banks
constexpr int LEVEL_UNROLL = 4;         // pairs of a thread under way together

struct SideSums {
    long long g, h;
};

struct NodeTotals {
    SideSums all;
    SideSums odd; // the pairs whose feature 0 is not below +inf: they go right at a node that does not split
};

struct LevelArgs {
    const uint8_t *bins; // [n_feat + 1][n]: the last row is 1 where feature 0 is not below +inf
    uint32_t n;
    int n_feat, depth;
    const SplitRecord *rec_in; // of the level before: [nodes][n_feat]
    const SideSums *left_in;   // ... the sums of those splits' left sides
    const NodeTotals *tot_in;  // ... [nodes]
    SplitRecord *rec_out;
    SideSums *left_out;
    NodeTotals *tot_out;
    const uint8_t *at_in; // node within the level before, one byte per pair (not read when that level has one node)
    uint8_t *at_out;
    const float *p_in, *y;
    float *p_out;
    long long *gq, *hq;
    uint8_t *nf; // the nodes of the level before, and (level 0) the leaves of the tree before
    float *nt, *leaf;
    double eta, lam;
    RefitScalars *sc;
};

struct Settled {
    uint16_t feat[128]; // of every node of the level before: a pair goes left when its bin of feat is at most bin
    uint16_t bin[128];
    SideSums side[256]; // (a tree's last level)
    float leaf[256];
};

// The level before (`level_before`, the last one of a tree when LEAVES is set): the test of every node, and its leaves.  N
// nodes of a wavefront at a time, everything they need requested before anything waits: at the start of a launch every load
// goes past the L2.
template <bool LEAVES, int N>
__device__ __forceinline__ void settle_nodes(const LevelArgs &a, int nodes, bool write, Settled &s)
{
    const int lane = threadIdx.x & 63, waves = blockDim.x >> 6;
    const bool bad = a.sc->bad != 0;
    for (int first = threadIdx.x >> 6; first < nodes; first += N * waves) {
        double best[N];
        uint32_t best_rank[N];
        SideSums left[N]; // of this lane's best
        NodeTotals total[N];
#pragma unroll
        for (int k = 0; k < N; ++k) {
            best[k] = 0.0;
            best_rank[k] = 0xFFFFFFFFu;
            left[k] = {0, 0};
            if (LEAVES) total[k] = a.tot_in[min(first + k * waves, nodes - 1)];
        }
        for (int f = lane; f < a.n_feat; f += 64) {
            SplitRecord o[N];
            SideSums l[N];
#pragma unroll
            for (int k = 0; k < N; ++k) {
                const uint64_t at = (uint64_t)min(first + k * waves, nodes - 1) * a.n_feat + f;
                o[k] = a.rec_in[at];
                if (LEAVES) l[k] = a.left_in[at]; // (of a feature without a split: left over, not used)
            }
#pragma unroll
            for (int k = 0; k < N; ++k)
                if (better_split(o[k].gain, o[k].rank, best[k], best_rank[k])) {
                    best[k] = o[k].gain;
                    best_rank[k] = o[k].rank;
                    if (LEAVES) left[k] = l[k];
                }
        }
#pragma unroll
        for (int k = 0; k < N; ++k) {
            const int node = first + k * waves;
            best_of_wave(best[k], best_rank[k]);
            const bool split = !bad && best_rank[k] != 0xFFFFFFFFu && best[k] > 0.0;
            if (node < nodes && lane == 0) {
                s.feat[node] = (uint16_t)(split ? best_rank[k] / BINS : a.n_feat);
                s.bin[node] = (uint16_t)(split ? best_rank[k] % BINS : 0);
                if (write) {
                    a.nf[node] = (uint8_t)(split ? best_rank[k] / BINS : 0);
                    a.nt[node] = split ? (float)((best_rank[k] % BINS) + 1) * 0.25f : __builtin_inff();
                }
            }
            if (LEAVES) {
                // the winner's sums from the lane that holds them
                const int from = __builtin_amdgcn_readfirstlane((int)(best_rank[k] / BINS)) & 63;
                const SideSums all = total[k].all, odd = total[k].odd;
                SideSums side = split ? SideSums{lane_value(left[k].g, from), lane_value(left[k].h, from)}
                                      : SideSums{all.g - odd.g, all.h - odd.h};
                if (lane) side = SideSums{all.g - side.g, all.h - side.h};
                if (node < nodes && lane < 2) s.side[2 * node + lane] = side;
            }
        }
    }
}

template <bool LEAVES>
__device__ __forceinline__ void settle_level(const LevelArgs &a, int level_before, bool write, Settled &s)
{
    const int nodes = 1 << level_before, waves = blockDim.x >> 6;
    if (nodes <= waves) settle_nodes<LEAVES, 1>(a, nodes, write, s);
    else if (LEAVES || nodes <= 2 * waves) settle_nodes<LEAVES, 2>(a, nodes, write, s); // (four with their sums spill)
    else settle_nodes<LEAVES, 4>(a, nodes, write, s);
    if (LEAVES) { // (a thread per leaf: a wavefront that divides for two leaves of a node takes as long as for 64)
        __syncthreads();
        if ((int)threadIdx.x < 2 * nodes) {
            const SideSums side = s.side[threadIdx.x];
            const float v = side.h && a.sc->bad == 0 ? (float)(-a.eta * (double)side.g / ((double)side.h + a.lam)) : 0.0f;
            s.leaf[threadIdx.x] = v;
            if (write) a.leaf[threadIdx.x] = v;
        }
    }
}

// where pair i goes from node j of the level before
__device__ __forceinline__ uint32_t child_of(const LevelArgs &a, const Settled &s, uint32_t j, uint32_t i)
{
    return 2 * j + (a.bins[(uint64_t)s.feat[j] * a.n + i] <= s.bin[j] ? 0u : 1u);
}

// first_tree: level 0 of the call's first tree, nothing to settle
template <bool ROOT>
__global__ __launch_bounds__(LEVEL_THREADS) void tree_level_kernel(LevelArgs a, int level, int first_tree)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char level_lds[];
    constexpr int CELLS = LEVEL_SLOTS * LEVEL_STRIDE;
    unsigned long long *hg = reinterpret_cast<unsigned long long *>(level_lds); // [LEVEL_SLOTS][LEVEL_STRIDE]
    unsigned long long *hh = hg + CELLS;
    __shared__ Settled settled;
    __shared__ unsigned long long odd_g[LEVEL_SLOTS], odd_h[LEVEL_SLOTS];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (ROOT && (int)blockIdx.x == a.n_feat) { // the call's first launch has one more block
        entry_quality(a.p_in, a.y, a.n, a.sc);
        return;
    }
    const int f = blockIdx.x, node0 = blockIdx.y * LEVEL_SLOTS;
    const int in_group = min(LEVEL_SLOTS, (1 << level) - node0);
    // Copies of each histogram while the level has few nodes, neighbouring lanes to different ones: features take few
    // values, and atomics of a wavefront on one cell go one after the other.
    const int copies = LEVEL_SLOTS / in_group; // (a power of two, like in_group)
    const bool write = blockIdx.x == 0 && blockIdx.y == 0;
    {
        uint4 *z = reinterpret_cast<uint4 *>(level_lds);
        for (int e = tid; e < CELLS * 16 / 16; e += LEVEL_THREADS) z[e] = make_uint4(0, 0, 0, 0);
        if (tid < LEVEL_SLOTS) odd_g[tid] = odd_h[tid] = 0;
    }
    const int level_before = ROOT ? a.depth - 1 : level - 1;
    const bool settles = !ROOT || !first_tree;
    const bool placed = settles && level_before > 0; // the level before had several nodes: at_in says which
    struct Pairs {
        uint32_t i[LEVEL_UNROLL], r[LEVEL_UNROLL];
        long long g[LEVEL_UNROLL], h[LEVEL_UNROLL];
        float p[LEVEL_UNROLL], y[LEVEL_UNROLL];
        uint8_t b[LEVEL_UNROLL], odd[LEVEL_UNROLL];
    } v;
    // (a wavefront past the last pair skips the group; its lanes past it take the last pair again, not counted)
    const uint32_t wave_first = (uint32_t)__builtin_amdgcn_readfirstlane(tid);
    auto past = [&](uint32_t base, int u) { return base - tid + wave_first + u * LEVEL_THREADS >= a.n; };
    auto request = [&](uint32_t base) {
#pragma unroll
        for (int u = 0; u < LEVEL_UNROLL; ++u) {
            if (past(base, u)) break;
            v.i[u] = min(base + u * LEVEL_THREADS, a.n - 1);
            v.b[u] = a.bins[(uint64_t)f * a.n + v.i[u]];
            v.odd[u] = f == 0 ? a.bins[(uint64_t)a.n_feat * a.n + v.i[u]] : (uint8_t)0;
            v.r[u] = placed ? a.at_in[v.i[u]] : 0;
            if (ROOT) {
                v.p[u] = a.p_in[v.i[u]];
                v.y[u] = a.y[v.i[u]];
            } else {
                v.g[u] = a.gq[v.i[u]];
            }
            if (settles) v.h[u] = a.hq[v.i[u]]; // (the second derivative is the same for every tree)
        }
    };
    request(tid); // on their way while the level before is settled
    __builtin_amdgcn_sched_barrier(0);
    if (settles) settle_level<ROOT>(a, level_before, write, settled);
    __syncthreads();
    for (uint32_t base = tid; base - tid < a.n; base += LEVEL_UNROLL * LEVEL_THREADS) {
        if (base != (uint32_t)tid) request(base);
        uint8_t right[LEVEL_UNROLL]; // the bin that sends a pair to a child, all requested together
        if (settles) {
#pragma unroll
            for (int u = 0; u < LEVEL_UNROLL; ++u) {
                if (past(base, u)) break;
                right[u] = a.bins[(uint64_t)settled.feat[v.r[u]] * a.n + v.i[u]];
            }
        }
#pragma unroll
        for (int u = 0; u < LEVEL_UNROLL; ++u) {
            if (past(base, u)) break;
            const uint32_t child = settles ? 2 * v.r[u] + (right[u] <= settled.bin[v.r[u]] ? 0u : 1u) : 0u;
            if (ROOT) {
                if (settles) v.p[u] = v.p[u] + settled.leaf[child];
                const double yi = (double)v.y[u], d = (double)v.p[u] - yi;
                v.g[u] = quantise(2.0 * d / yi);
                if (!settles) v.h[u] = quantise(2.0 / yi);
                v.r[u] = 0;
                if (write) {
                    a.p_out[v.i[u]] = v.p[u];
                    a.gq[v.i[u]] = v.g[u];
                    if (!settles) a.hq[v.i[u]] = v.h[u];
                }
            } else {
                v.r[u] = child;
                if (write) a.at_out[v.i[u]] = (uint8_t)child;
            }
            const uint32_t rr = v.r[u] - (uint32_t)node0; // wraps for nodes below the group
            if (rr < (uint32_t)in_group && base + u * LEVEL_THREADS < a.n) {
                const uint32_t cell = (rr * copies + (lane & (copies - 1))) * LEVEL_STRIDE + v.b[u];
                atomicAdd(&hg[cell], (unsigned long long)v.g[u]);
                atomicAdd(&hh[cell], (unsigned long long)v.h[u]);
                if (v.odd[u]) {
                    atomicAdd(&odd_g[rr], (unsigned long long)v.g[u]);
                    atomicAdd(&odd_h[rr], (unsigned long long)v.h[u]);
                }
            }
        }
    }
    __syncthreads();
    if (copies > 1) { // into the first copy
        for (int e = tid; e < in_group * 2 * BINS; e += LEVEL_THREADS) {
            const int node = e / (2 * BINS), bin = e % BINS;
            unsigned long long *cell = (e / BINS % 2 ? hh : hg) + node * copies * LEVEL_STRIDE + bin;
            unsigned long long sum = cell[0];
            for (int k = 1; k < copies; ++k) sum += cell[k * LEVEL_STRIDE];
            cell[0] = sum;
        }
        __syncthreads();
    }
    // a wavefront per node, 64 bins at a time; gains and ties as in tree_split_kernel.  An empty bin splits like the bin
    // before it, which has the lower rank, so only bins with pairs are evaluated, and stretches without any are skipped.
    if (wave >= in_group) return;
    const unsigned long long *node_g = hg + wave * copies * LEVEL_STRIDE, *node_h = hh + wave * copies * LEVEL_STRIDE;
    long long g[4], h[4];
    uint64_t filled[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        g[q] = (long long)node_g[64 * q + lane];
        h[q] = (long long)node_h[64 * q + lane];
        filled[q] = __ballot(h[q] != 0);
    }
    double best = 0.0, parent = 0.0;
    uint32_t best_rank = 0xFFFFFFFFu;
    SideSums best_left = {0, 0}, total = {0, 0};
    auto judge = [&](SideSums left, long long in_bin, int bin) {
        if (in_bin == 0 || bin >= 255 || left.h == total.h) return;
        const SideSums right = {total.g - left.g, total.h - left.h};
        const double gain = (double)left.g * (double)left.g / ((double)left.h + a.lam) +
                            (double)right.g * (double)right.g / ((double)right.h + a.lam) - parent;
        const uint32_t rank = (uint32_t)f * BINS + (uint32_t)bin;
        if (gain > best || (gain == best && gain > 0.0 && rank < best_rank)) {
            best = gain;
            best_rank = rank;
            best_left = left;
        }
    };
    auto parent_gain = [&] { return (double)total.g * (double)total.g / ((double)total.h + a.lam); };
    // the first and the last bin with pairs (none at all: 0 and 0)
    const int lowest = filled[0] ? __builtin_ctzll(filled[0]) : filled[1] ? 64 + __builtin_ctzll(filled[1]) :
                       filled[2] ? 128 + __builtin_ctzll(filled[2]) : filled[3] ? 192 + __builtin_ctzll(filled[3]) : 0;
    const int highest = filled[3] ? 255 - __builtin_clzll(filled[3]) : filled[2] ? 191 - __builtin_clzll(filled[2]) :
                        filled[1] ? 127 - __builtin_clzll(filled[1]) : filled[0] ? 63 - __builtin_clzll(filled[0]) : 0;
    if (highest - lowest < 64) {
        // they fit one scan, from the first of them on: as a rule, for values that are logarithms of one operator's schedules
        const int bin = lowest + lane;
        const long long gb = bin < BINS ? (long long)node_g[bin] : 0, hb = bin < BINS ? (long long)node_h[bin] : 0;
        const SideSums left = {wave_prefix_sum((int64_t)gb), wave_prefix_sum((int64_t)hb)};
        total = {last_lane(left.g), last_lane(left.h)};
        parent = parent_gain();
        judge(left, hb, bin);
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            total.g += g[q];
            total.h += h[q];
        }
        total = {last_lane(wave_prefix_sum((int64_t)total.g)), last_lane(wave_prefix_sum((int64_t)total.h))};
        parent = parent_gain();
        SideSums before = {0, 0};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (!filled[q]) continue;
            const long long pg = wave_prefix_sum((int64_t)g[q]), ph = wave_prefix_sum((int64_t)h[q]);
            judge({before.g + pg, before.h + ph}, h[q], 64 * q + lane);
            before.g += last_lane(pg);
            before.h += last_lane(ph);
        }
    }
    const uint32_t own_rank = best_rank;
    best_of_wave(best, best_rank);
    const uint64_t at = (uint64_t)(node0 + wave) * a.n_feat + f;
    if (best_rank != 0xFFFFFFFFu && own_rank == best_rank) a.left_out[at] = best_left; // (ranks are distinct: one lane)
    if (lane == 0) {
        a.rec_out[at] = SplitRecord{best, best_rank, 0};
        if (f == 0) a.tot_out[node0 + wave] = NodeTotals{total, {(long long)odd_g[wave], (long long)odd_h[wave]}};
    }
}

// The words of nodes for the scoring kernel, from the arrays: slots first, first + step, ... of those of `trees` trees
__device__ __forceinline__ void make_words(const uint8_t *nf, const float *nt, int n_feat, int depth, uint32_t trees, uint32_t *words,
                                           uint32_t first, uint32_t step)
{
    const uint32_t nodes = (1u << depth) - 1u;
    for (uint32_t e = first; e < trees << depth; e += step) {
        const uint32_t t = e >> depth, i = e & nodes;
        const uint64_t from = (uint64_t)t * nodes + (i ? i - 1 : 0); // word 0 is not read
        words[(t << depth) + mirrored(i)] = bf16_node(nt[from], min((uint32_t)nf[from], (uint32_t)n_feat - 1u));
    }
}

// Block 0: the last tree's last level, the pairs' final predictions, the mean Eq.-(1) loss, the call's results, and the words of
// the last tree; the others: the words of the trees before it.  nf, nt, words: of the call's first tree.
__global__ __launch_bounds__(1024) void tree_last_kernel(LevelArgs a, int n_rounds, const uint8_t *nf, const float *nt, uint32_t *words,
                                                         float *snr_out, float *loss_out)
{
    if (blockIdx.x > 0) {
        make_words(nf, nt, a.n_feat, a.depth, n_rounds - 1, words, (blockIdx.x - 1) * 1024 + threadIdx.x, (gridDim.x - 1) * 1024);
        return;
    }
    __shared__ Settled settled;
    __shared__ double scratch[512];
    if (n_rounds) settle_level<true>(a, a.depth - 1, true, settled);
    __syncthreads();
    double sum = 0.0;
    for (uint32_t i = threadIdx.x; i < a.n; i += 1024) {
        float p = a.p_in[i];
        if (n_rounds) p = p + settled.leaf[child_of(a, settled, a.depth > 1 ? a.at_in[i] : 0u, i)];
        const double yi = a.y[i], d = (double)p - yi;
        sum += d * d / yi;
    }
    if (n_rounds) { // (its last level was written by this block, before a barrier)
        const uint32_t t = (uint32_t)n_rounds - 1, tree_nodes = (1u << a.depth) - 1u;
        make_words(nf + (uint64_t)t * tree_nodes, nt + (uint64_t)t * tree_nodes, a.n_feat, a.depth, 1, words + ((uint64_t)t << a.depth), threadIdx.x, 1024);
    } else {
        entry_quality(a.p_in, a.y, a.n, a.sc);
    }
    sum = block_sum(sum, scratch);
    if (threadIdx.x == 0) {
        *snr_out = a.sc->snr;
        *loss_out = a.sc->bad ? a.sc->loss : (float)(sum / (double)a.n);
    }
}

// Most pairs the one-launch levels take.  Every block of such a level goes over all pairs, however few features there are;
// the three launches share the pairs between blocks, and their histograms cost less with fewer features.  So the lines lie
// lower with fewer features, and for deeper trees, whose lower levels spread a histogram's atomics over many nodes.  They
// are where eight rounds took no longer with one launch a level than with three, the least over features of some fifty
// values, of six values and those of sampled convolution schedules, and no higher than where a workspace for three launches
// holds what one needs (fewer than 16 features at depths 3 and 4).  Three launches' time over one's, six values / schedules:
//   48 features: depth 5 36864 pairs 1.19 / 1.30, 49152 1.00 / 1.22; depth 7 65536 1.33 / 1.02
//   32 features: depth 6 28672 1.07 / 1.08, 36864 1.00 / 1.06, 49152 0.88 / 0.92; depth 8 36864 1.45 / 1.17, 49152 1.35 / 0.96
//   16 features: depth 4 28672 1.05 / 1.34, 36864 0.98 / 1.33; depth 8 12288 1.35 / 1.13, 20480 1.15 / 0.92
//   8 features: depth 3 65536 1.08 / 1.54; depth 5 20480 1.11 / 1.18, 28672 0.95 / 1.00; 1 feature, depth 8: 12288 1.28 / 0.89
// 32 features, depth 6, 28672 pairs, eight rounds: 1164.8 us with three launches a level, 1056.2 with one (six values).
uint64_t level_max_pairs(const eck_trees *m)
{
    constexpr uint32_t MOST = 65536;
    // by depth from three on; fewer than 16, 32, 48 and 64 features
    constexpr uint32_t most[ECK_MAX_TREE_DEPTH - 2][4] = {{32768, 49152, MOST, MOST},   {22528, 28672, 36864, 36864},
                                                          {20480, 20480, 28672, 36864}, {12288, 14336, 28672, 49152},
                                                          {9216, 12288, 36864, 49152},  {7168, 12288, 36864, MOST}};
    if (m->depth < 3 || m->n_feat >= 64) return MOST;
    return most[m->depth - 3][m->n_feat / 16];
}

struct BoostWs {
    uint64_t scalars, y, p, gq, hq, at, bins, hist, partial, total;
    uint64_t p2, at2, rec, left, tot; // one launch per level: second halves of ping-pong pairs, the two levels' records
};

BoostWs boost_layout(const eck_trees *m, uint64_t n_pairs)
{
    auto up = [](uint64_t v) { return (v + 255) & ~255ull; };
    const uint64_t nodes = (uint64_t)1 << (m->depth - 1); // of the last level
    BoostWs w = {};
    uint64_t o = 0;
    w.scalars = o; o = up(o + sizeof(RefitScalars));
    w.y = o; o = up(o + n_pairs * 4);
    w.p = o; o = up(o + n_pairs * 4);
    w.gq = o; o = up(o + n_pairs * 8);
    w.hq = o; o = up(o + n_pairs * 8);
    w.bins = o; o = up(o + n_pairs * (uint64_t)(m->n_feat + 1));
    if (n_pairs <= level_max_pairs(m)) {
        w.p2 = o; o = up(o + n_pairs * 4);
        w.at = o; o = up(o + n_pairs);
        w.at2 = o; o = up(o + n_pairs);
        w.rec = o; o = up(o + 2 * nodes * m->n_feat * sizeof(SplitRecord));
        w.left = o; o = up(o + 2 * nodes * m->n_feat * sizeof(SideSums));
        w.tot = o; o = up(o + 2 * nodes * sizeof(NodeTotals));
    } else {
        w.at = o; o = up(o + n_pairs * 4);
        w.hist = o; o = up(o + nodes * m->n_feat * BINS * 3 * 8);
        w.partial = o; o = up(o + nodes * ((m->n_feat + SPLIT_FEATS - 1) / SPLIT_FEATS) * sizeof(SplitRecord));
        // a workspace made for many pairs serves fewer, too
        const uint64_t fewer = boost_layout(m, level_max_pairs(m)).total;
        if (o < fewer) o = fewer;
    }
    w.total = o;
    return w;
}

// the boosting rounds of treemodel_update, one launch per level
int32_t boost_levels(eck_trees *m, char *base, const BoostWs &w, uint64_t n_pairs, int32_t n_rounds, float eta, double lam,
                     float *snr_out, float *loss_out, hipStream_t st)
{
    const size_t nodes = ((size_t)1 << m->depth) - 1, leaves = (size_t)1 << m->depth, last_nodes = (size_t)1 << (m->depth - 1);
    RefitScalars *sc = reinterpret_cast<RefitScalars *>(base + w.scalars);
    LevelArgs a = {};
    a.bins = reinterpret_cast<const uint8_t *>(base + w.bins);
    a.n = (uint32_t)n_pairs;
    a.n_feat = m->n_feat;
    a.depth = m->depth;
    a.y = reinterpret_cast<const float *>(base + w.y);
    a.gq = reinterpret_cast<long long *>(base + w.gq);
    a.hq = reinterpret_cast<long long *>(base + w.hq);
    a.eta = (double)eta;
    a.lam = lam;
    a.sc = sc;
    SplitRecord *rec[2];
    SideSums *left[2];
    NodeTotals *tot[2];
    uint8_t *at[2] = {reinterpret_cast<uint8_t *>(base + w.at), reinterpret_cast<uint8_t *>(base + w.at2)};
    float *p[2] = {reinterpret_cast<float *>(base + w.p), reinterpret_cast<float *>(base + w.p2)};
    for (int k = 0; k < 2; ++k) {
        rec[k] = reinterpret_cast<SplitRecord *>(base + w.rec) + k * last_nodes * a.n_feat;
        left[k] = reinterpret_cast<SideSums *>(base + w.left) + k * last_nodes * a.n_feat;
        tot[k] = reinterpret_cast<NodeTotals *>(base + w.tot) + k * last_nodes;
    }
    constexpr size_t LDS = (size_t)LEVEL_SLOTS * LEVEL_STRIDE * 16;
    ECK_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(tree_level_kernel<true>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS));
    ECK_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(tree_level_kernel<false>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)LDS));
    int side = 0, p_side = 0; // which half of each pair holds the level before / the predictions
    // what a launch settles: level `before` of tree t (its nodes, and its leaves when that was the last level)
    auto settle = [&](size_t t, int before) {
        a.nf = m->d_feat + t * nodes + (((size_t)1 << before) - 1);
        a.nt = m->d_thr + t * nodes + (((size_t)1 << before) - 1);
        a.leaf = m->d_leaf + t * leaves;
        a.rec_in = rec[side];
        a.left_in = left[side];
        a.tot_in = tot[side];
        a.at_in = at[side];
    };
    for (int32_t r = 0; r < n_rounds; ++r) {
        const size_t t = (size_t)m->n_trees + r;
        for (int l = 0; l < m->depth; ++l) {
            if (l > 0) settle(t, l - 1);
            else if (r > 0) settle(t - 1, m->depth - 1);
            a.rec_out = rec[side ^ 1];
            a.left_out = left[side ^ 1];
            a.tot_out = tot[side ^ 1];
            a.at_out = at[side ^ 1];
            const dim3 grid((unsigned)m->n_feat, (unsigned)(((1 << l) + LEVEL_SLOTS - 1) / LEVEL_SLOTS));
            if (l == 0) {
                a.p_in = p[p_side];
                a.p_out = p[p_side ^ 1];
                hipLaunchKernelGGL(tree_level_kernel<true>, dim3(grid.x + (r == 0 ? 1 : 0)), dim3(LEVEL_THREADS), LDS, st, a, l, r == 0 ? 1 : 0);
                p_side ^= 1;
            } else {
                hipLaunchKernelGGL(tree_level_kernel<false>, grid, dim3(LEVEL_THREADS), LDS, st, a, l, 0);
            }
            side ^= 1;
        }
    }
    if (n_rounds > 0) settle((size_t)m->n_trees + n_rounds - 1, m->depth - 1);
    a.p_in = p[p_side];
    const size_t first = (size_t)m->n_trees;
    const unsigned word_blocks = n_rounds > 1 ? (unsigned)(((((size_t)n_rounds - 1) << m->depth) + 1023) / 1024) : 0;
    hipLaunchKernelGGL(tree_last_kernel, dim3(1 + (word_blocks < 64 ? word_blocks : 64)), dim3(1024), 0, st, a, n_rounds, m->d_feat + first * nodes,
                       m->d_thr + first * nodes, m->d_word + first * leaves, snr_out, loss_out);
    ECK_HIP_TRY(hipGetLastError());
    return ECK_OK;
}

} // namespace

extern "C" int32_t eck_trees_create(int32_t n_feat, int32_t depth, int32_t capacity, float base_score, eck_trees **out)
{
    if (!out) return ECK_EINVAL;
    *out = nullptr;
    if (n_feat < 1 || depth < 1 || capacity < 1 || !(base_score == base_score)) return ECK_EINVAL;
    if (n_feat > 256 || depth > ECK_MAX_TREE_DEPTH || capacity > 65536) return ECK_EUNSUPPORTED;
    eck_trees *m = new (std::nothrow) eck_trees();
    if (!m) return ECK_EDEVICE;
    m->n_feat = n_feat;
    m->depth = depth;
    m->capacity = capacity;
    m->n_trees = 0;
    m->base = base_score;
    const size_t nodes = ((size_t)1 << depth) - 1, leaves = (size_t)1 << depth;
    if (hipGetDevice(&m->device) != hipSuccess || hipMalloc((void **)&m->d_feat, capacity * nodes) != hipSuccess ||
        hipMalloc((void **)&m->d_thr, capacity * nodes * 4) != hipSuccess ||
        hipMalloc((void **)&m->d_leaf, capacity * leaves * 4) != hipSuccess ||
        hipMalloc((void **)&m->d_word, capacity * leaves * 4) != hipSuccess) {
        (void)hipGetLastError();
        if (m->d_feat) (void)hipFree(m->d_feat);
        if (m->d_thr) (void)hipFree(m->d_thr);
        if (m->d_leaf) (void)hipFree(m->d_leaf);
        if (m->d_word) (void)hipFree(m->d_word);
        delete m;
        return ECK_EDEVICE;
    }
    *out = m;
    return ECK_OK;
}

extern "C" void eck_trees_destroy(eck_trees *m)
{
    if (!m) return;
    (void)hipDeviceSynchronize();
    (void)hipFree(m->d_feat);
    (void)hipFree(m->d_thr);
    (void)hipFree(m->d_leaf);
    (void)hipFree(m->d_word);
    delete m;
}

extern "C" int32_t eck_trees_count(const eck_trees *m, int32_t *n_trees)
{
    if (!m || !n_trees) return ECK_EINVAL;
    *n_trees = m->n_trees;
    return ECK_OK;
}

extern "C" int32_t eck_trees_set(eck_trees *m, int32_t n_trees, const uint8_t *node_feat, const float *node_thr,
                                 const float *leaf, void *stream)
{
    if (!m || n_trees < 0) return ECK_EINVAL;
    if (n_trees > m->capacity) return ECK_ESHAPE;
    if (n_trees && (!node_feat || !node_thr || !leaf)) return ECK_EINVAL;
    const size_t nodes = ((size_t)1 << m->depth) - 1, leaves = (size_t)1 << m->depth;
    hipStream_t st = as_stream(stream);
    if (n_trees) {
        const uint32_t slots = (uint32_t)n_trees << m->depth;
        hipLaunchKernelGGL(tree_set_kernel, dim3((slots + 255) / 256), dim3(256), 0, st, node_feat, node_thr, leaf, m->n_feat,
                           m->depth, n_trees, m->d_feat, m->d_thr, m->d_leaf, m->d_word);
        ECK_HIP_TRY(hipGetLastError());
    }
    m->n_trees = n_trees;
    return ECK_OK;
}

extern "C" int32_t eck_trees_get(const eck_trees *m, uint8_t *node_feat, float *node_thr, float *leaf, void *stream)
{
    if (!m) return ECK_EINVAL;
    if (m->n_trees == 0) return ECK_OK;
    if (!node_feat || !node_thr || !leaf) return ECK_EINVAL;
    const size_t nodes = ((size_t)1 << m->depth) - 1, leaves = (size_t)1 << m->depth;
    hipStream_t st = as_stream(stream);
    const uint64_t slots = (uint64_t)m->n_trees * leaves;
    hipLaunchKernelGGL(tree_get_kernel, dim3((unsigned)(slots < 1024 * 256 ? (slots + 255) / 256 : 1024)), dim3(256), 0, st, m->d_feat, m->d_thr,
                       m->d_leaf, m->n_trees * nodes, slots, node_feat, node_thr, leaf);
    ECK_HIP_TRY(hipGetLastError());
    return ECK_OK;
}

extern "C" int32_t treemodel_score(const eck_trees *m, const void *feat, int32_t feat_dtype, uint64_t ld, uint64_t n,
                                   float *score_out, void *stream)
{
    if (!m || !feat || !score_out || n == 0) return ECK_EINVAL;
    if (feat_dtype != ECK_F32 && feat_dtype != ECK_BF16) return ECK_EINVAL;
    if (ld < n) return ECK_ESHAPE;
    if (n > (1ull << 40)) return ECK_EINVAL;
    return launch_score(m, m->n_trees, feat, feat_dtype, ld, n, score_out, as_stream(stream));
}

extern "C" uint64_t treemodel_update_workspace_bytes(const eck_trees *m, uint64_t n_pairs)
{
    if (!m || n_pairs == 0 || n_pairs > (1ull << 20)) return 0;
    return boost_layout(m, n_pairs).total;
}

extern "C" int32_t treemodel_update(eck_trees *m, const void *feat, int32_t feat_dtype, uint64_t ld,
                                    const float *energy_measured, uint64_t n_pairs, int32_t n_rounds, float eta,
                                    float lambda, float *snr_out, float *loss_out, void *ws, uint64_t ws_bytes,
                                    void *stream)
{
    if (!m || !feat || !energy_measured || !snr_out || !loss_out) return ECK_EINVAL;
    if (n_pairs == 0 || n_rounds < 0 || !(eta > 0.0f) || !(lambda >= 0.0f)) return ECK_EINVAL;
    if (feat_dtype != ECK_F32 && feat_dtype != ECK_BF16) return ECK_EINVAL;
    if (n_pairs > (1ull << 20)) return ECK_EUNSUPPORTED;
    if (ld < n_pairs || m->n_trees + n_rounds > m->capacity) return ECK_ESHAPE;
    const BoostWs w = boost_layout(m, n_pairs);
    if (!ws || ws_bytes < w.total) return ECK_EWORKSPACE;
    if ((uintptr_t)ws & 255) return ECK_EALIGN;

    hipStream_t st = as_stream(stream);
    char *base = static_cast<char *>(ws);
    RefitScalars *sc = reinterpret_cast<RefitScalars *>(base + w.scalars);
    float *y = reinterpret_cast<float *>(base + w.y), *p = reinterpret_cast<float *>(base + w.p);
    long long *gq = reinterpret_cast<long long *>(base + w.gq), *hq = reinterpret_cast<long long *>(base + w.hq);
    uint32_t *at = reinterpret_cast<uint32_t *>(base + w.at);
    uint8_t *bins = reinterpret_cast<uint8_t *>(base + w.bins);
    unsigned long long *hist = reinterpret_cast<unsigned long long *>(base + w.hist);
    SplitRecord *partial = reinterpret_cast<SplitRecord *>(base + w.partial);
    const unsigned split_groups = (unsigned)((m->n_feat + SPLIT_FEATS - 1) / SPLIT_FEATS);
    const int is_bf16 = feat_dtype == ECK_BF16;
    const uint32_t nodes = (1u << m->depth) - 1u, leaves = 1u << m->depth;
    const unsigned pair_blocks = (unsigned)((n_pairs + 255) / 256);
    const double lam = (double)lambda * FIX;

    hipLaunchKernelGGL(tree_prepare_kernel, dim3((unsigned)((n_pairs + 1023) / 1024), m->n_feat + 1), dim3(1024), 0, st, feat, is_bf16, ld, n_pairs,
                       m->n_feat, bins, energy_measured, y, sc);
    // predictions of the ensemble as it stands: the scoring kernel (fp32, base first, trees in order)
    int32_t rc = launch_score(m, m->n_trees, feat, feat_dtype, ld, n_pairs, p, st);
    if (rc != ECK_OK) return rc;
    if (n_pairs <= level_max_pairs(m)) {
        rc = boost_levels(m, base, w, n_pairs, n_rounds, eta, lam, snr_out, loss_out, st);
        if (rc != ECK_OK) return rc;
        m->n_trees += n_rounds;
        return ECK_OK;
    }
    hipLaunchKernelGGL(tree_quality_kernel, dim3(1), dim3(1024), 0, st, p, y, n_pairs, 0, sc);
    {
        // the histogram buffer starts clear; from then on the split kernel clears what it reads
        const uint64_t words = ((uint64_t)1 << (m->depth - 1)) * m->n_feat * BINS * 3;
        hipLaunchKernelGGL(tree_zero_kernel, dim3((unsigned)((words + 255) / 256)), dim3(256), 0, st, hist, words);
    }
    for (int32_t r = 0; r < n_rounds; ++r) {
        const size_t t = (size_t)m->n_trees + r;
        uint8_t *nf = m->d_feat + t * nodes;
        float *nt = m->d_thr + t * nodes;
        float *lw = m->d_leaf + t * leaves;
        hipLaunchKernelGGL(tree_grad_kernel, dim3(pair_blocks), dim3(256), 0, st, p, y, n_pairs, gq, hq, at, nf, nt, nodes);
        for (int l = 0; l < m->depth; ++l) {
            const uint32_t level_nodes = 1u << l, first = level_nodes - 1u;
            {
                unsigned slices = (unsigned)(n_pairs / 2048);
                slices = slices < 1 ? 1 : (slices > 64 ? 64 : slices);
                const unsigned groups = (level_nodes + LDS_HIST_NODES - 1) / LDS_HIST_NODES;
                hipLaunchKernelGGL(tree_hist_lds_kernel, dim3(slices, m->n_feat, groups), dim3(BLOCK), 0, st, bins, gq, hq,
                                   at, n_pairs, m->n_feat, first, level_nodes, hist);
            }
            hipLaunchKernelGGL(tree_split_kernel, dim3(level_nodes, split_groups), dim3(SPLIT_FEATS * 64), 0, st, hist,
                               m->n_feat, lam, partial);
            hipLaunchKernelGGL(tree_partition_kernel, dim3(pair_blocks), dim3(256), 0, st, feat, is_bf16, ld, n_pairs,
                               partial, split_groups, first, sc, nf, nt, at);
        }
        hipLaunchKernelGGL(tree_leaf_kernel, dim3(1), dim3(1024), 0, st, gq, hq, at, n_pairs, nodes, leaves, (double)eta,
                           lam, lw, sc);
        hipLaunchKernelGGL(tree_advance_kernel, dim3(pair_blocks), dim3(256), 0, st, p, at, lw, nodes, n_pairs);
    }
    hipLaunchKernelGGL(tree_quality_kernel, dim3(1), dim3(1024), 0, st, p, y, n_pairs, 1, sc);
    hipLaunchKernelGGL(tree_finish_kernel, dim3(1), dim3(64), 0, st, sc, snr_out, loss_out);
    if (n_rounds > 0) {
        const size_t t = (size_t)m->n_trees;
        hipLaunchKernelGGL(tree_set_kernel, dim3((unsigned)((((size_t)n_rounds << m->depth) + 255) / 256)), dim3(256), 0, st,
                           m->d_feat + t * nodes, m->d_thr + t * nodes, nullptr, m->n_feat, m->depth, n_rounds, nullptr, nullptr,
                           nullptr, m->d_word + t * leaves);
    }
    ECK_HIP_TRY(hipGetLastError());
    m->n_trees += n_rounds;
    return ECK_OK;
}
