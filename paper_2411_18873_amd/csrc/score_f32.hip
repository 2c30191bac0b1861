// Forward pass of fp32 models on the matrix cores (HIP, gfx950): costmodel_score for ECK_F32 models of any hidden
// widths (Alg. 1: LatencyEvaAndPick, EnergyModelEvaAndPick; Sec. 5.4).
//
// The network is evaluated transposed, rows = hidden units (weights), columns = candidates, every fp32 number as the sum of
// three bfloat16 ones and every product as the six largest of their products, summed in fp32 (f32_split.h): sixteen times the
// fp32 matrix rate, for six times the products.  A block's wavefronts share a layer's 16-unit tiles as evenly as they go and
// read the same activations from LDS, which holds their parts as [part][unit / 8][candidate][unit % 8].  The weights' parts
// are made when the state changes and stream from the L2, one load at a time between matrix instructions.
// Models with weights that have no such parts, candidates with features that have none, and models whose first layer has no
// more than sixteen units are worked out in fp32 products instead.
//
// What bounds it: matrix instructions and the LDS reads of the activations behind them (a part of four candidate tiles is read
// for twelve matrix instructions), for narrow models the features.  Measured, against fp32 matrix instructions (which reached
// 121-135 of their 153 TFLOP/s): 64-256-256-1 on 100003 candidates 152 -> 92 us (179 TFLOP/s of fp32 products, 1070 of bfloat16
// ones; 90-100 by the clock a card sustains), 64-128-128-1 on 2^18 125 -> 82, 64-512-512-1 on 100003 500 -> 320 and on 1536
// 22.6 -> 20.1, 32-64-64-1 on 6400 6.3 -> 4.3 and on 2^20 152 -> 119.  (64-512-512-1 took 423 and 22.5 with 256 units of the first
// layer in LDS at a time and the second layer's sums of 256 units, for which the first was worked out twice.)  Errors
// against 64 bits, relative to the scores' norm (before in brackets): 512 units 2.5-3.4e-8 (6.1-6.4e-8), 256 3.1-3.6e-8
// (6.2-6.6e-8), 128 3.1-4.2e-8 (6.6-8.5e-8), 64 3.9-4.4e-8 (7.4-9.1e-8), 200 and 96 3.6-4.0e-8 (6.8-9.4e-8).
#include <type_traits>

#include "f32_split.h"
#include "f32_tiles.h"
#include "lanes.h"

using namespace eck;
using namespace eck::split;

namespace {

using f32::f32x4;
using f32::RSRC_FLAGS;

struct F32Net {
    const unsigned char *packed; // fragments of both hidden layers ...
    const uint32_t *flags;       // ... and in so many words (at most 144) whether they hold weights outside the parts' range
    int words;
    const float *w1, *b1, *w2, *b2, *w3, *b3;
    int F, H1, H2;
};

// Sums of M x CT tiles: the largest product of each pair apart from the others, so that it is rounded once per group of 32
// inputs and the others at their own size
template <int M, int CT>
struct Sums {
    f32x4 large[M][CT], small[M][CT];
};

// s[j][ct] += W^T x for J tiles from `first_tile` on, over `groups` groups of 32 inputs, and CT tiles of candidates.  layer:
// byte offset of its fragments; act: granules (16 bytes: eight units of one candidate) of part 0, this wavefront's first
// candidate; `cands` granules to a row, `part_step` to a part.  AHEAD: the next group's activations are read while this one is
// multiplied.
template <int J, bool AHEAD, int M, int CT>
__device__ __forceinline__ void product(__amdgpu_buffer_rsrc_t weights, uint32_t layer, int groups, int first_tile, const u32x4 *act,
                                        int cands, int part_step, int lane, Sums<M, CT> &s)
{
    constexpr int SETS = J * CT <= 4 ? 2 : 1; // weights requested two groups ahead where the registers hold them, else one
    const int last = groups - 1;
    const u32x4 *from = act + (lane >> 4) * cands + (lane & 15);
    bf16x8 a[SETS][J][PARTS], b[AHEAD ? 2 : 1][PARTS][CT];
    auto fetch = [&](int g, int j, bf16x8(&to)[PARTS]) {
        const uint32_t at = layer + ((uint32_t)(first_tile + j) * groups + min(g, last)) * (PARTS * 1024u);
#pragma unroll
        for (int i = 0; i < PARTS; ++i)
            to[i] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(weights, 16 * lane, at + 1024u * i, 0));
    };
    auto read = [&](int g, bf16x8(&to)[PARTS][CT]) {
#pragma unroll
        for (int i = 0; i < PARTS; ++i)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
                to[i][ct] = __builtin_bit_cast(bf16x8, from[i * part_step + 4 * min(g, last) * cands + 16 * ct]);
    };
#pragma unroll
    for (int k = 0; k < SETS; ++k)
#pragma unroll
        for (int j = 0; j < J; ++j) fetch(k, j, a[k][j]);
    if (AHEAD) read(0, b[0]);
    auto group = [&](int g, auto odd) {
        constexpr int P = decltype(odd)::value, S = P % SETS, B = AHEAD ? P : 0;
        if (AHEAD) read(g + 1, b[AHEAD ? P ^ 1 : 0]);
        else read(g, b[0]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < J; ++j) {
            constexpr int WEIGHT[6] = {2, 0, 1, 1, 0, 0}, INPUT[6] = {0, 2, 1, 0, 1, 0};
#pragma unroll
            for (int k = 0; k < 6; ++k)
#pragma unroll
                for (int ct = 0; ct < CT; ++ct) {
                    f32x4 &to = k < 5 ? s.small[j][ct] : s.large[j][ct];
                    to = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[S][j][WEIGHT[k]], b[B][INPUT[k]][ct], to, 0, 0, 0);
                }
            __builtin_amdgcn_sched_barrier(0);
            fetch(g + SETS, j, a[S][j]);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    int g = 0;
    for (; g + 2 <= groups; g += 2) {
        group(g, std::integral_constant<int, 0>());
        group(g + 1, std::integral_constant<int, 1>());
    }
    if (g < groups) group(g, std::integral_constant<int, 0>());
}

// acc[j][ct] = b + W^T x in fp32 products, for J tiles of sixteen units from `first_tile` on and CT tiles of candidates.  act: the
// activations of units 0-3 of this wavefront's first candidate, `cands` candidates to a row.  The weights come from the
// parameters, requested two groups of sixteen inputs ahead, one load between matrix instructions.  (Rows of several
// tiles interleaved would take one wide load for J, but give sums of an order that depends on J.)
template <int J, int CT, int M>
__device__ __forceinline__ void plain_product(const f32::F32Layer &l, int first_tile, const f32x4 *act, int cands, int p, int c,
                                              f32x4 (&acc)[M][CT])
{
    const int whole = l.K / 16, last = whole - 1;
    auto slice = [&](int j) { return f32::Slice<1>(l, 16 * (first_tile + j), p, c); };
    float even[4][J], odd[4][J]; // weights of an even and an odd group; past the end the last whole group again
    auto fetch = [&](int g, int t, float(&a)[J]) {
#pragma unroll
        for (int j = 0; j < J; ++j) {
            float one[1];
            slice(j).row(g, t, one);
            a[j] = one[0];
        }
    };
    if (whole) {
#pragma unroll
        for (int t = 0; t < 4; ++t) fetch(0, t, even[t]);
#pragma unroll
        for (int t = 0; t < 4; ++t) fetch(min(1, last), t, odd[t]);
    }
#pragma unroll
    for (int j = 0; j < J; ++j) {
        f32x4 bias;
#pragma unroll
        for (int q = 0; q < 4; ++q) bias[q] = l.b[min(16 * (first_tile + j) + 4 * p + q, l.H - 1)];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[j][ct] = bias;
    }
    const f32x4 *from = act + p * cands + c;
    f32x4 be[CT], bo[CT]; // activations of an even and an odd group
    auto read = [&](int g, f32x4(&b)[CT]) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) b[ct] = from[4 * g * cands + 16 * ct];
    };
    auto step = [&](int t, const float(&a)[J], const f32x4(&b)[CT]) {
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) acc[j][ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b[ct][t], acc[j][ct], 0, 0, 0);
    };
    auto group = [&](int g, float(&a)[4][J], const f32x4(&b)[CT], f32x4(&next)[CT]) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            step(t, a[t], b);
            __builtin_amdgcn_sched_barrier(0);
            fetch(min(g + 2, last), t, a[t]);
            if (t == 0) read(min(g + 1, last), next);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    int g = 0;
    read(0, be);
    for (; g + 2 <= whole; g += 2) {
        group(g, even, be, bo);
        group(g + 1, odd, bo, be);
    }
    if (g < whole) {
#pragma unroll
        for (int t = 0; t < 4; ++t) step(t, even[t], be);
    }
    if (l.K % 16) {
        read(whole, be);
#pragma unroll
        for (int j = 0; j < J; ++j) {
            float tail[4][1];
            slice(j).partial_group(whole, tail);
#pragma unroll
            for (int t = 0; t < 4; ++t) even[t][j] = tail[t][0];
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) step(t, even[t], be);
    }
}

// blockDim = 64 * unit_slots * cand_slots: wavefront (us, cs) works on share us of every layer for the CT candidate
// tiles of slot cs.  Every sum has an order that depends on the widths alone, so a candidate's score depends neither on
// n nor on its place.  M: most 16-unit tiles per wavefront of the units that are worked on at a time, all of the first
// layer's.  BY_PARTS: products of parts, and fp32 ones where a model or a candidate needs them; else fp32 ones alone.
template <int CT, int M, bool BY_PARTS, bool WITH_MIN>
__device__ __forceinline__ void score_block(const F32Net &net, const float *__restrict__ feat, uint64_t ld, uint64_t n,
                                            float *__restrict__ out, int unit_slots, int x_rows, int h_rows, int act_bytes,
                                            const MinArgs &mn, uint64_t skip, uint32_t block)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char f32_lds[];
    const int tid = threadIdx.x, lane = tid & 63, p = lane >> 4, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = (int)blockDim.x / 64;
    const int us = wave % unit_slots, cs = wave / unit_slots;
    const int cands = waves / unit_slots * (16 * CT);
    float *sum_l = reinterpret_cast<float *>(f32_lds + act_bytes); // [tiles of the second layer][cands]
    const int out_tiles = tiles_of(net.H2);
    uint32_t *odd_l = reinterpret_cast<uint32_t *>(sum_l + out_tiles * cands); // [cands], then whether there is any
    const uint64_t base = skip + (uint64_t)block * cands;
    // this wavefront's share of so many tiles: the first shares are a tile larger when they do not divide
    auto share_of = [&](int tiles, int *first) {
        const int base_tiles = tiles / unit_slots, more = tiles % unit_slots;
        *first = us * base_tiles + min(us, more);
        return base_tiles + (us < more ? 1 : 0);
    };
    auto for_tiles = [](int tiles, auto go) {
        if constexpr (M == 4) {
            if (tiles == 4) go(std::integral_constant<int, 4>());
            else if (tiles == 3) go(std::integral_constant<int, 3>());
        }
        if constexpr (M >= 2) {
            if (tiles == 2) go(std::integral_constant<int, 2>());
        }
        if (tiles == 1) go(std::integral_constant<int, 1>());
    };
    // the output's weights of the units this lane holds of M tiles of the second layer (requested before the layer's product: a
    // load behind it was waited for, 0.25 us a call)
    auto output_weights = [&](int first, float(&w)[M][4]) {
#pragma unroll
        for (int j = 0; j < M; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) w[j][q] = net.w3[min(16 * (first + j) + 4 * p + q, net.H2 - 1)];
    };
    // the output's part of a tile, whichever wavefront worked it out; value(q, ct): the sums of its units 4p + q
    auto tile_output = [&](int tile, const float(&w)[4], auto value, auto takes) {
        float y[CT] = {};
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int unit = 16 * tile + 4 * p + q;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) y[ct] = unit < net.H2 ? fmaf(fmaxf(value(q, ct), 0.0f), w[q], y[ct]) : y[ct];
        }
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) {
            y[ct] += __uint_as_float(lane_exchange(__float_as_uint(y[ct]), 16));
            y[ct] += __uint_as_float(lane_exchange(__float_as_uint(y[ct]), 32));
            const int cand = 16 * (cs * CT + ct) + c;
            if (p == 0 && takes(cand)) sum_l[tile * cands + cand] = y[ct];
        }
    };
    // The second layer as many units at a time as the sums of M tiles take
    const int most2 = unit_slots * (16 * M);
    bool outside = !BY_PARTS; // the model's weights do not all have parts
    if constexpr (BY_PARTS) {
        u32x4 *x_l = reinterpret_cast<u32x4 *>(f32_lds); // features [3][x_rows][cands], then activations [3][h_rows][cands]
        for (int e = tid; e <= cands; e += blockDim.x) odd_l[e] = 0;
        uint32_t flagged = net.flags[min(lane, net.words - 1)]; // (looked at behind the features, which are waited for in any case)
        if (net.words > 64) flagged |= net.flags[min(lane + 64, net.words - 1)] | net.flags[min(lane + 128, net.words - 1)];

        for (int e = tid; e < net.F / 8 * cands; e += blockDim.x) { // 32 or 64 features
            const int cand = e % cands, eight = e / cands;
            const uint64_t col = base + cand < n ? base + cand : n - 1;
            float v[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) v[t] = feat[(uint64_t)(8 * eight + t) * ld + col];
            uint32_t least = 0xFFFFFFFFu;
#pragma unroll
            for (int t = 0; t < 8; ++t) least = min(least, magnitude_order(__float_as_uint(v[t])));
            u32x4 to[PARTS];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                uint32_t part[PARTS];
                split_two(v[2 * t], v[2 * t + 1], part);
#pragma unroll
                for (int i = 0; i < PARTS; ++i) to[i][t] = part[i];
            }
            if (least < magnitude_order(LEAST_INPUT)) to[2][0] = 0x7FC07FC0u; // (its sums become NaNs, as with infinities)
#pragma unroll
            for (int i = 0; i < PARTS; ++i) x_l[(i * x_rows + eight) * cands + cand] = to[i];
        }
        outside = __ballot(flagged != 0) != 0;
        __syncthreads();
        if (!outside) {
            const __amdgpu_buffer_rsrc_t weights = __builtin_amdgcn_make_buffer_rsrc(
                const_cast<unsigned char *>(net.packed), 0, fragments(net.F, net.H1, net.H2) * (PARTS * 1024), RSRC_FLAGS);
            const uint32_t layer2 = fragments1(net.F, net.H1) * (PARTS * 1024u);
            const int groups1 = groups_of(net.F), groups2 = groups_of(net.H1);
            auto run = [&](int tiles, uint32_t layer, int groups, int first_tile, int part_step, auto ahead, auto &to) {
                for_tiles(tiles, [&](auto j) {
                    product<decltype(j)::value, decltype(ahead)::value>(weights, layer, groups, first_tile, x_l + cs * (16 * CT), cands, part_step,
                                                                        lane, to);
                });
            };
            auto start = [&](const float *b, int H, int first_tile, auto &to) {
#pragma unroll
                for (int j = 0; j < M; ++j) {
                    f32x4 v;
#pragma unroll
                    for (int q = 0; q < 4; ++q) v[q] = b[min(16 * (first_tile + j) + 4 * p + q, H - 1)];
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) {
                        to.large[j][ct] = v;
                        to.small[j][ct] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
                    }
                }
            };
            // zero times everything a candidate's sums held: a NaN once one of them was not finite
            float odd[CT] = {};
            {
                int first1;
                const int tiles1 = share_of(tiles_of(net.H1), &first1);
                Sums<M, CT> sum1;
                start(net.b1, net.H1, first1, sum1);
                run(tiles1, 0, groups1, first1, x_rows * cands, std::false_type(), sum1);
                __syncthreads(); // every wavefront has read the features: their place takes the activations
#pragma unroll
                for (int j = 0; j < M; ++j) {
                    if (j >= tiles1) break;
                    const int in = 16 * (first1 + j) + 4 * p; // this lane's four units
#pragma unroll
                    for (int ct = 0; ct < CT; ++ct) {
                        float v[4];
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const float sum = sum1.large[j][ct][q] + sum1.small[j][ct][q];
                            odd[ct] = fmaf(sum, 0.0f, odd[ct]);
                            // (a unit past H1 is zero; its weights in the next layer are, too)
                            v[q] = in + q < net.H1 ? fmaxf(sum, 0.0f) : 0.0f;
                        }
                        uint32_t lo[PARTS], hi[PARTS];
                        split_two(v[0], v[1], lo);
                        split_two(v[2], v[3], hi);
#pragma unroll
                        for (int i = 0; i < PARTS; ++i) {
                            u32x4 *row = x_l + (i * h_rows + in / 8) * cands + 16 * (cs * CT + ct) + c;
                            reinterpret_cast<uint2 *>(row)[in / 4 % 2] = make_uint2(lo[i], hi[i]);
                        }
                    }
                }
                // inputs of the last group that no tile covers
                if (tiles_of(net.H1) % 2) {
                    for (int e = tid; e < 2 * PARTS * cands; e += blockDim.x)
                        x_l[(e / (2 * cands) * h_rows + 2 * tiles_of(net.H1) + e / cands % 2) * cands + e % cands] = u32x4{0, 0, 0, 0};
                }
                __syncthreads();
            }
            for (int v0 = 0; v0 < net.H2; v0 += most2) {
                int first2;
                const int tiles2 = share_of(tiles_of(min(most2, net.H2 - v0)), &first2);
                first2 += v0 / 16;
                Sums<M, CT> sum2;
                float w3[M][4];
                start(net.b2, net.H2, first2, sum2);
                output_weights(first2, w3);
                run(tiles2, layer2, groups2, first2, h_rows * cands, std::true_type(), sum2);
#pragma unroll
                for (int j = 0; j < M; ++j) {
                    if (j >= tiles2) break;
                    tile_output(
                        first2 + j, w3[j],
                        [&](int q, int ct) {
                            const float sum = sum2.large[j][ct][q] + sum2.small[j][ct][q];
                            odd[ct] = fmaf(sum, 0.0f, odd[ct]);
                            return sum;
                        },
                        [](int) { return true; });
                }
            }
#pragma unroll
            for (int ct = 0; ct < CT; ++ct)
                if (odd[ct] != odd[ct]) odd_l[16 * (cs * CT + ct) + c] = odd_l[cands] = 1;
            __syncthreads();
        }
    }
    // The same in fp32 products: for the block, if the model needs them, else for its candidates whose numbers do
    if (outside || odd_l[cands]) {
        f32x4 *act = reinterpret_cast<f32x4 *>(f32_lds); // [unit / 4][cands][unit % 4], features and then activations
        const f32x4 *mine = act + cs * (16 * CT);
        for (int e = tid; e < net.F / 4 * cands; e += blockDim.x) {
            const int cand = e % cands, four = e / cands;
            const uint64_t col = base + cand < n ? base + cand : n - 1;
            f32x4 v;
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] = feat[(uint64_t)(4 * four + t) * ld + col];
            act[e] = v;
        }
        __syncthreads();
        auto run = [&](int tiles, const f32::F32Layer &l, int first_tile, f32x4(&acc)[M][CT]) {
            for_tiles(tiles, [&](auto j) { plain_product<decltype(j)::value>(l, first_tile, mine, cands, p, c, acc); });
        };
        f32x4 acc[M][CT];
        int first1;
        const int tiles1 = share_of(tiles_of(net.H1), &first1);
        run(tiles1, {net.w1, net.b1, net.F, net.H1}, first1, acc);
        __syncthreads();
#pragma unroll
        for (int j = 0; j < M; ++j) {
            if (j >= tiles1) break;
            const int in = 16 * (first1 + j) + 4 * p;
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) {
                f32x4 v;
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] = in + q < net.H1 ? fmaxf(acc[j][ct][q], 0.0f) : 0.0f;
                act[in / 4 * cands + 16 * (cs * CT + ct) + c] = v;
            }
        }
        __syncthreads();
        for (int v0 = 0; v0 < net.H2; v0 += most2) {
            int first2;
            const int tiles2 = share_of(tiles_of(min(most2, net.H2 - v0)), &first2);
            first2 += v0 / 16;
            float w3[M][4];
            output_weights(first2, w3);
            run(tiles2, {net.w2, net.b2, net.H1, net.H2}, first2, acc);
#pragma unroll
            for (int j = 0; j < M; ++j) {
                if (j >= tiles2) break;
                tile_output(first2 + j, w3[j], [&](int q, int ct) { return acc[j][ct][q]; }, [&](int cand) { return outside || odd_l[cand]; });
            }
        }
        __syncthreads();
    }
    if (tid >= ((cands + 63) & ~63)) return; // (whole wavefronts)
    const uint64_t cand = base + tid;
    const bool mine = tid < cands && cand < n;
    const int at = min(tid, cands - 1);
    // (up to 32 parts one after the other in fp32 are the largest error of a score)
    double parts = net.b3[0];
    for (int t = 0; t < out_tiles; ++t) parts += sum_l[t * cands + at];
    const float total = (float)parts;
    if (mine) out[cand] = total;
    if (WITH_MIN) {
        uint32_t key = 0xFFFFFFFFu;
        if (mine && (!mn.legal || mn.legal[cand]) && total == total) key = score_order_key(total);
        // A wavefront's candidates lie in one segment as a rule: one atomic for them, and none where the segment's least key, as
        // last seen, is no larger (it only falls).  With an atomic for every sixteen candidates a launch waited for those on one
        // key: 2^20 candidates of 32-64-64-1 in one segment 765 us, now 147
        // (130 without minima).
        auto lower = [&](uint64_t seg, uint32_t k) {
            if (k < __hip_atomic_load(mn.min_key + seg, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP))
                (void)__hip_atomic_fetch_min(mn.min_key + seg, k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        };
        const uint64_t first = base + (tid & ~63), end = base + min(cands, (tid & ~63) + 64), last = (end < n ? end : n) - 1;
        if (first >= n) return;
        const uint64_t seg = first / mn.seg_len;
        if (last / mn.seg_len == seg) {
            key = wave_least(key);
            if ((tid & 63) == 0 && key != 0xFFFFFFFFu) lower(seg, key);
        } else if (key != 0xFFFFFFFFu) {
            lower(cand / mn.seg_len, key);
        }
    }
}

// The first `whole` blocks take CT candidate tiles a slot, `skip` candidates together; the others, in the last round of blocks,
// LAST_CT.
template <int CT, int M, bool BY_PARTS, bool WITH_MIN, int LAST_CT = CT>
__global__ __launch_bounds__(512, 2) void score_f32_kernel(F32Net net, const float *__restrict__ feat, uint64_t ld,
                                                           uint64_t n, float *__restrict__ out, int unit_slots, int x_rows,
                                                           int h_rows, int act_bytes, MinArgs mn, uint32_t whole, uint64_t skip)
{
    if (LAST_CT == CT || blockIdx.x < whole)
        score_block<CT, M, BY_PARTS, WITH_MIN>(net, feat, ld, n, out, unit_slots, x_rows, h_rows, act_bytes, mn, 0, blockIdx.x);
    else
        score_block<LAST_CT, M, BY_PARTS, WITH_MIN>(net, feat, ld, n, out, unit_slots, x_rows, h_rows, act_bytes, mn, skip,
                                                   blockIdx.x - whole);
}

template <bool WITH_MIN>
int32_t launch(const eck_model *m, const float *feat, uint64_t ld, uint64_t n, float *out, const MinArgs &mn, hipStream_t st)
{
    const int F = m->widths[0], H1 = m->widths[1], H2 = m->widths[2];
    if ((n + 15) / 16 > 0x7FFFFFFFull) return ECK_EUNSUPPORTED;
    const float *s = m->d_state;
    const unsigned char *packed = (const unsigned char *)m->d_packed;
    const F32Net net{packed, reinterpret_cast<const uint32_t *>(packed + (uint64_t)fragments(F, H1, H2) * (PARTS * 1024)),
                     (int)flag_words(F, H1, H2), s + m->off_w[0], s + m->off_b[0], s + m->off_w[1], s + m->off_b[1],
                     s + m->off_w[2], s + m->off_b[2], F, H1, H2};
    const int widest = H1 > H2 ? H1 : H2;
    const uint64_t tiles = (n + 15) / 16;
    const bool by_parts = H1 > 16;
    // Two unit tiles per wavefront and four candidate tiles (64 candidates a block): a weight is read for four, an activation
    // for two.  Fewer candidates where blocks that large would leave compute units without one (64-256-256-1, us with 1 / 2 /
    // 4 candidate tiles: 1000 9 / 10 / -, 6400 17 / 10.7 / 14, 16000 34 / 21 / 15, 100003 199 / 126 / 95); two at most, and
    // four unit tiles, where the first layer has more than 256 units.  Narrower models with one unit
    // tile per wavefront until the chip is full (64-128-128-1: 6400 6.2 against 6.8, 16000 7.9 and 8.9, 30000 14.6 and 11;
    // 32-64-64-1: 30000 6.4 and 6.9, 60000 11 and 8.8), those of 32 units or less always (64-30-20-1 on 2^20: 116-118
    // against 130).
    int ct = tiles <= 256 ? 1 : tiles <= 512 || H1 > 256 ? 2 : 4, per = H1 > 256 ? 4 : 2, unit_slots = 8, cand_slots = 1;
    if (!by_parts) {
        // In fp32 products, which need no pass over parts: a group of 32 inputs would be half zeros in the second layer, and a
        // first layer of one tile is its features' parts.  us, former fp32 instructions / products of parts / these: 32-16-16-1
        // 6400 3.6 / 4.5 / 3.5, 100003 7.2 / 8.3 / 7.4, 2^20 51 / 53 / 41; 64-16-16-1 30000 5.2 / 6.8 / 5.3, 100003 10.2 / 12.8 / 10.3;
        // 64-16-64-1 4096 5.3 / 4.2 / 3.8, 2^18 28 / 38 / 28; 64-16-512-1 4096 5.7 / 6.4 / 5.8, 100003 52 / 57 / 41.  Errors as fp32
        // instructions have (64-16-512-1 0.7-1.0e-7 of the scores' norm; of parts 0.4-0.5e-7).  One wavefront a tile of the
        // second layer until the chip is full, then fewer of more tiles; the lines lie where measured times cross.
        per = widest > 256 && tiles <= 256 ? 4 : 1;
        if (widest <= 16) {
            unit_slots = 1;
            cand_slots = tiles <= 1024 ? 1 : 4;
            ct = tiles <= 3072 || (F == 64 && tiles > 8192) ? 1 : 2;
        } else if (widest <= 64) {
            unit_slots = tiles <= 5632 ? 4 : 2;
            cand_slots = 4 / unit_slots;
            ct = tiles <= 512 ? 1 : tiles <= 1536 || (F == 64 && tiles > 8192) ? 2 : 4;
        } else {
            unit_slots = tiles <= 512 || (widest > 128 && tiles <= 3072) ? 8 : 4;
            ct = tiles <= 256 ? 1 : tiles <= 512 || (widest <= 128 && tiles <= 1536) ? 2 : 4;
        }
    } else if (widest <= 32) {
        per = 1;
        unit_slots = cand_slots = 2;
        if (ct > 2) ct = 2;
    } else if (widest <= 64) {
        per = tiles <= 2048 ? 1 : 2;
        unit_slots = 4 / per;
    } else if (widest <= 128) {
        per = tiles <= 1024 ? 1 : 2;
        unit_slots = 8 / per;
    }
    const int cands = 16 * ct * cand_slots, x_rows = F / 8, h_rows = 4 * groups_of(H1);
    const int threads = 64 * unit_slots * cand_slots;
    const int part_rows = by_parts ? PARTS * (x_rows > h_rows ? x_rows : h_rows) : 0, plain_rows = (F > H1 ? F : H1 + 15) / 16 * 4;
    const size_t act_bytes = (size_t)(part_rows > plain_rows ? part_rows : plain_rows) * cands * 16;
    const size_t lds = act_bytes + ((size_t)tiles_of(H2) * cands + cands + 1) * 4;
    // Eight wavefronts of blocks of 64 candidates fill a compute unit (their registers), so a launch takes whole rounds of
    // them; what a last round short of blocks would do goes over the whole chip in blocks of 16 or 32 candidates.  Rounds
    // and us with such blocks, without: 64-256-256-1 1.1 23.5, 28.0; 1.4 24.7, 27.9; 3.1 52.0, 55.8; 64-512-512-1, of 32
    // candidates before, 16 now: 1.1 45.0, 46.3; 1.4 47.2, 47.4; 3.1 95.6, 96.8; 64-128-128-1, two blocks a unit: 1.1
    // 15.4, 18.1; 3.1 36.4, 38.4; from an eighth of a round on slower (1.25 18.2, 18.2; 2.2 29.3, 28.3), and for narrower
    // models, with no rounds to speak of, from three rounds on.
    const uint64_t blocks = (n + cands - 1) / cands;
    uint64_t whole = blocks, grid = blocks;
    int last_ct = ct;
    if (by_parts && unit_slots >= 4 && ct == (H1 > 256 ? 2 : 4)) {
        int cus = 256;
        (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, m->device);
        const uint64_t round = (uint64_t)cus * (8 / unit_slots), left = blocks % round;
        if (left && left <= (unit_slots == 8 ? round / 2 : round / 8)) {
            last_ct = ct == 2 || left <= round / 4 ? 1 : 2;
            whole = blocks - left;
            const uint64_t few = 16 * (uint64_t)last_ct;
            grid = whole + (n - whole * cands + few - 1) / few;
        }
    }
    auto kern = !by_parts ? (per == 4   ? score_f32_kernel<1, 4, false, WITH_MIN>
                             : ct == 4 ? score_f32_kernel<4, 1, false, WITH_MIN>
                             : ct == 2 ? score_f32_kernel<2, 1, false, WITH_MIN>
                                       : score_f32_kernel<1, 1, false, WITH_MIN>)
                : per == 4 ? (last_ct < ct ? score_f32_kernel<2, 4, true, WITH_MIN, 1>
                              : ct == 2    ? score_f32_kernel<2, 4, true, WITH_MIN>
                                           : score_f32_kernel<1, 4, true, WITH_MIN>)
                : per == 2 ? (last_ct < ct ? (last_ct == 1 ? score_f32_kernel<4, 2, true, WITH_MIN, 1>
                                                           : score_f32_kernel<4, 2, true, WITH_MIN, 2>)
                              : ct == 4 ? score_f32_kernel<4, 2, true, WITH_MIN>
                              : ct == 2 ? score_f32_kernel<2, 2, true, WITH_MIN>
                                        : score_f32_kernel<1, 2, true, WITH_MIN>)
                           : (ct == 4   ? score_f32_kernel<4, 1, true, WITH_MIN>
                              : ct == 2 ? score_f32_kernel<2, 1, true, WITH_MIN>
                                        : score_f32_kernel<1, 1, true, WITH_MIN>);
    ECK_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(threads), lds, st, net, feat, ld, n, out, unit_slots, x_rows, h_rows,
                       (int)act_bytes, mn, (uint32_t)whole, whole * cands);
    ECK_HIP_TRY(hipGetLastError());
    return ECK_OK;
}

} // namespace

int32_t eck::score_f32(const eck_model *m, const float *feat, uint64_t ld, uint64_t n, float *out, const MinArgs *mn,
                       hipStream_t st)
{
    return mn ? launch<true>(m, feat, ld, n, out, *mn, st) : launch<false>(m, feat, ld, n, out, MinArgs{nullptr, 1, nullptr, 0}, st);
}
