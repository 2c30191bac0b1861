// Forward pass of fp32 models on the matrix cores (HIP, gfx950): costmodel_score for ECK_F32 models of any hidden
// widths (Alg. 1: LatencyEvaAndPick, EnergyModelEvaAndPick; Sec. 5.4).
//
// The network is evaluated transposed, as in the bf16 kernel, on the tiles of f32_tiles.h.  A block's wavefronts share a
// layer's tiles between them as evenly as they go and all read the same activations from LDS.  Weights come straight from
// the parameter vector through the L1: they need neither LDS nor packing.
//
// What bounds it: the fp32 matrix rate (a library product reaches 153 TFLOP/s on this card).  Measured, 64-512-512-1 on
// 32768 candidates: 135 TFLOP/s (144 us; 139 us when the weight loads are left out); 64-256-256-1 on 98304: 121, on 100003
// (a last round of few blocks): 108 (152 us).  The vector kernels before it: 16-18 TFLOP/s (1191 us, 931 us).  What it
// took: weight loads without vector instructions for their addresses (buffer loads with a scalar row offset: 64-bit lane
// addresses cost a quarter of the matrix time), issued one at a time between matrix instructions.
#include <type_traits>

#include "f32_tiles.h"

using namespace eck;
using namespace eck::f32;

namespace {

struct F32Net {
    F32Layer l1, l2;
    const float *w3, *b3;
};

// acc[j][ct] = b + W^T x for a slice and CT tiles of candidates; act: the activations of units 0-3 of this wavefront's
// first candidate, `cands` candidates to a row.  Register q of tile j at quarter p is unit first + J (4p + q) + j.
template <int J, int CT>
__device__ __forceinline__ void slice_product(const F32Layer &l, int first, const f32x4 *act, int cands, int p, int c,
                                              f32x4 (&acc)[4][CT])
{
    const Slice<J> slice(l, first, p, c);
    const int whole = l.K / 16;
    // weights of an even and an odd group; past the end the last whole group again
    float even[4][J], odd[4][J];
    if (whole) {
#pragma unroll
        for (int t = 0; t < 4; ++t) slice.row(0, t, even[t]);
#pragma unroll
        for (int t = 0; t < 4; ++t) slice.row(min(1, whole - 1), t, odd[t]);
    }
#pragma unroll
    for (int j = 0; j < J; ++j) {
        f32x4 bias;
#pragma unroll
        for (int q = 0; q < 4; ++q) bias[q] = l.b[min(first + J * (4 * p + q) + j, l.H - 1)];
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) acc[j][ct] = bias;
    }
    const f32x4 *from = act + p * cands + c;
    f32x4 be[CT], bo[CT]; // activations of an even and an odd group
    auto read_act = [&](int g, f32x4(&b)[CT]) {
#pragma unroll
        for (int ct = 0; ct < CT; ++ct) b[ct] = from[4 * g * cands + 16 * ct];
    };
    auto step = [&](int t, const float (&a)[J], const f32x4 (&b)[CT]) {
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) acc[j][ct] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b[ct][t], acc[j][ct], 0, 0, 0);
    };
    // Two groups per trip, without a branch inside (at one the compiler copies every accumulator, behind a wait for the
    // matrix unit).  The weights of a step are requested for two groups on as soon as the step's matrix instructions are
    // issued: one load at a time, because a wavefront that issues several in a row waits for the load path and leaves
    // the matrix unit idle (all of a group at once: 93 TFLOP/s; none at all, reusing stale weights: 136), and pinned
    // there, because left alone the compiler moves them together.
    const int last = whole - 1;
    int g = 0;
    read_act(0, be);
    for (; g + 2 <= whole; g += 2) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            step(t, even[t], be);
            __builtin_amdgcn_sched_barrier(0);
            slice.row(min(g + 2, last), t, even[t]);
            if (t == 0) read_act(g + 1, bo);
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            step(t, odd[t], bo);
            __builtin_amdgcn_sched_barrier(0);
            slice.row(min(g + 3, last), t, odd[t]);
            if (t == 0) read_act(min(g + 2, last), be);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    if (g < whole) {
#pragma unroll
        for (int t = 0; t < 4; ++t) step(t, even[t], be);
    }
    if (l.K % 16) {
        read_act(whole, be);
        slice.partial_group(whole, even);
#pragma unroll
        for (int t = 0; t < 4; ++t) step(t, even[t], be);
    }
}

// blockDim = 64 * unit_slots * cand_slots: wavefront (us, cs) works on share us of every layer for the CT candidate
// tiles of slot cs.  Every sum has an order that depends on the widths alone, so a candidate's score depends neither on
// n nor on its place.
template <int CT, bool WITH_MIN>
__global__ __launch_bounds__(512, 2) void score_f32_kernel(F32Net net, const float *__restrict__ feat, uint64_t ld,
                                                           uint64_t n, float *__restrict__ out, int unit_slots, int rows4,
                                                           MinArgs mn)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char f32_lds[];
    f32x4 *act = reinterpret_cast<f32x4 *>(f32_lds); // [rows4][cands]
    const int tid = threadIdx.x, lane = tid & 63, p = lane >> 4, c = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int us = wave % unit_slots, cs = wave / unit_slots;
    const int cands = (int)(blockDim.x / 64) / unit_slots * (16 * CT);
    float *part = reinterpret_cast<float *>(act + (int64_t)rows4 * cands); // [unit_slots][cands]
    const uint64_t base = (uint64_t)blockIdx.x * cands;

    for (int e = tid; e < net.l1.K / 4 * cands; e += blockDim.x) { // 32 or 64 features
        const int cand = e % cands, four = e / cands;
        const uint64_t col = base + cand < n ? base + cand : n - 1;
        f32x4 v;
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = feat[(uint64_t)(4 * four + t) * ld + col];
        act[e] = v;
    }
    __syncthreads();
    const f32x4 *mine = act + cs * (16 * CT);
    f32x4 acc[4][CT];
    // this wavefront's share of the 16-unit tiles of a layer: the first shares are a tile larger when they do not divide
    auto share_of = [&](const F32Layer &l, int *first) {
        const int tiles = (l.H + 15) / 16, base_tiles = tiles / unit_slots, more = tiles % unit_slots;
        *first = 16 * (us * base_tiles + min(us, more));
        return base_tiles + (us < more ? 1 : 0);
    };
    int first1, first2;
    const int tiles1 = share_of(net.l1, &first1), tiles2 = share_of(net.l2, &first2);
    auto product = [&](const F32Layer &l, int tiles, int first) {
        if (tiles == 4) slice_product<4, CT>(l, first, mine, cands, p, c, acc);
        else if (tiles == 3) slice_product<3, CT>(l, first, mine, cands, p, c, acc);
        else if (tiles == 2) slice_product<2, CT>(l, first, mine, cands, p, c, acc);
        else if (tiles == 1) slice_product<1, CT>(l, first, mine, cands, p, c, acc);
    };
    product(net.l1, tiles1, first1);
    __syncthreads(); // every wavefront has read the features: their place takes the first hidden layer
    auto store = [&](auto tiles) {
        constexpr int J = decltype(tiles)::value;
        const int unit0 = first1 + 4 * J * p; // this lane's 4 J consecutive units
#pragma unroll
        for (int ct = 0; ct < CT; ++ct)
#pragma unroll
            for (int m = 0; m < J; ++m) {
                f32x4 v;
                // (a unit past H1 is zero; its weights in the next layer are, too)
#pragma unroll
                for (int t = 0; t < 4; ++t) {
                    const int e = 4 * m + t;
                    v[t] = unit0 + e < net.l1.H ? fmaxf(acc[e % J][ct][e / J], 0.0f) : 0.0f;
                }
                if (unit0 / 4 + m < rows4) act[(unit0 / 4 + m) * cands + 16 * (cs * CT + ct) + c] = v;
            }
    };
    if (tiles1 == 4) store(std::integral_constant<int, 4>());
    else if (tiles1 == 3) store(std::integral_constant<int, 3>());
    else if (tiles1 == 2) store(std::integral_constant<int, 2>());
    else if (tiles1 == 1) store(std::integral_constant<int, 1>());
    __syncthreads();
    float y[CT] = {};
    product(net.l2, tiles2, first2);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (j >= tiles2) break;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int unit = first2 + tiles2 * (4 * p + q) + j;
            const float w = net.w3[min(unit, net.l2.H - 1)];
#pragma unroll
            for (int ct = 0; ct < CT; ++ct) y[ct] = unit < net.l2.H ? fmaf(fmaxf(acc[j][ct][q], 0.0f), w, y[ct]) : y[ct];
        }
    }
#pragma unroll
    for (int ct = 0; ct < CT; ++ct) {
        y[ct] += __shfl_xor(y[ct], 16);
        y[ct] += __shfl_xor(y[ct], 32);
        if (p == 0) part[us * cands + 16 * (cs * CT + ct) + c] = y[ct];
    }
    __syncthreads();
    if (tid >= cands) return;
    const uint64_t cand = base + tid;
    float total = net.b3[0];
    for (int s = 0; s < unit_slots; ++s) total += part[s * cands + tid];
    if (cand < n) out[cand] = total;
    if (WITH_MIN) {
        uint32_t key = 0xFFFFFFFFu;
        if (cand < n && (!mn.legal || mn.legal[cand]) && total == total) key = score_order_key(total);
        // sixteen neighbouring candidates lie in one segment as a rule: one atomic for them
        const uint64_t head = base + (tid & ~15), last = head + 15 < n ? head + 15 : n - 1;
        if (head >= n) return;
        const uint64_t seg = head / mn.seg_len;
        if (last / mn.seg_len == seg) {
#pragma unroll
            for (int off = 8; off > 0; off >>= 1) key = min(key, (uint32_t)__shfl_xor((int)key, off));
            if ((tid & 15) == 0 && key != 0xFFFFFFFFu)
                (void)__hip_atomic_fetch_min(mn.min_key + seg, key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        } else if (key != 0xFFFFFFFFu) {
            (void)__hip_atomic_fetch_min(mn.min_key + cand / mn.seg_len, key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}

template <bool WITH_MIN>
int32_t launch(const eck_model *m, const float *feat, uint64_t ld, uint64_t n, float *out, const MinArgs &mn, hipStream_t st)
{
    const int F = m->widths[0], H1 = m->widths[1], H2 = m->widths[2];
    if ((n + 31) / 32 > 0x7FFFFFFFull) return ECK_EUNSUPPORTED;
    const F32Net net{{m->d_state + m->off_w[0], m->d_state + m->off_b[0], F, H1},
                     {m->d_state + m->off_w[1], m->d_state + m->off_b[1], H1, H2},
                     m->d_state + m->off_w[2], m->d_state + m->off_b[2]};
    const int widest = H1 > H2 ? H1 : H2, unit_slots = (widest + 63) / 64; // at most eight
    // As few wavefronts as four tiles each allow share a layer (two tiles each: 67.7 against 63.4 us, 64-128-128-1 on
    // 131072 candidates; 165 against 153 us, 64-256-256-1 on 100003).  Four candidate tiles per wavefront quarter the
    // weight reads per candidate; fewer when blocks that large would leave compute units without two of them.  At least
    // four wavefronts a block (63 against 94 us at 128 units), as long as that leaves enough blocks, too.  Narrow models with
    // many candidates wait for the features: two candidate tiles leave the registers for twice as many wavefronts (2^20
    // candidates, four against two: 32-1-1-1 65.8 and 53.3 us, 32-64-64-1 160 and 153; 2^18 15.5 and 14.1, 41 and 41; 2^17
    // 8.0 and 8.2, 20.1 and 22.2).
    const uint64_t tiles = (n + 15) / 16;
    int cand_slots = unit_slots < 4 ? 4 / unit_slots : 1, ct = unit_slots == 1 && tiles >= 16384 ? 2 : 4;
    while (ct > 1 && tiles < 512ull * cand_slots * ct) ct /= 2;
    while (cand_slots > 1 && tiles < 512ull * cand_slots * ct) cand_slots /= 2;
    const int cands = 16 * ct * cand_slots, rows4 = ((F > H1 ? F : H1) + 15) / 16 * 4;
    const size_t lds = (size_t)rows4 * cands * 16 + (size_t)unit_slots * cands * 4;
    auto kern = ct == 4 ? score_f32_kernel<4, WITH_MIN> : ct == 2 ? score_f32_kernel<2, WITH_MIN> : score_f32_kernel<1, WITH_MIN>;
    ECK_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void *>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(kern, dim3((unsigned)((n + cands - 1) / cands)), dim3(64 * unit_slots * cand_slots), lds, st, net, feat,
                       ld, n, out, unit_slots, rows4, mn);
    ECK_HIP_TRY(hipGetLastError());
    return ECK_OK;
}

} // namespace

int32_t eck::score_f32(const eck_model *m, const float *feat, uint64_t ld, uint64_t n, float *out, const MinArgs *mn,
                       hipStream_t st)
{
    return mn ? launch<true>(m, feat, ld, n, out, *mn, st) : launch<false>(m, feat, ld, n, out, MinArgs{nullptr, 1, nullptr, 0}, st);
}
