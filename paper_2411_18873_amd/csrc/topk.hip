// Selection under the "low latency first, then least energy" objective
// (Sec. 4.3, 4.4; Alg. 1 LatencyEvaAndPick / EnergyModelEvaAndPick).  HIP, gfx950.
//
// Method: a tournament of exact block-local selections.  Every candidate is the composite key
// (order-preserving score bits, index within its segment); composites of one segment are distinct, so
// "the k smallest" is a unique set and ties fall to the lower index.  Level 0 reads the score arrays
// ONCE: a block takes a chunk of one segment, keeps the composites of its feasible candidates in
// registers, finds its own k smallest with a radix select on LDS histograms (nothing leaves the
// block) and writes just those.  Every further level does the same on the lists of the level before
// it, until one block per segment holds the segment's k smallest, sorts them in LDS and writes the
// result.  The k smallest of a segment are among the k smallest of each chunk, so the result is exact;
// no global atomics, no flags between blocks: blocks only meet at kernel boundaries, and the output does
// not depend on execution order.  Inside a block: a cheap upper bound on its k-th smallest key first (from
// the least key of every thread), then the few candidates under the bound are sorted; a radix select on LDS histograms takes
// over when many remain.
#include <mutex>

#include "eck_internal.h"
#include "lanes.h"

using namespace eck;

namespace {

constexpr int DIGIT_BITS = 11;
constexpr int BINS = 1 << DIGIT_BITS;
#ifndef ECK_TOPK_ITEMS
#define ECK_TOPK_ITEMS 16
#endif
constexpr int ITEMS = ECK_TOPK_ITEMS;                // composites a thread holds
constexpr uint64_t NONE = ~0ull;         // no candidate (a NaN score never makes a composite, so no composite is all ones)
constexpr uint32_t LATMIN_PARTS = 256;   // most per-block latency minima per segment
constexpr int SCAN_CHUNK = 4096;         // candidates per block of the scan under the latency gate ...
constexpr uint32_t SCAN_LIST = 128;      // ... entries of its list ...
constexpr uint32_t SCAN_PARTS = 1024;    // ... and most of its blocks per segment

enum Pred { PRED_PLAIN = 0, PRED_THRESHOLD = 1, PRED_RANK = 2 };
// (SRC_SCANNED: the scores, of which scan_kernel listed those that may be feasible)
enum Source { SRC_SCORES_VEC = 0, SRC_SCORES = 1, SRC_LIST = 2, SRC_SCANNED_VEC = 3, SRC_SCANNED = 4 };

__device__ __forceinline__ float key_to_float(uint32_t k)
{
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

struct SelectArgs {
    const float *energy;
    const float *latency;
    const uint8_t *legal;
    uint64_t seg_len;
    uint32_t idx_bits;          // composite = key << idx_bits | idx
    float slack_factor;         // alpha - 1 (THRESHOLD)
    int alpha_inf;
    const uint32_t *lat_parts;  // THRESHOLD: [S][lat_parts_n] least latency order keys, one per block of latmin_kernel
    uint32_t lat_parts_n;       // 0: one block holds the whole segment and finds the least key itself
    const uint32_t *listed;     // SRC_SCANNED: [S][lat_parts_n] candidates under the gate of every chunk's own minimum ...
    const uint64_t *scan_lists; // ... and [S][lat_parts_n][SCAN_LIST] the first of them, latency bits << 32 | index
    const uint64_t *list_in;    // SRC_LIST: [S][list_len] composites of the level before, NONE where empty
    uint64_t list_len;
    uint64_t *list_out;         // not the last level: [S][gridDim.x][k]
    uint32_t k;                 // composites this tournament selects; RANK: by latency, m_latency of them ...
    uint32_t k_energy;          // ... among which the last level selects this many by energy (else 0)
    uint32_t *idx_out;          // last level: the result
    float *energy_out;
    uint32_t *count_out;
};

// ---------------------------------------------------------------- the latency gate (THRESHOLD)

// tau = L_min + (alpha - 1) |L_min|, product and sum rounded separately; `best`: the order key of L_min, all ones when
// nothing is legal (nothing will be feasible then either)
__device__ __forceinline__ float gate_above(uint32_t best, float slack_factor)
{
    if (best == 0xFFFFFFFFu) return __builtin_inff();
    const float lmin = key_to_float(best);
    return __fadd_rn(lmin, __fmul_rn(slack_factor, fabsf(lmin)));
}

// least order key of a legal, non-NaN latency in this block's slice of the segment; no atomics, so nothing
// has to be initialised: every block writes its slot
template <bool VEC>
__global__ __launch_bounds__(256) void latmin_kernel(const float *__restrict__ latency, const uint8_t *__restrict__ legal,
                                                     uint64_t seg_len, uint64_t slice, uint32_t *__restrict__ parts)
{
    const uint32_t s = blockIdx.y;
    const uint64_t seg_base = (uint64_t)s * seg_len;
    const uint64_t lo = (uint64_t)blockIdx.x * slice, hi = lo + slice < seg_len ? lo + slice : seg_len;
    uint32_t best = 0xFFFFFFFFu;
    if (VEC) {
        for (uint64_t i = lo + 4ull * threadIdx.x; i < hi; i += 4ull * 256) {
            const uint64_t g = seg_base + i;
            uint32_t flags = 0x01010101u;
            if (legal) flags = *reinterpret_cast<const uint32_t *>(legal + g);
            if (!flags) continue;
            const float4 l = *reinterpret_cast<const float4 *>(latency + g);
            const float lv[4] = {l.x, l.y, l.z, l.w};
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (((flags >> (8 * t)) & 0xFFu) && lv[t] == lv[t]) best = min(best, score_order_key(lv[t]));
        }
    } else {
        for (uint64_t i = lo + threadIdx.x; i < hi; i += 256) {
            const uint64_t g = seg_base + i;
            if (legal && !legal[g]) continue;
            const float l = latency[g];
            if (l == l) best = min(best, score_order_key(l));
        }
    }
    best = wave_least(best);
    __shared__ uint32_t wave_best[4];
    if ((threadIdx.x & 63) == 0) wave_best[threadIdx.x >> 6] = best;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w) best = min(best, wave_best[w]);
        parts[(uint64_t)s * gridDim.x + blockIdx.x] = best;
    }
}

// One pass over latencies and flags for both the least latency and what lies under the gate.  A block takes SCAN_CHUNK
// candidates of a segment, finds their least legal latency and lists those under the gate that this least latency would
// open: a superset of the chunk's feasible candidates as long as the segment's gate lies no higher, which the next launch
// checks, as it does that the list has not overflowed (it reads the chunk again otherwise).  Where a gate admits few,
// the latencies are thus read once and energies only for the listed.  Bound by the stream of latencies and flags.  64
// segments of 2^18, alpha = 1.1: 14.5-16 us here and 9 in the next launch, where a pass for the minima alone takes 14.2 and the
// next one, reading the latencies again, 21.2; where the gate admits everything, 15 and 31 against 14 and 33.
template <bool VEC>
__global__ __launch_bounds__(256) void scan_kernel(const float *__restrict__ latency, const uint8_t *__restrict__ legal,
                                                   uint64_t seg_len, float slack_factor, uint32_t *__restrict__ least,
                                                   uint32_t *__restrict__ listed, uint64_t *__restrict__ lists)
{
    constexpr int PER = SCAN_CHUNK / 256;
    __shared__ uint32_t wave_best[4], cursor;
    const uint64_t seg_base = (uint64_t)blockIdx.y * seg_len, start = (uint64_t)blockIdx.x * SCAN_CHUNK;
    const uint64_t slot = (uint64_t)blockIdx.y * gridDim.x + blockIdx.x;
    if (threadIdx.x == 0) cursor = 0;
    float l[PER];
    uint32_t on = 0; // bit j: candidate j is legal and its latency a number
    auto index_of = [&](int j) -> uint64_t {
        return VEC ? start + ((uint64_t)(j / 4) * 256 + threadIdx.x) * 4 + j % 4 : start + (uint64_t)j * 256 + threadIdx.x;
    };
    if (VEC) {
        // every load of the thread before anything waits; groups past the end re-read the segment's first group
        float4 l4[PER / 4];
        uint32_t flags[PER / 4];
#pragma unroll
        for (int j = 0; j < PER / 4; ++j) {
            const uint64_t i = index_of(4 * j), g = seg_base + (i < seg_len ? i : 0);
            flags[j] = legal ? *reinterpret_cast<const uint32_t *>(legal + g) : 0x01010101u;
            l4[j] = *reinterpret_cast<const float4 *>(latency + g);
        }
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            l[j] = j % 4 == 0 ? l4[j / 4].x : j % 4 == 1 ? l4[j / 4].y : j % 4 == 2 ? l4[j / 4].z : l4[j / 4].w;
            if (((flags[j / 4] >> (8 * (j % 4))) & 0xFFu) && index_of(j) < seg_len && l[j] == l[j]) on |= 1u << j;
        }
    } else {
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            const uint64_t i = index_of(j), g = seg_base + (i < seg_len ? i : 0);
            l[j] = latency[g];
            if (i < seg_len && (!legal || legal[g]) && l[j] == l[j]) on |= 1u << j;
        }
    }
    uint32_t best = 0xFFFFFFFFu;
#pragma unroll
    for (int j = 0; j < PER; ++j) best = min(best, (on >> j) & 1u ? score_order_key(l[j]) : 0xFFFFFFFFu);
    best = wave_least(best);
    if ((threadIdx.x & 63) == 0) wave_best[threadIdx.x >> 6] = best;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < 4; ++w) best = min(best, wave_best[w]);
    const float tau = gate_above(best, slack_factor);
    uint32_t under = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j)
        if (l[j] <= tau) under |= 1u << j;
    under &= on;
    // places by a prefix sum over the wavefront and one LDS atomic (an atomic per thread: 10 us more where a gate admits
    // everything); a wavefront that overflows the list alone writes nothing
    const uint32_t mine = (uint32_t)__popc(under);
    const uint32_t upto = wave_prefix_sum(mine);
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)upto, 63);
    uint32_t at = 0;
    if ((threadIdx.x & 63) == 0 && total) at = atomicAdd(&cursor, total);
    at = (uint32_t)__builtin_amdgcn_readfirstlane((int)at);
    if (total && total <= SCAN_LIST && at < SCAN_LIST) {
        at += upto - mine;
#pragma unroll
        for (int j = 0; j < PER; ++j)
            if ((under >> j) & 1u) {
                if (at < SCAN_LIST) lists[slot * SCAN_LIST + at] = ((uint64_t)__float_as_uint(l[j]) << 32) | index_of(j);
                ++at;
            }
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        least[slot] = best;
        listed[slot] = cursor;
    }
}

// ---------------------------------------------------------------- one level of the tournament

constexpr uint32_t NO_KEY = 0xFFFFFFFFu; // the order key of no number (only a NaN pattern maps to it): "not a candidate"
constexpr uint32_t SMALL = 1024;         // a selection among at most this many composites is ranked directly
constexpr uint32_t BOUNDED = 512;        // selections of more are not bounded: at least as many lie under any bound

// order key of a legal candidate's value under predicate PRED, or NO_KEY if infeasible
template <int PRED>
__device__ __forceinline__ uint32_t feasible_key(float e, float l, float tau)
{
    if (PRED == PRED_THRESHOLD && !(l <= tau)) return NO_KEY;
    const float value = PRED == PRED_RANK ? l : e;
    return value != value ? NO_KEY : score_order_key(value);
}

// LDS of a block: the digit histogram of the radix select, or the arrays of the direct ranking (never both at
// once), a handful of words, and (last level) the sort buffer behind them
template <int T>
struct Shared {
    union {
        uint32_t hist[BINS];
        uint64_t pool[SMALL]; // the composites left after the bound, then the selection in ascending order
    };
    uint32_t wave_sum[T / 64];
    uint64_t wave_bound[T / 64];
    uint32_t found_digit, found_below, found_count, cursor;
    uint32_t lat_min;
    uint64_t any_composite; // radix select: one of the block's composites, to find the leading bits all of them share
};

// the 64 values of a wavefront in ascending order over the lanes (bitonic sorting network)
template <class V>
__device__ __forceinline__ V wave_sort(V v)
{
    const uint32_t lane = threadIdx.x & 63;
#pragma unroll
    for (uint32_t size = 2; size <= 64; size <<= 1)
#pragma unroll
        for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
            const V other = lane_exchange(v, stride);
            const bool keep_min = ((lane & stride) == 0) == ((lane & size) == 0);
            const V lo = v < other ? v : other, hi = v < other ? other : v;
            v = keep_min ? lo : hi;
        }
    return v;
}

// A bound on the block's k-th smallest value, from the least value of every thread (V = order key or composite,
// `none` = the largest value of V, which stands for "nothing").  Each of the W wavefronts contributes
// need = ceil(k / W) values that are at most its part of the bound, k or more in all, so the k-th smallest of the
// block does not exceed the largest part.  A wavefront's part: the need-th smallest of its 64 sorted values (for
// need <= 2 the larger of the minima of `need` halves of the wavefront does: six exchange steps instead of 21).  `none` when some wavefront has too few values (then nothing may be dropped) or k is too
// large for this.
template <int T, class V>
__device__ __forceinline__ V block_bound(V least, uint32_t k, V none, Shared<T> &sh)
{
    constexpr uint32_t W = T / 64;
    const uint32_t need = (k + W - 1) / W;
    if (need > 64) return none;
    V part;
    if (need <= 2) {
        const uint32_t groups = need, lanes = 64 / groups;
        part = least;
#pragma unroll
        for (uint32_t stride = 1; stride < 64; stride <<= 1) {
            const V other = lane_exchange(part, stride);
            const V lo = part < other ? part : other, hi = part < other ? other : part;
            part = stride < lanes ? lo : hi;
        }
    } else {
        const V sorted = wave_sort<V>(least);
        uint64_t picked = (uint32_t)__shfl((int)(uint32_t)sorted, (int)(need - 1));
        if (sizeof(V) == 8)
            picked |= (uint64_t)(uint32_t)__shfl((int)(uint32_t)((uint64_t)sorted >> 32), (int)(need - 1)) << 32;
        part = (V)picked;
    }
    if ((threadIdx.x & 63) == 0) sh.wave_bound[threadIdx.x >> 6] = part;
    __syncthreads();
    uint64_t bound = 0;
#pragma unroll
    for (uint32_t w = 0; w < W; ++w) bound = sh.wave_bound[w] > bound ? sh.wave_bound[w] : bound;
    return (V)bound; // one wavefront without enough values makes `none` the bound
}

// Sorts the `kept` (<= SMALL) composites of sh.pool: runs of 64 in registers, a wavefront each, then the place of a
// composite is the number of smaller ones in every run, by binary search (composites are distinct).  (Counting the smaller
// ones entry by entry, shared between the threads, is as fast up to some 150; 512 among 256 threads took 10 us.)
template <int T>
__device__ __forceinline__ void rank_pool(uint32_t kept, Shared<T> &sh)
{
    constexpr int W = T / 64, PER = SMALL / 64 > W ? SMALL / 64 / W : 1;
    const uint32_t runs = (kept + 63) / 64, lane = threadIdx.x & 63;
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    uint64_t v[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const uint32_t run = wave + (uint32_t)(i * W), at = 64 * run + lane;
        v[i] = NONE;
        if (run >= runs) continue;
        if (at < kept) v[i] = sh.pool[at];
        v[i] = wave_sort<uint64_t>(v[i]);
        sh.pool[at] = v[i];
    }
    __syncthreads();
    if (runs <= 1) return;
    uint32_t place[PER];
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        place[i] = 0;
        if (wave + (uint32_t)(i * W) >= runs) continue;
        for (uint32_t q = 0; q < runs; q += 4) { // four searches at a time: one by one their reads wait for each other
            uint32_t below[4] = {0, 0, 0, 0};
#pragma unroll
            for (uint32_t step = 32; step > 0; step >>= 1)
#pragma unroll
                for (int t = 0; t < 4; ++t) below[t] += sh.pool[64 * (q + t) + below[t] + step - 1] < v[i] ? step : 0;
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                below[t] += sh.pool[64 * (q + t) + below[t]] < v[i];
                place[i] += q + t < runs ? below[t] : 0; // (past the last run: left over, not counted)
            }
        }
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < PER; ++i)
        if (v[i] != NONE) sh.pool[place[i]] = v[i];
    __syncthreads();
}

// Radix select from the top digit down over the composites a thread holds (NONE entries do not count): the
// composite that exactly k of them do not exceed (there are at least k).  Histogram of the digit over the
// composites that match the digits fixed so far, prefix sums over the bins, the bin holding the wanted rank
// fixes the next digit; ends as soon as a whole bin is wanted.
template <int T>
__device__ uint64_t radix_threshold(const uint64_t (&c)[ITEMS], uint32_t k, uint32_t total_bits, Shared<T> &sh)
{
    constexpr int PER = BINS / T; // consecutive bins per thread in the scan
    // The leading bits that all composites of the block share select nothing: scores of one segment lie in a narrow
    // range, so without this the first digit (sign, exponent, two mantissa bits) sends every composite to a
    // handful of bins, whose LDS atomics serialise, and a pass is spent on it.
    uint64_t mine = NONE;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) mine = c[j] != NONE ? c[j] : mine;
    __syncthreads(); // the words used below may still be read from what came before
    if (mine != NONE) sh.any_composite = mine; // whichever thread's store lands last
    __syncthreads();
    const uint64_t ref = sh.any_composite;
    uint64_t differ = 0;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) differ |= c[j] != NONE ? c[j] ^ ref : 0;
#pragma unroll
    for (uint32_t stride = 32; stride > 0; stride >>= 1) differ |= lane_exchange(differ, stride);
    if ((threadIdx.x & 63) == 0) sh.wave_bound[threadIdx.x >> 6] = differ;
    __syncthreads();
    differ = 0;
#pragma unroll
    for (int w = 0; w < T / 64; ++w) differ |= sh.wave_bound[w];
    if (differ == 0) return ref; // a single composite
    uint32_t top = 64 - (uint32_t)__clzll((long long)differ);
    top = top < total_bits ? top : total_bits;
    uint64_t prefix = top < 64 ? (ref >> top) << top : 0;
    uint32_t remaining = k;
    for (;;) {
        const uint32_t bits = top < (uint32_t)DIGIT_BITS ? top : (uint32_t)DIGIT_BITS;
        const uint32_t shift = top - bits, mask = (1u << bits) - 1;
        __syncthreads(); // the histogram's space and found_* may still be read from the pass (or the use) before
#pragma unroll
        for (int j = 0; j < PER; ++j) sh.hist[threadIdx.x * PER + j] = 0;
        __syncthreads();
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const uint64_t v = c[j];
            // (a shift by 64 is undefined: the first pass of a 64-bit composite has no digits above it)
            const bool in_prefix = top >= 64 || (v >> top) == (prefix >> top);
            if (v != NONE && in_prefix) atomicAdd(&sh.hist[(uint32_t)(v >> shift) & mask], 1u);
        }
        __syncthreads();
        uint32_t local[PER], sum = 0;
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            local[j] = sh.hist[threadIdx.x * PER + j];
            sum += local[j];
        }
        const uint32_t incl = wave_prefix_sum(sum);
        if ((threadIdx.x & 63) == 63) sh.wave_sum[threadIdx.x >> 6] = incl;
        __syncthreads();
        uint32_t below = incl - sum;
#pragma unroll
        for (int w = 0; w < T / 64; ++w)
            if (w < (int)(threadIdx.x >> 6)) below += sh.wave_sum[w];
#pragma unroll
        for (int j = 0; j < PER; ++j) {
            if (below < remaining && remaining <= below + local[j]) {
                sh.found_digit = threadIdx.x * PER + j;
                sh.found_below = below;
                sh.found_count = local[j];
            }
            below += local[j];
        }
        __syncthreads();
        const uint64_t digit = sh.found_digit;
        const uint32_t under = sh.found_below, count = sh.found_count;
        prefix |= digit << shift;
        remaining -= under;
        if (shift == 0 || remaining == count) return prefix | ((shift ? (1ull << shift) : 1ull) - 1);
        top = shift;
    }
}

// The block's min(k, #candidates) smallest composites, c[j] = NONE standing for "no candidate" (entries above the
// bound are set to NONE on the way).  Returns their number n.  Either *ranked is set and sh.pool[0 .. n)
// holds them in ascending order, or it is clear and they are the composites c[j] <= *thr.
// `kept`: how many entries of c are candidates within the bound; when at most SMALL, they are already in
// sh.pool (the caller compacted them while it built c) and get ranked directly; more go through the radix
// select.  `bounded`: a bound was applied, which only happens when at least k candidates lie within it.
template <int T>
__device__ uint32_t select_kept(const uint64_t (&c)[ITEMS], uint32_t kept, bool bounded, uint32_t k, uint32_t total_bits,
                                Shared<T> &sh, bool *ranked, uint64_t *thr)
{
    const uint32_t n = kept < k ? kept : k;
    *thr = NONE - 1; // every composite is below NONE
    *ranked = false;
    if (kept <= SMALL) {
        rank_pool<T>(kept, sh);
        *ranked = true;
        return n;
    }
    if (!bounded && kept <= k) return n; // all of them, in no order
    *thr = radix_threshold<T>(c, k, total_bits, sh);
    return n;
}

// Appends the composites c[j] for which take(j) to the pool, which sh.cursor counts; those past its end are counted only.
// Places from ballots, one LDS atomic per wavefront.  (An atomic per composite, each behind the answer to the one before:
// up to 1 us.)
template <int T, class Take>
__device__ __forceinline__ void append(const uint64_t (&c)[ITEMS], Take take, Shared<T> &sh)
{
    uint64_t on[ITEMS];
    uint32_t total = 0;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        on[j] = __ballot(take(j));
        total += (uint32_t)__popcll(on[j]);
    }
    if (!total) return;
    uint32_t base = 0;
    if ((threadIdx.x & 63) == 0) base = atomicAdd(&sh.cursor, total);
    base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        if (!on[j]) continue;
        const uint32_t at = __builtin_amdgcn_mbcnt_hi((uint32_t)(on[j] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)on[j], base));
        if (take(j) && at < SMALL) sh.pool[at] = c[j];
        base += (uint32_t)__popcll(on[j]);
    }
}

// The number of the candidates c[j] != NONE, which are compacted into the pool as far as they go.  sh.cursor must have been
// set to zero, and the pool's space be free.
template <int T>
__device__ __forceinline__ uint32_t keep_all(const uint64_t (&c)[ITEMS], Shared<T> &sh)
{
    __syncthreads();
    append<T>(c, [&](int j) { return c[j] != NONE; }, sh);
    __syncthreads();
    return sh.cursor;
}

// The candidates among c, of which `least` is the least, bounded and the survivors compacted into the pool, which sh.cursor
// counts (it must have been set to zero); returns their number.
template <int T>
__device__ __forceinline__ uint32_t bound_candidates(uint64_t (&c)[ITEMS], uint64_t least, uint32_t k, Shared<T> &sh, bool *bounded)
{
    const uint64_t bound = block_bound<T, uint64_t>(least, k, NONE, sh);
    *bounded = bound != NONE;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) c[j] = c[j] > bound ? NONE : c[j]; // bound == NONE keeps everything
    append<T>(c, [&](int j) { return c[j] != NONE; }, sh);
    __syncthreads();
    return sh.cursor;
}

// The block's share of a list of composites (the selections of the level before): held in c, bounded, the
// survivors compacted into the pool.
template <int T>
__device__ __forceinline__ void gather_list(const uint64_t *in, uint64_t list_len, uint64_t start, uint32_t k,
                                            Shared<T> &sh, uint64_t (&c)[ITEMS], uint32_t *kept, bool *bounded)
{
    const uint64_t share = list_len - start < (uint64_t)(T * ITEMS) ? list_len - start : (uint64_t)(T * ITEMS);
    if (k > BOUNDED) {
        // no bound can leave few enough for the direct ranking: plain coalesced loads, everything kept
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const uint64_t i = (uint64_t)j * T + threadIdx.x;
            c[j] = i < share ? in[start + i] : NONE;
        }
        *bounded = false;
        *kept = keep_all<T>(c, sh);
        return;
    }
    // Neighbouring threads share a list, `near` of them, every near-th entry each, and the lists go round the wavefronts: the
    // lists of blocks that ranked their selection are ascending, so the least entries of the threads are the first of each
    // list and the bound comes out tight (64 lists of 128: 200 of 8192 entries left; 900 where a thread takes consecutive
    // entries, which were then too many to rank directly).  Consecutive entries where whole lists do not go into the threads.
    uint32_t per_thread = (uint32_t)((share + T - 1) / T), near = 0; // per_thread <= ITEMS
#pragma unroll 1
    for (uint32_t per = per_thread; per <= (uint32_t)ITEMS && !near; ++per) {
        uint32_t n = 1;
        while (n * per < k) n *= 2;
        if (n <= 64 && (uint64_t)(T / n) * k >= share) near = n, per_thread = per;
    }
    const uint32_t lane = threadIdx.x & 63, wave = threadIdx.x >> 6, stride = near ? near : 1;
    const uint32_t at = near ? lane % near : 0; // in the list
    const uint32_t first = near ? (lane / near * (T / 64) + wave) * k + at : threadIdx.x * per_thread;
    const uint32_t room = near ? (k - at + near - 1) / near : per_thread; // (at < k + near)
    uint64_t least = NONE;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
        const uint32_t i = first + (uint32_t)j * stride;
        uint64_t v = NONE;
        if ((uint32_t)j < per_thread && (uint32_t)j < room && i < share) v = in[start + i];
        c[j] = v;
        least = v < least ? v : least;
    }
    *kept = bound_candidates<T>(c, least, k, sh, bounded);
}

// the least of a key over the block
template <int T>
__device__ __forceinline__ uint32_t block_least(uint32_t best, Shared<T> &sh)
{
    best = wave_least(best);
    if (threadIdx.x == 0) sh.lat_min = 0xFFFFFFFFu;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) atomicMin(&sh.lat_min, best);
    __syncthreads();
    return sh.lat_min;
}

// The block's chunk of T * ITEMS candidates of segment s (four consecutive candidates per load where VEC allows
// it): order keys of the feasible ones, bounded, the survivors turned into composites (held in c and compacted into
// the pool).  `known`: the least of the segment's minima, or null: not looked yet.
template <int T, int SRC, int PRED>
__device__ __forceinline__ void gather_scores(const SelectArgs &a, uint32_t s, Shared<T> &sh, uint64_t (&c)[ITEMS],
                                              uint32_t *kept, bool *bounded, const uint32_t *known)
{
    constexpr bool NEED_E = PRED != PRED_RANK, NEED_L = PRED != PRED_PLAIN;
    const uint64_t seg_base = (uint64_t)s * a.seg_len;
    const uint64_t start = (uint64_t)blockIdx.x * (T * ITEMS);
    // VEC: every load of the thread is issued here, before anything waits; none depends on another (the flags
    // decide afterwards).  Groups past the end of the segment re-read its first group and are discarded.
    // Exception: under a finite latency gate few candidates are feasible as a rule, so the energies are fetched
    // afterwards and only for groups of four that hold a feasible candidate -- a second round trip for those, but
    // close to half the bytes of the pass stay unread.
    constexpr bool ENERGY_LATER = PRED == PRED_THRESHOLD && SRC == SRC_SCORES_VEC;
    const bool energy_later = ENERGY_LATER && !a.alpha_inf;
    uint32_t flags[ITEMS / 4];
    float4 e[ITEMS / 4], l[ITEMS / 4];
    if (SRC == SRC_SCORES_VEC) {
#pragma unroll
        for (int j = 0; j < ITEMS / 4; ++j) {
            const uint64_t i = start + ((uint64_t)j * T + threadIdx.x) * 4;
            const uint64_t g = seg_base + (i < a.seg_len ? i : 0); // seg_len is a multiple of 4 on this path
            flags[j] = a.legal ? *reinterpret_cast<const uint32_t *>(a.legal + g) : 0x01010101u;
            if (NEED_L) l[j] = *reinterpret_cast<const float4 *>(a.latency + g);
            if (NEED_E && !energy_later) e[j] = *reinterpret_cast<const float4 *>(a.energy + g);
        }
    }
    // the gate, while the loads are under way
    float tau = 0.0f;
    if (PRED == PRED_THRESHOLD) {
        // L_min from the per-block minima
        if (a.alpha_inf) {
            tau = __builtin_inff();
        } else {
            uint32_t best = 0xFFFFFFFFu;
            for (uint32_t p = threadIdx.x; !known && p < a.lat_parts_n; p += T) best = min(best, a.lat_parts[(uint64_t)s * a.lat_parts_n + p]);
            if (a.lat_parts_n == 0) { // the segment is this block's chunk
                if (SRC == SRC_SCORES_VEC) {
#pragma unroll
                    for (int j = 0; j < ITEMS / 4; ++j) {
                        const uint64_t i = start + ((uint64_t)j * T + threadIdx.x) * 4;
                        const float lv[4] = {l[j].x, l[j].y, l[j].z, l[j].w};
#pragma unroll
                        for (int t = 0; t < 4; ++t)
                            if (i < a.seg_len && ((flags[j] >> (8 * t)) & 0xFFu) && lv[t] == lv[t]) best = min(best, score_order_key(lv[t]));
                    }
                } else {
#pragma unroll
                    for (int j = 0; j < ITEMS; ++j) {
                        const uint64_t i = start + (uint64_t)j * T + threadIdx.x;
                        if (i < a.seg_len && (!a.legal || a.legal[seg_base + i])) {
                            const float v = a.latency[seg_base + i];
                            if (v == v) best = min(best, score_order_key(v));
                        }
                    }
                }
            }
            tau = gate_above(known ? *known : block_least<T>(best, sh), a.slack_factor);
        }
    }
    // order keys of the feasible candidates (32 bits each: the index is implied by the position), their least
    // per thread, the bound from those
    uint32_t key[ITEMS], least = NO_KEY;
    auto index_of = [&](int j) -> uint32_t {
        if (SRC == SRC_SCORES_VEC) return (uint32_t)(start + ((uint64_t)(j / 4) * T + threadIdx.x) * 4 + (j % 4));
        return (uint32_t)(start + (uint64_t)j * T + threadIdx.x);
    };
    if (SRC == SRC_SCORES_VEC) {
        if (ENERGY_LATER && energy_later) {
            // keep the flags of the feasible candidates only, then fetch the energies of the groups that have any
#pragma unroll
            for (int j = 0; j < ITEMS / 4; ++j) {
                const float lv[4] = {l[j].x, l[j].y, l[j].z, l[j].w};
                uint32_t f = flags[j];
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    if (!(lv[t] <= tau)) f &= ~(0xFFu << (8 * t));
                flags[j] = f;
            }
#pragma unroll
            for (int j = 0; j < ITEMS / 4; ++j) {
                const uint64_t i = start + ((uint64_t)j * T + threadIdx.x) * 4;
                e[j] = float4{0.0f, 0.0f, 0.0f, 0.0f};
                if (flags[j] && i < a.seg_len) e[j] = *reinterpret_cast<const float4 *>(a.energy + seg_base + i);
            }
        }
#pragma unroll
        for (int j = 0; j < ITEMS / 4; ++j) {
            const uint64_t i = start + ((uint64_t)j * T + threadIdx.x) * 4;
            const uint32_t f = i < a.seg_len ? flags[j] : 0u;
            const float ev[4] = {NEED_E ? e[j].x : 0.0f, NEED_E ? e[j].y : 0.0f, NEED_E ? e[j].z : 0.0f, NEED_E ? e[j].w : 0.0f};
            const float lv[4] = {NEED_L ? l[j].x : 0.0f, NEED_L ? l[j].y : 0.0f, NEED_L ? l[j].z : 0.0f, NEED_L ? l[j].w : 0.0f};
#pragma unroll
            for (int t = 0; t < 4; ++t)
                key[4 * j + t] = ((f >> (8 * t)) & 0xFFu) ? feasible_key<PRED>(ev[t], lv[t], tau) : NO_KEY;
        }
    } else {
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const uint64_t i = start + (uint64_t)j * T + threadIdx.x;
            uint32_t v = NO_KEY;
            if (i < a.seg_len) {
                const uint64_t g = seg_base + i;
                if (!a.legal || a.legal[g])
                    v = feasible_key<PRED>(NEED_E ? a.energy[g] : 0.0f, NEED_L ? a.latency[g] : 0.0f, tau);
            }
            key[j] = v;
        }
    }
    if (a.k > BOUNDED) {
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) c[j] = key[j] != NO_KEY ? ((uint64_t)key[j] << a.idx_bits) | index_of(j) : NONE;
        *bounded = false;
        *kept = keep_all<T>(c, sh);
        return;
    }
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) least = min(least, key[j]);
    const uint32_t bound = block_bound<T, uint32_t>(least, a.k, NO_KEY, sh);
    *bounded = bound != NO_KEY;
    __syncthreads();
    // the candidates within the bound (all of one key, ties included) become composites
    const uint32_t most = bound == NO_KEY ? NO_KEY - 1 : bound;
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) c[j] = key[j] <= most ? ((uint64_t)key[j] << a.idx_bits) | index_of(j) : NONE;
    append<T>(c, [&](int j) { return key[j] <= most; }, sh);
    __syncthreads();
    *kept = sh.cursor;
}

// The same from what scan_kernel listed of the chunk, one list entry per thread: false when the lists do not tell (one
// overflowed, or the segment's gate lies above the one that a list was made under), the same answer in every thread.
// *best: the least of the segment's minima.
template <int T>
__device__ __forceinline__ bool gather_scanned(const SelectArgs &a, uint32_t s, Shared<T> &sh, uint64_t (&c)[ITEMS],
                                               uint32_t *kept, bool *bounded, uint32_t *best)
{
    constexpr uint32_t LISTS = (uint32_t)(T * ITEMS) / SCAN_CHUNK; // of this block's chunk; at most SMALL entries
    static_assert(LISTS * SCAN_LIST <= SMALL && LISTS * SCAN_LIST <= (uint32_t)T, "");
    const uint32_t *least = a.lat_parts + (uint64_t)s * a.lat_parts_n, *listed = a.listed + (uint64_t)s * a.lat_parts_n;
    const uint32_t first = blockIdx.x * LISTS, mine = threadIdx.x / SCAN_LIST;
    // every thread looks at all of the block's lists, so that no barrier has to bring their answers together
    uint32_t count[LISTS], own[LISTS];
#pragma unroll
    for (uint32_t k = 0; k < LISTS; ++k) {
        const uint32_t at = min(first + k, a.lat_parts_n - 1);
        count[k] = listed[at];
        own[k] = least[at];
    }
    uint64_t entry = 0; // (past the list's end: left over from earlier calls, not looked at)
    if (mine < LISTS && first + mine < a.lat_parts_n) entry = a.scan_lists[((uint64_t)s * a.lat_parts_n + first + mine) * SCAN_LIST + threadIdx.x % SCAN_LIST];
    uint32_t lowest = 0xFFFFFFFFu;
    for (uint32_t p = threadIdx.x; p < a.lat_parts_n; p += T) lowest = min(lowest, least[p]);
    lowest = wave_least(lowest);
    if ((threadIdx.x & 63) == 0) sh.wave_sum[threadIdx.x >> 6] = lowest;
    __syncthreads();
#pragma unroll
    for (uint32_t w = 0; w < T / 64; ++w) lowest = min(lowest, sh.wave_sum[w]);
    *best = lowest;
    const float tau = gate_above(lowest, a.slack_factor);
    uint32_t from = 0; // entries of this thread's list that may be feasible
#pragma unroll
    for (uint32_t k = 0; k < LISTS; ++k) {
        // A list whose least latency lies above the gate has nothing to give, however long it is (one of a sorted array; nothing
        // legal and a gate that is no number do the same)
        if (first + k >= a.lat_parts_n || !(key_to_float(own[k]) <= tau)) continue;
        if (count[k] > SCAN_LIST || !(tau <= gate_above(own[k], a.slack_factor))) return false;
        if (mine == k) from = count[k];
    }
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) c[j] = NONE;
    if (threadIdx.x % SCAN_LIST < from && __uint_as_float((uint32_t)(entry >> 32)) <= tau) {
        const float e = a.energy[(uint64_t)s * a.seg_len + (uint32_t)entry];
        if (e == e) {
            c[0] = ((uint64_t)score_order_key(e) << a.idx_bits) | (uint32_t)entry;
            sh.pool[atomicAdd(&sh.cursor, 1u)] = c[0];
        }
    }
    __syncthreads();
    *kept = sh.cursor;
    *bounded = false;
    return true;
}

// Selection among the gathered composites, then either the block's k slots of list_out (unused slots NONE) or,
// last level, the result.
template <int T>
__device__ __forceinline__ void select_and_emit(const SelectArgs &a, uint32_t s, uint64_t (&c)[ITEMS], uint32_t kept,
                                                bool bounded, bool last_level, bool bound_energies, Shared<T> &sh,
                                                uint64_t *sort_buf)
{
    bool ranked;
    uint64_t thr;
    uint32_t n_selected = select_kept<T>(c, kept, bounded, a.k, 32 + a.idx_bits, sh, &ranked, &thr);
    const uint32_t k_out = a.k_energy ? a.k_energy : a.k;
    if (last_level && a.k_energy) {
        // RANK: these are the segment's fastest.  Their energies, fetched by index, take the latencies' place, and the
        // same selection runs once more, on what the block holds: no second pass over the score arrays.  More than are
        // sorted directly are bounded first where it pays: the 1100 or 4096 fastest of 16384 and their 64 of least energy, 24.4
        // us without the bound, 20.4 with it.
        if (ranked) {
#pragma unroll
            for (int j = 0; j < ITEMS; ++j) {
                const uint32_t i = (uint32_t)j * T + threadIdx.x;
                c[j] = i < n_selected ? sh.pool[i] : NONE; // (at most SMALL)
            }
        }
#pragma unroll
        for (int j = 0; j < ITEMS; ++j) {
            const uint64_t idx = c[j] & ((1ull << a.idx_bits) - 1);
            uint64_t next = NONE;
            if (c[j] != NONE && (ranked || c[j] <= thr)) {
                const float e = a.energy[(uint64_t)s * a.seg_len + idx];
                if (e == e) next = ((uint64_t)score_order_key(e) << a.idx_bits) | idx;
            }
            c[j] = next;
        }
        __syncthreads(); // everything of the first selection has been read
        if (threadIdx.x == 0) sh.cursor = 0;
        bounded = false;
        if (bound_energies && n_selected > SMALL && k_out <= BOUNDED / 4) {
            uint64_t least = NONE;
#pragma unroll
            for (int j = 0; j < ITEMS; ++j) least = c[j] < least ? c[j] : least;
            kept = bound_candidates<T>(c, least, k_out, sh, &bounded);
        } else {
            kept = keep_all<T>(c, sh);
        }
        n_selected = select_kept<T>(c, kept, bounded, k_out, 32 + a.idx_bits, sh, &ranked, &thr);
    }
    if (!last_level) {
        uint64_t *out = a.list_out + ((uint64_t)s * gridDim.x + blockIdx.x) * a.k;
        if (ranked) {
            for (uint32_t i = threadIdx.x; i < n_selected; i += T) out[i] = sh.pool[i];
        } else {
            __syncthreads(); // the histogram's space is done with
            if (threadIdx.x == 0) sh.cursor = 0;
            __syncthreads();
#pragma unroll
            for (int j = 0; j < ITEMS; ++j)
                if (c[j] <= thr) out[atomicAdd(&sh.cursor, 1u)] = c[j]; // NONE > thr; exactly n_selected qualify
        }
        for (uint32_t i = n_selected + threadIdx.x; i < a.k; i += T) out[i] = NONE;
        return;
    }
    // last level: the selection in ascending order, then unpack
    const uint64_t idx_mask = (1ull << a.idx_bits) - 1;
    auto emit = [&](uint32_t i, uint64_t v) {
        const bool valid = i < n_selected;
        a.idx_out[(uint64_t)s * k_out + i] = valid ? (uint32_t)(v & idx_mask) : 0xFFFFFFFFu;
        a.energy_out[(uint64_t)s * k_out + i] = valid ? key_to_float((uint32_t)(v >> a.idx_bits)) : __builtin_inff();
    };
    if (threadIdx.x == 0) a.count_out[s] = n_selected;
    if (ranked) {
        for (uint32_t i = threadIdx.x; i < k_out; i += T) emit(i, i < n_selected ? sh.pool[i] : 0);
        return;
    }
    // bitonic sort of the selection (padded to a power of two with NONE)
    uint32_t pow2 = 2;
    while (pow2 < k_out) pow2 <<= 1;
    for (uint32_t i = threadIdx.x; i < pow2; i += T) sort_buf[i] = NONE;
    if (threadIdx.x == 0) sh.cursor = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < ITEMS; ++j)
        if (c[j] <= thr) sort_buf[atomicAdd(&sh.cursor, 1u)] = c[j];
    __syncthreads();
    if (pow2 <= (uint32_t)T) {
        // one element per thread: steps whose partner sits in the same wavefront exchange registers, only the
        // wider ones go through LDS (10 of the 55 steps for 1024 elements)
        const uint32_t i = threadIdx.x;
        uint64_t v = i < pow2 ? sort_buf[i] : NONE;
        for (uint32_t size = 2; size <= pow2; size <<= 1) {
            const bool ascending = (i & size) == 0;
            auto merge = [&](uint32_t stride, uint64_t other) {
                const bool lower = (i & stride) == 0; // this thread keeps the smaller one of an ascending pair
                const uint64_t lo = v < other ? v : other, hi = v < other ? other : v;
                v = (lower == ascending) ? lo : hi;
            };
            for (uint32_t stride = size >> 1; stride >= 64; stride >>= 1) {
                __syncthreads(); // the reads of the step before are done
                if (i < pow2) sort_buf[i] = v;
                __syncthreads();
                merge(stride, i < pow2 ? sort_buf[i ^ stride] : NONE);
            }
#pragma unroll
            for (uint32_t stride = 32; stride > 0; stride >>= 1)
                if (stride < size) merge(stride, lane_exchange(v, stride));
        }
        if (i < k_out) emit(i, v);
        return;
    }
    for (uint32_t size = 2; size <= pow2; size <<= 1)
        for (uint32_t stride = size >> 1; stride > 0; stride >>= 1) {
            for (uint32_t t = threadIdx.x; t < pow2 / 2; t += T) {
                const uint32_t lo = 2 * t - (t & (stride - 1)); // index with the `stride` bit clear
                const uint32_t hi = lo + stride;
                const bool ascending = (lo & size) == 0;
                const uint64_t x = sort_buf[lo], y = sort_buf[hi];
                if ((x > y) == ascending) {
                    sort_buf[lo] = y;
                    sort_buf[hi] = x;
                }
            }
            __syncthreads();
        }
    for (uint32_t i = threadIdx.x; i < k_out; i += T) emit(i, i < n_selected ? sort_buf[i] : 0);
}

// One block = T threads x ITEMS candidates of segment blockIdx.y: a chunk of the score arrays, or the same number
// of composites of the list the level before wrote.  With one block per segment (gridDim.x == 1) this is the
// last level and writes the result; otherwise the block's selection goes to its k slots of list_out and a further
// launch works on the lists.  (Letting the block that finishes a segment last merge the lists inside the same
// launch was tried: on this chip blocks of one launch sit on eight dies with separate L2 caches, so lists and
// tickets have to be written through to memory -- device-scope stores and atomics, or a release fence, which
// writes the whole L2 back -- and that costs far more than the second launch: 73 us and 400 us against 32.  Blocks of one
// die can hand over in its L2, 0.73 us (crew.h); a merge of each die's lists before the last launch has not been tried.)
template <int T, int SRC, int PRED, bool CROWDED = false>
__global__ __launch_bounds__(T, CROWDED ? 8 : 1) void select_kernel(SelectArgs a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds_raw[];
    Shared<T> &sh = *reinterpret_cast<Shared<T> *>(lds_raw);
    uint64_t *sort_buf = reinterpret_cast<uint64_t *>(lds_raw + ((sizeof(Shared<T>) + 15) & ~(size_t)15));
    const uint32_t s = blockIdx.y;
    uint64_t c[ITEMS];
    uint32_t kept;
    bool bounded;
    // the pool's cursor starts at zero (ordered before its use by the barriers of the gather step)
    if (threadIdx.x == 0) sh.cursor = 0;
    if (SRC == SRC_LIST) gather_list<T>(a.list_in + (uint64_t)s * a.list_len, a.list_len, (uint64_t)blockIdx.x * (T * ITEMS), a.k, sh, c, &kept, &bounded);
    else if (SRC == SRC_SCANNED_VEC || SRC == SRC_SCANNED) {
        uint32_t best;
        if (!gather_scanned<T>(a, s, sh, c, &kept, &bounded, &best))
            gather_scores<T, SRC == SRC_SCANNED_VEC ? SRC_SCORES_VEC : SRC_SCORES, PRED>(a, s, sh, c, &kept, &bounded, &best);
    } else gather_scores<T, SRC, PRED>(a, s, sh, c, &kept, &bounded, nullptr);
    // (RANK: a whole segment's candidates lie spread over what the threads hold, and a radix select over them is slow; a short
    // segment or a list of selections is dense, and some wavefronts may hold none of it)
    const bool spread = SRC != SRC_LIST && a.seg_len > 4 * (T - 64);
    select_and_emit<T>(a, s, c, kept, bounded, gridDim.x == 1, spread, sh, sort_buf);
}

// ---------------------------------------------------------------- host side

// Threads per block for the least workspace: 1024 (chunks of 16384) when k is large, so that a level still shrinks its
// input at least fourfold, or when the whole job is too small to fill the chip anyway and fewer levels matter more; 256
// (chunks of 4096) otherwise.
int threads_for(uint64_t seg_len, uint32_t n_seg, uint32_t k)
{
    if (k > 256) return 1024;
    const uint64_t blocks = (uint64_t)n_seg * ((seg_len + 4095) / 4096);
    return blocks < 512 ? 1024 : 256;
}

struct Plan {
    int threads, list_threads; // of a block on the scores, and on lists
    uint64_t blocks0;          // level-0 blocks per segment
    uint64_t list_a, list_b;   // composites per segment in the two list buffers (level 0 writes A)
};

// launches on lists until one block holds what is left of a segment
int list_levels(uint64_t list_len, uint32_t k, uint64_t chunk)
{
    int levels = 1;
    for (uint64_t blocks = (list_len + chunk - 1) / chunk; blocks > 1; blocks = (blocks * k + chunk - 1) / chunk) ++levels;
    return levels;
}

// `roomy`: the workspace is as large as the queries say; else the plan that the least workspace is for.  Smaller blocks wait
// less at their barriers and put more compute units to work, larger ones leave shorter lists; the lines lie where the
// measured times cross (us, blocks of 256 / 512 / 1024 threads on the scores, each with its best block on the lists):
//   k = 16 of 2^16  11 / 13 / 12.5, of 2^21  16 / 13.5 / 14;  k = 64 of 2^20  17 / 14.6 / 14.9, of 2^21  - / 17.2 / 16.8;
//   128 of 2^18  16 / 14.6 / 15.6, of 2^20  - / 17.7 / 16.8;  256 of 2^18  - / 18.6 / 18.8, of 2^20  42 / 30 / 21.5;
//   512 of 2^18  36 / 26.6 / 24.5;  1024 of 2^20  50 / 44 / 48;  64 segments of 2^18: k = 32  32.8 / 32 / -, 128  39 / 36 / 43.
//   One block a segment, of 6400: k = 128  - / 6.8 / 8.1, 512  - / 14.8 / 18.5;  of 4096: 16  6.9 / 6.9 / 6.9, RANK 32
//   7.4 / 7.7 / 9.4, 256  12.3 / 7.2 / 8.1, 512  17.8 / 13.9 / 11.2;  of 8192: 512  - / 15.3 / 11.5.
Plan plan_for(uint64_t seg_len, uint32_t n_seg, uint32_t k, bool roomy)
{
    Plan p;
    p.threads = p.list_threads = threads_for(seg_len, n_seg, k);
    auto chunk = [](int threads) { return (uint64_t)threads * ITEMS; };
    auto blocks = [&](int threads) { return (seg_len + chunk(threads) - 1) / chunk(threads); };
    if (roomy && seg_len <= chunk(1024)) {
        p.threads = seg_len <= chunk(256) && k <= 64 ? 256 : seg_len <= chunk(512) && k <= 256 ? 512 : 1024;
    } else if (roomy) {
        p.threads = k <= 48 ? 256 : k <= 256 ? 512 : 1024;
        if (p.threads == 256 && (blocks(256) * k > 4096 || n_seg * blocks(256) >= 2048)) p.threads = 512;
        if (p.threads == 512 && blocks(512) * k > 8192) p.threads = 1024;
        if (k > BOUNDED && k <= 1024 && list_levels(blocks(512) * k, k, chunk(1024)) == list_levels(blocks(1024) * k, k, chunk(1024)))
            p.threads = 512;
        p.list_threads = 256;
        while (p.list_threads < 1024 && (blocks(p.threads) * k > chunk(p.list_threads) || 2 * k > (uint32_t)p.list_threads))
            p.list_threads *= 2;
    }
    p.blocks0 = blocks(p.threads);
    p.list_a = p.blocks0 > 1 ? p.blocks0 * k : 0;
    const uint64_t blocks1 = (p.list_a + chunk(p.list_threads) - 1) / chunk(p.list_threads);
    p.list_b = blocks1 > 1 ? blocks1 * k : 0;
    return p;
}

struct WsLayout {
    uint64_t lat_parts, list_a, list_b, scan_lists, listed, total;
};

// whether, and in how many chunks, scan_kernel takes a segment (every block of the next launch reads the minima of all of
// its segment's chunks, hence the limit)
uint64_t scan_parts(uint64_t seg_len, uint64_t blocks0)
{
    const uint64_t parts = (seg_len + SCAN_CHUNK - 1) / SCAN_CHUNK;
    return blocks0 > 1 && parts <= SCAN_PARTS ? parts : 0;
}

// m_latency: the latency gate of a RANK-mode call when it does not admit the whole segment, else 0.  (The larger of the
// two plans: a workspace made for a gate serves a call without one, too.)
WsLayout ws_layout(uint64_t seg_len, uint32_t n_seg, uint32_t k, uint32_t m_latency, bool roomy)
{
    Plan p = plan_for(seg_len, n_seg, k, roomy);
    const uint64_t parts = roomy ? n_seg * scan_parts(seg_len, p.blocks0) : 0;
    if (m_latency && m_latency < seg_len) {
        const Plan q = plan_for(seg_len, n_seg, m_latency, roomy);
        p.list_a = p.list_a > q.list_a ? p.list_a : q.list_a;
        p.list_b = p.list_b > q.list_b ? p.list_b : q.list_b;
    }
    WsLayout w;
    w.lat_parts = 0;
    w.list_a = w.lat_parts + (uint64_t)n_seg * LATMIN_PARTS * sizeof(uint32_t);
    w.list_b = w.list_a + (uint64_t)n_seg * p.list_a * sizeof(uint64_t);
    w.scan_lists = w.list_b + (uint64_t)n_seg * p.list_b * sizeof(uint64_t);
    w.listed = w.scan_lists + parts * SCAN_LIST * sizeof(uint64_t); // (with the minima: two words per chunk)
    w.total = w.listed + 2 * parts * sizeof(uint32_t);
    return w;
}

// what the queries say
uint64_t workspace_for(uint64_t seg_len, uint32_t n_seg, uint32_t k, uint32_t m_latency)
{
    const uint64_t least = ws_layout(seg_len, n_seg, k, m_latency, false).total, more = ws_layout(seg_len, n_seg, k, m_latency, true).total;
    return least > more ? least : more;
}

bool sizes_ok(uint64_t n, uint32_t n_seg, uint32_t k)
{
    return n && n_seg && k && n % n_seg == 0 && k <= n / n_seg && n / n_seg <= 0xFFFFFFFEull && k <= ECK_MAX_K &&
           n_seg <= 65535;
}

template <int T, int SRC, int PRED, bool CROWDED = false>
void launch_select(const SelectArgs &a, uint32_t blocks, uint32_t n_seg, hipStream_t st)
{
    size_t lds = (sizeof(Shared<T>) + 15) & ~(size_t)15;
    if (blocks == 1) {
        uint32_t pow2 = 2;
        while (pow2 < (a.k_energy ? a.k_energy : a.k)) pow2 <<= 1;
        lds += (size_t)pow2 * sizeof(uint64_t);
    }
    hipLaunchKernelGGL((select_kernel<T, SRC, PRED, CROWDED>), dim3(blocks, n_seg), dim3(T), lds, st, a);
}

template <int T, int PRED>
void launch_level0(const SelectArgs &a, uint32_t blocks, uint32_t n_seg, bool vec, hipStream_t st)
{
    if constexpr (PRED == PRED_THRESHOLD) {
        if (a.listed) {
            // Blocks of 1024 threads: two to a compute unit, for a few spilled registers, where a launch has more blocks than
            // units; what a block waits for before it knows whether its lists tell is then hidden (64 segments of 2^18,
            // everything admitted: k = 512 95.8 -> 82 us, 1024 114 -> 101; one segment of 2^18, 16 blocks, 27.7 and 28.8)
            if (T == 1024 && vec && (uint64_t)blocks * n_seg > 256) launch_select<1024, SRC_SCANNED_VEC, PRED, true>(a, blocks, n_seg, st);
            else if (vec) launch_select<T, SRC_SCANNED_VEC, PRED>(a, blocks, n_seg, st);
            else launch_select<T, SRC_SCANNED, PRED>(a, blocks, n_seg, st);
            return;
        }
    }
    if (vec) launch_select<T, SRC_SCORES_VEC, PRED>(a, blocks, n_seg, st);
    else launch_select<T, SRC_SCORES, PRED>(a, blocks, n_seg, st);
}

// All levels of one selection of a.k per segment: level 0 on the score arrays, further levels on the lists.
// The last level writes idx/energy/count.
template <int PRED>
int32_t run_tournament(SelectArgs a, uint32_t n_seg, bool vec, bool roomy, uint64_t *list_a, uint64_t *list_b, hipStream_t st)
{
    const Plan p = plan_for(a.seg_len, n_seg, a.k, roomy);
    const uint64_t chunk = (uint64_t)p.list_threads * ITEMS;
    uint64_t blocks = p.blocks0;
    if (blocks > 0x7FFFFFFFull) return ECK_EUNSUPPORTED;
    a.list_out = list_a;
    if (p.threads == 256) launch_level0<256, PRED>(a, (uint32_t)blocks, n_seg, vec, st);
    else if (p.threads == 512) launch_level0<512, PRED>(a, (uint32_t)blocks, n_seg, vec, st);
    else launch_level0<1024, PRED>(a, (uint32_t)blocks, n_seg, vec, st);
    uint64_t *in = list_a, *out = list_b;
    while (blocks > 1) {
        a.list_in = in;
        a.list_len = blocks * a.k;
        a.list_out = out;
        blocks = (a.list_len + chunk - 1) / chunk;
        if (p.list_threads == 256) launch_select<256, SRC_LIST, PRED_PLAIN>(a, (uint32_t)blocks, n_seg, st);
        else if (p.list_threads == 512) launch_select<512, SRC_LIST, PRED_PLAIN>(a, (uint32_t)blocks, n_seg, st);
        else launch_select<1024, SRC_LIST, PRED_PLAIN>(a, (uint32_t)blocks, n_seg, st);
        uint64_t *t = in;
        in = out;
        out = t;
    }
    ECK_HIP_TRY(hipGetLastError());
    return ECK_OK;
}

} // namespace

extern "C" uint64_t topk_select_workspace_bytes(uint64_t n, uint32_t n_segments, uint32_t k)
{
    if (!sizes_ok(n, n_segments, k)) return 0;
    return workspace_for(n / n_segments, n_segments, k, 0);
}

extern "C" uint64_t topk_select_rank_workspace_bytes(uint64_t n, uint32_t n_segments, uint32_t k, uint32_t m_latency)
{
    if (!sizes_ok(n, n_segments, k) || m_latency == 0) return 0;
    const uint64_t seg_len = n / n_segments;
    if (m_latency < seg_len && m_latency > ECK_MAX_K) return 0;
    return workspace_for(seg_len, n_segments, k, m_latency < seg_len ? m_latency : 0);
}

namespace {

// argument checks shared by the entry points; *need = bytes of workspace the call takes
int32_t check_arguments(const float *energy, const float *latency, uint64_t n, uint32_t n_segments, uint32_t k, int32_t mode,
                        float alpha, uint32_t m_latency, const uint32_t *idx_out, const float *energy_out,
                        const uint32_t *count_out, bool *stage_a, uint64_t *need)
{
    if (!energy || !idx_out || !energy_out || !count_out || n == 0 || k == 0 || n_segments == 0) return ECK_EINVAL;
    if (mode != ECK_SELECT_THRESHOLD && mode != ECK_SELECT_RANK) return ECK_EINVAL;
    if (latency && mode == ECK_SELECT_THRESHOLD && !(alpha >= 1.0f)) return ECK_EINVAL;
    if (latency && mode == ECK_SELECT_RANK && m_latency == 0) return ECK_EINVAL;
    if (n % n_segments || k > n / n_segments || n / n_segments > 0xFFFFFFFEull || n_segments > 65535) return ECK_ESHAPE;
    if (k > ECK_MAX_K) return ECK_EUNSUPPORTED;
    const uint64_t seg_len = n / n_segments;
    // a latency gate that admits the whole segment needs no first stage
    *stage_a = latency && mode == ECK_SELECT_RANK && m_latency < seg_len;
    if (*stage_a && m_latency > ECK_MAX_K) return ECK_EUNSUPPORTED;
    *need = ws_layout(seg_len, n_segments, k, *stage_a ? m_latency : 0, false).total;
    return ECK_OK;
}

} // namespace

int32_t eck::topk_select_impl(const float *energy, const float *latency, const uint8_t *legal, uint64_t n,
                              uint32_t n_segments, uint32_t k, int32_t mode, float alpha, uint32_t m_latency,
                              uint32_t *idx_out, float *energy_out, uint32_t *count_out, void *ws, uint64_t ws_bytes,
                              void *stream, const uint32_t *known_min)
{
    bool stage_a;
    uint64_t need;
    const int32_t bad = check_arguments(energy, latency, n, n_segments, k, mode, alpha, m_latency, idx_out, energy_out,
                                        count_out, &stage_a, &need);
    if (bad != ECK_OK) return bad;
    if (!ws || ws_bytes < need) return ECK_EWORKSPACE;
    if ((uintptr_t)ws & 15) return ECK_EALIGN;
    const uint64_t seg_len = n / n_segments;
    WsLayout w = ws_layout(seg_len, n_segments, k, stage_a ? m_latency : 0, true);
    const bool roomy = ws_bytes >= w.total;
    if (!roomy) w = ws_layout(seg_len, n_segments, k, stage_a ? m_latency : 0, false);
    const uint64_t blocks0 = plan_for(seg_len, n_segments, k, roomy).blocks0;

    SelectArgs a = {};
    a.energy = energy;
    a.latency = latency;
    a.legal = legal;
    a.seg_len = seg_len;
    a.idx_bits = 1;
    while (a.idx_bits < 32 && (1ull << a.idx_bits) < a.seg_len) ++a.idx_bits;
    a.slack_factor = alpha - 1.0f;
    a.alpha_inf = __builtin_isinf(alpha) ? 1 : 0;
    a.k = k;
    a.idx_out = idx_out;
    a.energy_out = energy_out;
    a.count_out = count_out;
    uint32_t *lat_parts = reinterpret_cast<uint32_t *>((char *)ws + w.lat_parts);
    uint64_t *list_a = reinterpret_cast<uint64_t *>((char *)ws + w.list_a);
    uint64_t *list_b = reinterpret_cast<uint64_t *>((char *)ws + w.list_b);

    hipStream_t st = as_stream(stream);
    // four candidates per load when every group of four is aligned in all three arrays
    const bool vec = seg_len % 4 == 0 && ((uintptr_t)energy & 15) == 0 && (!latency || ((uintptr_t)latency & 15) == 0) &&
                     (!legal || ((uintptr_t)legal & 3) == 0);
    if (!latency) return run_tournament<PRED_PLAIN>(a, n_segments, vec, roomy, list_a, list_b, st);
    if (mode == ECK_SELECT_THRESHOLD) {
        if (!a.alpha_inf && known_min) {
            // L_min came with the call (one order key per segment)
            a.lat_parts = known_min;
            a.lat_parts_n = 1;
        } else if (const uint64_t chunks = roomy ? scan_parts(seg_len, blocks0) : 0; !a.alpha_inf && chunks) {
            // one pass over the latencies finds the least one and what its gate may admit
            uint32_t *listed = reinterpret_cast<uint32_t *>((char *)ws + w.listed), *least = listed + n_segments * chunks;
            uint64_t *lists = reinterpret_cast<uint64_t *>((char *)ws + w.scan_lists);
            const dim3 grid((uint32_t)chunks, n_segments);
            if (vec) hipLaunchKernelGGL(scan_kernel<true>, grid, dim3(256), 0, st, latency, legal, seg_len, a.slack_factor, least, listed, lists);
            else hipLaunchKernelGGL(scan_kernel<false>, grid, dim3(256), 0, st, latency, legal, seg_len, a.slack_factor, least, listed, lists);
            a.lat_parts = least;
            a.lat_parts_n = (uint32_t)chunks;
            a.listed = listed;
            a.scan_lists = lists;
        } else if (!a.alpha_inf && blocks0 > 1) {
            // L_min first: one pass over the latencies, a slice of the segment per block (a segment that one block
            // holds needs none: that block finds it, 4 us less)
            uint64_t parts = (seg_len + 4095) / 4096;
            if (parts > LATMIN_PARTS) parts = LATMIN_PARTS;
            uint64_t slice = (seg_len + parts - 1) / parts;
            slice = (slice + 1023) & ~1023ull; // whole groups of four per thread
            parts = (seg_len + slice - 1) / slice;
            if (vec) hipLaunchKernelGGL(latmin_kernel<true>, dim3((uint32_t)parts, n_segments), dim3(256), 0, st, latency, legal,
                                        seg_len, slice, lat_parts);
            else hipLaunchKernelGGL(latmin_kernel<false>, dim3((uint32_t)parts, n_segments), dim3(256), 0, st, latency, legal,
                                    seg_len, slice, lat_parts);
            a.lat_parts = lat_parts;
            a.lat_parts_n = (uint32_t)parts;
        }
        return run_tournament<PRED_THRESHOLD>(a, n_segments, vec, roomy, list_a, list_b, st);
    }
    if (!stage_a) {
        // every legal candidate with a latency that is a number passes the gate
        SelectArgs b = a;
        b.alpha_inf = 1;
        return run_tournament<PRED_THRESHOLD>(b, n_segments, vec, roomy, list_a, list_b, st);
    }
    // the m_latency fastest by latency, of these k by energy in the last level's block: two launches where a second
    // tournament over the gated scores took four (45 us on 2^20, 128 fastest, k = 64; 31 with one, and 19.4 with blocks and lists
    // as plan_for cuts them, sorted pools and tight bounds)
    a.k = m_latency;
    a.k_energy = k;
    return run_tournament<PRED_RANK>(a, n_segments, vec, roomy, list_a, list_b, st);
}

extern "C" int32_t topk_select(const float *energy, const float *latency, const uint8_t *legal, uint64_t n,
                               uint32_t n_segments, uint32_t k, int32_t mode, float alpha, uint32_t m_latency,
                               uint32_t *idx_out, float *energy_out, uint32_t *count_out, void *ws, uint64_t ws_bytes,
                               void *stream)
{
    return topk_select_impl(energy, latency, legal, n, n_segments, k, mode, alpha, m_latency, idx_out, energy_out,
                            count_out, ws, ws_bytes, stream, nullptr);
}

extern "C" int32_t topk_select_known_min(const float *energy, const float *latency, const uint8_t *legal, uint64_t n,
                                         uint32_t n_segments, uint32_t k, float alpha, const uint32_t *latency_min_key,
                                         uint32_t *idx_out, float *energy_out, uint32_t *count_out, void *ws,
                                         uint64_t ws_bytes, void *stream)
{
    if (!latency || !latency_min_key) return ECK_EINVAL;
    return topk_select_impl(energy, latency, legal, n, n_segments, k, ECK_SELECT_THRESHOLD, alpha, 0, idx_out, energy_out,
                            count_out, ws, ws_bytes, stream, latency_min_key);
}

// ---------------------------------------------------------------- the entry point that allocates nothing

namespace {
constexpr int MAX_DEVICES = 64;
// the workspace of topk_select_static: one copy per GPU the library runs on, held until the process ends
__device__ __align__(256) unsigned char scratch[ECK_TOPK_STATIC_BYTES];
void *scratch_address[MAX_DEVICES]; // per device: where that device's copy of `scratch` lives
std::mutex scratch_mutex;
} // namespace

extern "C" int32_t topk_select_static(const float *energy, const float *latency, const uint8_t *legal, uint64_t n,
                                      uint32_t n_segments, uint32_t k, int32_t mode, float alpha, uint32_t m_latency,
                                      uint32_t *idx_out, float *energy_out, uint32_t *count_out, void *stream)
{
    bool stage_a;
    uint64_t need;
    const int32_t bad = check_arguments(energy, latency, n, n_segments, k, mode, alpha, m_latency, idx_out, energy_out,
                                        count_out, &stage_a, &need);
    if (bad != ECK_OK) return bad;
    if (need > ECK_TOPK_STATIC_BYTES) return ECK_EWORKSPACE;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        return ECK_EDEVICE;
    }
    if (dev < 0 || dev >= MAX_DEVICES) return ECK_EUNSUPPORTED;
    void *ws;
    {
        // the array's name is a host-side stand-in; its address on the current device is looked up once per device
        std::lock_guard<std::mutex> guard(scratch_mutex);
        if (!scratch_address[dev]) {
            void *found = nullptr;
            if (hipGetSymbolAddress(&found, HIP_SYMBOL(scratch)) != hipSuccess || !found) {
                (void)hipGetLastError();
                return ECK_EDEVICE;
            }
            scratch_address[dev] = found;
        }
        ws = scratch_address[dev];
    }
    // nothing in the workspace has to start at zero: every word a kernel reads was written by an earlier kernel of
    // the same call
    return topk_select_impl(energy, latency, legal, n, n_segments, k, mode, alpha, m_latency, idx_out, energy_out,
                            count_out, ws, ECK_TOPK_STATIC_BYTES, stream, nullptr);
}
