// What the refits of all model forms share (HIP, gfx950): the measured energies made labels, and sums over a block.
#pragma once
#include "crew.h"
#include "lanes.h"

namespace eck {

// Sum over the 1024 threads of a block in double, in a fixed order: halves added to halves, by LDS down to a wavefront, then by
// exchanges.  The sum is thread 0's; scratch: 512 doubles, free again after a barrier.
__device__ __forceinline__ double block_sum(double v, double *scratch)
{
    const int tid = threadIdx.x;
    for (int off = 512; off >= 64; off >>= 1) {
        if (tid >= off && tid < 2 * off) scratch[tid - off] = v;
        __syncthreads();
        if (tid < off) v += scratch[tid];
        __syncthreads();
    }
    if (tid < 64) {
#pragma unroll
        for (uint32_t off = 32; off > 0; off >>= 1) v += lane_exchange(v, off);
    }
    return v;
}

// One block of 1024 threads: validates the measured energies and normalises them by their maximum (fp32 division).
__device__ __forceinline__ void make_labels(const float *__restrict__ e, uint64_t n, float *__restrict__ y, RefitScalars *sc)
{
    __shared__ float wave_max[16];
    __shared__ uint32_t wave_bad[16];
    constexpr int KEEP = 4; // energies a thread still holds for the second pass
    float mx = 0.0f, kept[KEEP];
    uint32_t bad = 0;
    auto look = [&](float v) {
        if (!(v > 0.0f) || v == __builtin_inff()) bad = 1;
        mx = fmaxf(mx, v);
    };
#pragma unroll
    for (int k = 0; k < KEEP; ++k) {
        const uint64_t i = threadIdx.x + 1024ull * k;
        kept[k] = e[i < n ? i : n - 1];
    }
#pragma unroll
    for (int k = 0; k < KEEP; ++k) look(kept[k]);
    for (uint64_t i = threadIdx.x + 1024ull * KEEP; i < n; i += 1024) look(e[i]);
#pragma unroll
    for (uint32_t off = 32; off > 0; off >>= 1) {
        mx = fmaxf(mx, __uint_as_float(lane_exchange(__float_as_uint(mx), off)));
        bad |= lane_exchange(bad, off);
    }
    if ((threadIdx.x & 63) == 0) {
        wave_max[threadIdx.x >> 6] = mx;
        wave_bad[threadIdx.x >> 6] = bad;
    }
    __syncthreads();
    mx = wave_max[0];
    bad = wave_bad[0];
#pragma unroll
    for (int w = 1; w < 16; ++w) {
        mx = fmaxf(mx, wave_max[w]);
        bad |= wave_bad[w];
    }
#pragma unroll
    for (int k = 0; k < KEEP; ++k) {
        const uint64_t i = threadIdx.x + 1024ull * k;
        if (i < n) y[i] = kept[k] / mx;
    }
    for (uint64_t i = threadIdx.x + 1024ull * KEEP; i < n; i += 1024) y[i] = e[i] / mx;
    if (threadIdx.x == 0) {
        sc->emax = mx;
        sc->bad = bad;
        sc->snr = sc->loss = __builtin_nanf("");
    }
}

// The sum of the Eq.-(1) terms of a minibatch in double, in a fixed order: PARTS sums, of every PARTS-th 64 rows each, along a wavefront,
// then the parts in order.  Part by part, by a wavefront each ...
template <int PARTS>
__device__ __forceinline__ double loss_part(const float *terms, int rows, int part, int lane)
{
    double s = 0.0;
#pragma unroll 8
    for (int r = 64 * part + lane; r < rows; r += 64 * PARTS) s += (double)terms[r];
#pragma unroll
    for (uint32_t off = 32; off > 0; off >>= 1) s += lane_exchange(s, off);
    return s;
}
// ... or all by one wavefront of a crew, whose rows are few
template <int PARTS>
__device__ __forceinline__ double loss_sum_fresh(const float *terms, int rows, int lane)
{
    double s[PARTS] = {};
    for (int r = lane; r < rows; r += 64 * PARTS) {
#pragma unroll
        for (int p = 0; p < PARTS; ++p) {
            const float term = fresh_float<true>(terms, 4u * min(r + 64 * p, rows - 1), 0);
            s[p] += r + 64 * p < rows ? (double)term : 0.0; // (no term is below zero)
        }
    }
#pragma unroll
    for (uint32_t off = 32; off > 0; off >>= 1) {
#pragma unroll
        for (int p = 0; p < PARTS; ++p) s[p] += lane_exchange(s[p], off);
    }
#pragma unroll
    for (int p = 1; p < PARTS; ++p) s[0] += s[p];
    return s[0];
}

// One block of 1024 threads: sum y^2 / sum (p - y)^2, thread 0's
__device__ __forceinline__ float signal_to_noise(const float *__restrict__ p, const float *__restrict__ y, uint64_t n)
{
    __shared__ double scratch[512];
    double signal = 0.0, noise = 0.0;
    for (uint64_t i = threadIdx.x; i < n; i += 1024) {
        const double yi = y[i], d = (double)p[i] - yi;
        signal += yi * yi;
        noise += d * d;
    }
    signal = block_sum(signal, scratch);
    noise = block_sum(noise, scratch);
    return (float)(signal / noise);
}

} // namespace eck
