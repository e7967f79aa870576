// blockselect.h -- one workgroup's exact type-7 quantile of n non-negative
// doubles (eq. 8's percentile; numpy "linear" interpolation): the order
// statistic by radix select on the IEEE bit patterns, the next one beside it.
// Used by the single run's and the batched runs' percentile and by the
// predictive bands.
//
// Bound by the passes over the data (L2 to one compute unit) and by barriers.
// A pass finds the highest bit in which the values differ, a second one
// histograms the 11 bits from there (values of one stage share sign, exponent
// and often more, so digits at fixed places would send every value to the same
// few bins and the same LDS words), a third collects the bin that holds the
// rank, which is finished in LDS; only bins of more than kKeep values are
// histogrammed again, at most until their values are equal.  Three passes where
// six fixed digits for two ranks took twelve: 32768 values x 453 rows x 3
// quantiles 1226 -> 427 us.
#pragma once

#include <hip/hip_runtime.h>

#include "kernels.h"

namespace abcsmc {
namespace bsel {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / kWave;
constexpr int kBins = 2048;
constexpr int kKeep = 256;  // values finished in LDS, a thread each

struct Shared {
    unsigned int h[kBins];
    unsigned long long keep[kKeep];
    unsigned long long lo[kWaves], hi[kWaves];
    unsigned int sum[kWaves];
    unsigned int n_keep, bin, below, count;
    unsigned long long xa, xb;
};

__device__ __forceinline__ unsigned long long wave_min64(unsigned long long v)
{
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        const unsigned long long o = __shfl_xor(v, off, kWave);
        v = o < v ? o : v;
    }
    return v;
}
__device__ __forceinline__ unsigned long long wave_max64(unsigned long long v)
{
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) {
        const unsigned long long o = __shfl_xor(v, off, kWave);
        v = o > v ? o : v;
    }
    return v;
}

__device__ __forceinline__ unsigned long long bits_of(double v)
{
    // distances and counts are never negative; a NaN sorts above +inf
    return (unsigned long long)__double_as_longlong(v);
}

// Ranks r0, r1 of the two order statistics that the type-7 quantile alpha of n
// values lies between, and the quantile from them (numpy's arithmetic).
__device__ __forceinline__ void ranks7(int n, double alpha, int& r0, int& r1)
{
    const double v = ((double)n - 1.0) * alpha;
    if (v >= (double)n - 1.0) {
        r0 = r1 = n - 1;
    } else if (v < 0.0) {
        r0 = r1 = 0;
    } else {
        r0 = (int)__builtin_floor(v);
        r1 = r0 + 1;
    }
}

__device__ __forceinline__ double interpolate7(int n, double alpha, unsigned long long xa_bits, unsigned long long xb_bits)
{
    int r0, r1;
    ranks7(n, alpha, r0, r1);
    const double xa = __longlong_as_double((long long)xa_bits), xb = __longlong_as_double((long long)xb_bits);
    if (r0 == r1) return xa;
    const double v = ((double)n - 1.0) * alpha;
    const double g = v - __builtin_floor(v);
    const double diff = xb - xa;
    return g >= 0.5 ? xb - diff * (1.0 - g) : xa + diff * g;
}

// A thread's share of x[k], k < n: every kThreads-th value, read from memory in
// each pass, or read once into registers (n <= K kThreads).
struct FromMemory {
    const double* __restrict__ x;
    int n;
    template <class F>
    __device__ __forceinline__ void each(F f) const
    {
#pragma unroll 8
        for (int k = threadIdx.x; k < n; k += kThreads) f(bits_of(x[k]));
    }
};

template <int K>
struct FromRegisters {
    double v[K];
    int n;
    __device__ __forceinline__ FromRegisters(const double* x, int n) : n(n)
    {
#pragma unroll
        for (int i = 0; i < K; ++i) v[i] = i * kThreads + (int)threadIdx.x < n ? x[i * kThreads + threadIdx.x] : 0.0;
    }
    template <class F>
    __device__ __forceinline__ void each(F f) const
    {
#pragma unroll
        for (int i = 0; i < K; ++i)
            if (i * kThreads + (int)threadIdx.x < n) f(bits_of(v[i]));
    }
};

// Bits of the order statistics rank and rank + 1 (all ones if there is none)
// of n values (1 <= n < 2^31), in S.xa and S.xb; every thread of the kThreads
// calls it.
template <class Values>
__device__ __forceinline__ void order_pair(const Values& values, int n, unsigned int rank, Shared& S)
{
    const int t = threadIdx.x, w = t / kWave, lane = t & (kWave - 1);
    // the range of the values
    unsigned long long lo = ~0ull, hi = 0ull;
    values.each([&](unsigned long long b) {
        lo = b < lo ? b : lo;
        hi = b > hi ? b : hi;
    });
    lo = wave_min64(lo);
    hi = wave_max64(hi);
    if (lane == 0) {
        S.lo[w] = lo;
        S.hi[w] = hi;
    }
    __syncthreads();
    lo = wave_min64(S.lo[lane & (kWaves - 1)]);
    hi = wave_max64(S.hi[lane & (kWaves - 1)]);
    unsigned int count = (unsigned int)n;  // values in [lo, hi], the rank counted from there
    // values in [lo, hi] (a range of one prefix) until they are few or equal
    while (count > (unsigned)kKeep && lo != hi) {
        const int top = 63 - __builtin_clzll(lo ^ hi);
        const int sh = top > 10 ? top - 10 : 0;
        const unsigned long long base = lo >> sh;
        for (int b = t; b < kBins; b += kThreads) S.h[b] = 0u;
        __syncthreads();
        values.each([&](unsigned long long b) {
            if (b >= lo && b <= hi) atomicAdd(&S.h[(unsigned)((b >> sh) - base)], 1u);
        });
        __syncthreads();
        // exclusive prefix of the bins, two a thread
        const unsigned int h0 = S.h[2 * t], h1 = S.h[2 * t + 1];
        unsigned int incl = h0 + h1;
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            const unsigned int o = __shfl_up(incl, off, kWave);
            if (lane >= off) incl += o;
        }
        if (lane == kWave - 1) S.sum[w] = incl;
        __syncthreads();
        unsigned int below = incl - h0 - h1;
        for (int i = 0; i < w; ++i) below += S.sum[i];
        if (rank >= below && rank - below < h0 + h1) {
            const bool second = rank - below >= h0;
            S.bin = 2 * t + (second ? 1 : 0);
            S.below = below + (second ? h0 : 0);
            S.count = second ? h1 : h0;
        }
        __syncthreads();
        rank -= S.below;
        count = S.count;
        const unsigned long long first = (base + S.bin) << sh, last = first + ((1ull << sh) - 1ull);
        lo = first > lo ? first : lo;
        hi = last < hi ? last : hi;
        __syncthreads();
    }
    // the values in [lo, hi] (their number is known to be small, or they are
    // equal) and the smallest value above them
    const bool equal = lo == hi;
    if (t == 0) S.n_keep = 0;
    __syncthreads();
    unsigned long long above = ~0ull;
    values.each([&](unsigned long long b) {
        if (b > hi) above = b < above ? b : above;
        else if (!equal && b >= lo) S.keep[atomicAdd(&S.n_keep, 1u)] = b;
    });
    above = wave_min64(above);
    if (lane == 0) S.lo[w] = above;
    __syncthreads();
    above = wave_min64(S.lo[lane & (kWaves - 1)]);
    if (equal) {
        if (t == 0) {
            S.xa = lo;
            S.xb = rank + 1 < count ? lo : above;
        }
    } else {
        if (t == 0 && rank + 1 >= count) S.xb = above;
        if (t < (int)count) {
            const unsigned long long mine = S.keep[t];
            unsigned int less = 0;
            for (int i = 0; i < (int)count; ++i) {
                const unsigned long long o = S.keep[i];
                less += (o < mine || (o == mine && i < t)) ? 1u : 0u;
            }
            if (less == rank) S.xa = mine;
            if (less == rank + 1) S.xb = mine;
        }
    }
    __syncthreads();
}

// The quantile; every thread gets it.
template <class Values>
__device__ __forceinline__ double quantile7(const Values& values, int n, double alpha, Shared& S)
{
    int r0, r1;
    ranks7(n, alpha, r0, r1);
    order_pair(values, n, (unsigned int)r0, S);
    const double r = interpolate7(n, alpha, S.xa, S.xb);
    __syncthreads();
    return r;
}

}  // namespace bsel
}  // namespace abcsmc
