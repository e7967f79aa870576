// sort.hip -- ascending bitonic sort of 64-bit keys in place, of one array or
// of many side by side (SortSpans: regions whose lengths are powers of two,
// pad with UINT64_MAX).  Callers make keys unique (payload index in the low
// bits), so the order is fully determined.  Strides below 2048 run inside LDS;
// larger strides run two per launch where they can (four keys per thread).
// Two arrays of the same spans can be sorted by the same launches (grid.y
// selects the array), which halves the launches of the weight pass.
//
// Bound by latency: a step's barrier or launch costs more than its keys.  A
// thread's pair lies within its wave's 128 keys for strides up to 64, and
// those steps (56 of a tile's 66, 7 of a merge's 11) only order the wave's own
// LDS accesses: a tile launch over 131072 keys 25 -> 14 us, over 2 x 1.2 million
// 75 -> 59 (with a barrier after every step, before).
#include "kernels.h"

namespace abcsmc {

namespace {

constexpr int kSortThreads = 1024;
constexpr int kSortTile = 2 * kSortThreads;  // keys per LDS tile
constexpr int kTileBits = 11;
static_assert(kSortTile == 1 << kTileBits, "");

__device__ __forceinline__ void cmpx(unsigned long long& a, unsigned long long& b, bool up)
{
    if ((a > b) == up) {
        const unsigned long long t = a;
        a = b;
        b = t;
    }
}

// After a step of stride j, before one of stride next.
__device__ __forceinline__ void step_done(int j, int next)
{
    if (j > kWave || next > kWave) {
        __syncthreads();
    } else {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
}

// Every bitonic stage up to the tile size (k = 2 .. 2048), directions taken
// from the global index so tiles combine into the global network.  The last
// stage of a region (k = its length) ascends wherever the region lies.
__global__ __launch_bounds__(kSortThreads) void bitonic_tile_kernel(unsigned long long* keys0, unsigned long long* keys1,
                                                                   SortSpans sp)
{
    __shared__ unsigned long long s[kSortTile];
    unsigned long long* keys = blockIdx.y ? keys1 : keys0;
    const size_t base = (size_t)blockIdx.x * kSortTile;
    const int t = threadIdx.x;
    s[t] = keys[base + t];
    s[t + kSortThreads] = keys[base + t + kSortThreads];
    __syncthreads();
#pragma unroll
    for (int b = 1; b <= kTileBits; ++b) {
        const int k = 1 << b;
        for (int j = k >> 1; j > 0; j >>= 1) {
            const int i = ((t & ~(j - 1)) << 1) | (t & (j - 1));
            const size_t g = base + (size_t)i;
            if (g < sp.n[b]) cmpx(s[i], s[i + j], (g & (size_t)k) == 0 || g >= sp.n[b + 1]);
            step_done(j, j > 1 ? j >> 1 : k);
        }
    }
    __syncthreads();
    keys[base + t] = s[t];
    keys[base + t + kSortThreads] = s[t + kSortThreads];
}

// Strides j < 2048 of stage k (k > 2048) inside LDS; past: keys of regions
// longer than k.
__global__ __launch_bounds__(kSortThreads) void bitonic_merge_tile_kernel(unsigned long long* keys0,
                                                                         unsigned long long* keys1, size_t k, size_t past)
{
    __shared__ unsigned long long s[kSortTile];
    unsigned long long* keys = blockIdx.y ? keys1 : keys0;
    const size_t base = (size_t)blockIdx.x * kSortTile;
    const int t = threadIdx.x;
    s[t] = keys[base + t];
    s[t + kSortThreads] = keys[base + t + kSortThreads];
    __syncthreads();
    const bool up = (base & k) == 0 || base >= past;  // the whole tile lies in one k-block
#pragma unroll
    for (int j = kSortTile >> 1; j > 0; j >>= 1) {
        const int i = ((t & ~(j - 1)) << 1) | (t & (j - 1));
        cmpx(s[i], s[i + j], up);
        step_done(j, j >> 1);
    }
    __syncthreads();
    keys[base + t] = s[t];
    keys[base + t + kSortThreads] = s[t + kSortThreads];
}

// One global compare-exchange step (stage k, stride j >= 2048).
__global__ __launch_bounds__(kBlock) void bitonic_step_kernel(unsigned long long* keys0, unsigned long long* keys1,
                                                              size_t n, size_t k, size_t j, size_t past)
{
    unsigned long long* keys = blockIdx.y ? keys1 : keys0;
    const size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (t >= n / 2) return;
    const size_t i = ((t & ~(j - 1)) << 1) | (t & (j - 1));
    unsigned long long a = keys[i], b = keys[i + j];
    cmpx(a, b, (i & k) == 0 || i >= past);
    keys[i] = a;
    keys[i + j] = b;
}

// Two consecutive global steps of stage k, strides j and h = j/2 (h >= 2048):
// thread t owns the keys i, i + h, i + j, i + j + h with i = (t / h) 2j + t % h,
// all in one 2j-block and so in one k-block (2j <= k): the stride-j pairs
// (i, i + j), (i + h, i + j + h), then the stride-h pairs (i, i + h),
// (i + j, i + j + h).  Every key belongs to exactly one thread.
__global__ __launch_bounds__(kBlock) void bitonic_step2_kernel(unsigned long long* keys0, unsigned long long* keys1,
                                                               size_t n, size_t k, size_t j, size_t past)
{
    unsigned long long* keys = blockIdx.y ? keys1 : keys0;
    const size_t t = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (t >= n / 4) return;
    const size_t h = j >> 1;
    const size_t i = ((t & ~(h - 1)) << 2) | (t & (h - 1));
    unsigned long long a = keys[i], b = keys[i + h], c = keys[i + j], d = keys[i + j + h];
    const bool up = (i & k) == 0 || i >= past;
    cmpx(a, c, up);
    cmpx(b, d, up);
    cmpx(a, b, up);
    cmpx(c, d, up);
    keys[i] = a;
    keys[i + h] = b;
    keys[i + j] = c;
    keys[i + j + h] = d;
}

}  // namespace

size_t sort_padded_size(size_t n)
{
    size_t p = kSortTile;
    while (p < n) p <<= 1;
    return p;
}

size_t sort_span_slots(size_t n) { return (n + kSortTile - 1) / kSortTile * kSortTile; }

void launch_sort_spans(unsigned long long* keys0, unsigned long long* keys1, const SortSpans& sp, hipStream_t s)
{
    const unsigned arrays = keys1 ? 2u : 1u;
    const dim3 bt(kSortThreads), bs(kBlock);
    hipLaunchKernelGGL(bitonic_tile_kernel, dim3((unsigned)(sort_span_slots(sp.n[0]) / kSortTile), arrays), bt, 0, s, keys0,
                       keys1, sp);
    for (int b = kTileBits + 1; b < kSortLevels - 1 && sp.n[b]; ++b) {
        const size_t n = sp.n[b], k = (size_t)1 << b, past = sp.n[b + 1];
        const dim3 g1((unsigned)((n / 2 + kBlock - 1) / kBlock), arrays);
        const dim3 g2((unsigned)((n / 4 + kBlock - 1) / kBlock), arrays);
        size_t j = k >> 1;
        for (; j >= 2 * (size_t)kSortTile; j >>= 2)
            hipLaunchKernelGGL(bitonic_step2_kernel, g2, bs, 0, s, keys0, keys1, n, k, j, past);
        if (j >= (size_t)kSortTile) hipLaunchKernelGGL(bitonic_step_kernel, g1, bs, 0, s, keys0, keys1, n, k, j, past);
        hipLaunchKernelGGL(bitonic_merge_tile_kernel, dim3((unsigned)(n / kSortTile), arrays), bt, 0, s, keys0, keys1, k,
                           past);
    }
}

void launch_sort_u64_pair(unsigned long long* keys0, unsigned long long* keys1, size_t n_pow2, hipStream_t s)
{
    SortSpans sp{};
    for (int b = 0; b < kSortLevels && ((size_t)1 << b) <= n_pow2; ++b) sp.n[b] = n_pow2;
    launch_sort_spans(keys0, keys1, sp, s);
}

}  // namespace abcsmc
