// smc.hip -- SMC stage machinery around the proposal kernel:
//   resample   prior set, eq. 10 weights and the integer CDF of eq. 11
//   weights    N x M importance-weight row sums, windowed, FP64
//   normalise  W = softmax(log-weights), effective sample size
//   select     exact type-7 percentile of eq. 8
// All reductions combine per-block partials in a fixed order, so every result
// is bitwise reproducible run to run.
#include "blockselect.h"
#include "dmath.h"
#include "kernels.h"
#include "wterm.h"

#include <algorithm>

namespace abcsmc {

namespace {

constexpr int kChunk = 1024;            // elements per block of the resample kernels
constexpr int kPer = kChunk / kBlock;   // elements per thread (contiguous)

__device__ __forceinline__ unsigned long long block_sum_u64(unsigned long long v, unsigned long long* sh)
{
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int off = kBlock / 2; off > 0; off >>= 1) {
        if (t < off) sh[t] += sh[t + off];
        __syncthreads();
    }
    const unsigned long long r = sh[0];
    __syncthreads();
    return r;
}

__device__ __forceinline__ double block_sum_f64(double v, double* sh)
{
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int off = kBlock / 2; off > 0; off >>= 1) {
        if (t < off) sh[t] += sh[t + off];
        __syncthreads();
    }
    const double r = sh[0];
    __syncthreads();
    return r;
}

__device__ __forceinline__ double block_max_f64(double v, double* sh)
{
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int off = kBlock / 2; off > 0; off >>= 1) {
        if (t < off) sh[t] = sh[t] > sh[t + off] ? sh[t] : sh[t + off];
        __syncthreads();
    }
    const double r = sh[0];
    __syncthreads();
    return r;
}

// Exclusive scan of one value per thread (Hillis-Steele in LDS); *total gets the sum.
__device__ __forceinline__ unsigned long long block_excl_scan_u64(unsigned long long v, unsigned long long* sh,
                                                                  unsigned long long* total)
{
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int off = 1; off < kBlock; off <<= 1) {
        const unsigned long long x = t >= off ? sh[t - off] : 0ull;
        __syncthreads();
        sh[t] += x;
        __syncthreads();
    }
    const unsigned long long incl = sh[t];
    *total = sh[kBlock - 1];
    __syncthreads();
    return incl - v;
}

// ---------------------------------------------------------------------------
// Prior set of the stage (eq. 9): particles of the previous stage with
// d < eps (d <= eps when none is strictly below); weight eps - d (eq. 10),
// quantised q_k = floor((w_k / w_max) 2^40) (all survivors q = 1 when
// w_max = 0); cdf = inclusive prefix sum of q, exact in uint64 (eq. 11 draws
// r uniform in [0, cdf[N-1]) and takes the first k with cdf[k] > r).  Also
// packs (u_k, q_k) of every q_k > 0 in index order for the weight kernel.
// Three passes over blocks of 1024 particles: statistics, per-block sums,
// write-out with the block's exclusive offset.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void resample_stats_kernel(ResampleArgs a)
{
    __shared__ unsigned long long shu[kBlock];
    __shared__ double shd[kBlock];
    if (blockIdx.x == 0 && threadIdx.x == 0) a.ctr->ts[kTsBegin] = wall_clock64();
    const int k0 = blockIdx.x * kChunk;
    unsigned long long ns = 0;
    double wmx = 0.0;
    for (int i = 0; i < kPer; ++i) {
        const int k = k0 + i * kBlock + threadIdx.x;
        if (k < a.N) {
            const double d = a.d_prev[k];
            if (d < a.eps) {
                ++ns;
                const double w = a.eps - d;
                wmx = w > wmx ? w : wmx;
            }
        }
    }
    ns = block_sum_u64(ns, shu);
    wmx = block_max_f64(wmx, shd);
    if (threadIdx.x == 0) {
        a.sc.u0[blockIdx.x] = ns;
        a.sc.d0[blockIdx.x] = wmx;
    }
}

// Global prior-set mode from the per-block statistics (same order in every block).
__device__ __forceinline__ void resample_mode(const ResampleArgs& a, bool& strict, double& wmax,
                                              unsigned long long* shu, double* shd)
{
    const int G = gridDim.x;
    unsigned long long ns = 0;
    double wmx = 0.0;
    for (int b = threadIdx.x; b < G; b += kBlock) {
        ns += a.sc.u0[b];
        wmx = a.sc.d0[b] > wmx ? a.sc.d0[b] : wmx;
    }
    ns = block_sum_u64(ns, shu);
    wmx = block_max_f64(wmx, shd);
    strict = ns > 0;
    wmax = strict ? wmx : 0.0;
}

__device__ __forceinline__ unsigned long long quantise(double d, double eps, bool strict, double wmax)
{
    const bool in = strict ? (d < eps) : (d <= eps);
    if (!in) return 0ull;
    return wmax > 0.0 ? (unsigned long long)__builtin_floor(((eps - d) / wmax) * 0x1p40) : 1ull;
}

__global__ __launch_bounds__(kBlock) void resample_count_kernel(ResampleArgs a)
{
    __shared__ unsigned long long shu[kBlock];
    __shared__ double shd[kBlock];
    bool strict;
    double wmax;
    resample_mode(a, strict, wmax, shu, shd);
    const int k0 = blockIdx.x * kChunk + threadIdx.x * kPer;
    unsigned long long sq = 0, sc = 0;
    for (int i = 0; i < kPer; ++i) {
        const int k = k0 + i;
        if (k < a.N) {
            const unsigned long long q = quantise(a.d_prev[k], a.eps, strict, wmax);
            sq += q;
            sc += q > 0;
        }
    }
    sq = block_sum_u64(sq, shu);
    sc = block_sum_u64(sc, shu);
    if (threadIdx.x == 0) {
        a.sc.u1[blockIdx.x] = sq;
        a.sc.u2[blockIdx.x] = sc;
    }
}

__global__ __launch_bounds__(kBlock) void resample_write_kernel(ResampleArgs a)
{
    __shared__ unsigned long long shu[kBlock];
    __shared__ double shd[kBlock];
    bool strict;
    double wmax;
    resample_mode(a, strict, wmax, shu, shd);
    // exclusive offsets of this block (and the survivor total for the last block)
    const int G = gridDim.x;
    unsigned long long oq = 0, oc = 0, tc = 0;
    for (int b = threadIdx.x; b < G; b += kBlock) {
        const unsigned long long q = a.sc.u1[b], c = a.sc.u2[b];
        if (b < (int)blockIdx.x) {
            oq += q;
            oc += c;
        }
        tc += c;
    }
    oq = block_sum_u64(oq, shu);
    oc = block_sum_u64(oc, shu);
    tc = block_sum_u64(tc, shu);
    const int k0 = blockIdx.x * kChunk + threadIdx.x * kPer;
    unsigned long long q[kPer];
    unsigned long long sq = 0, sc = 0;
    for (int i = 0; i < kPer; ++i) {
        const int k = k0 + i;
        q[i] = k < a.N ? quantise(a.d_prev[k], a.eps, strict, wmax) : 0ull;
        sq += q[i];
        sc += q[i] > 0;
    }
    unsigned long long tot;
    unsigned long long run = oq + block_excl_scan_u64(sq, shu, &tot);
    unsigned long long col = oc + block_excl_scan_u64(sc, shu, &tot);
    for (int i = 0; i < kPer; ++i) {
        const int k = k0 + i;
        if (k >= a.N) break;
        run += q[i];
        a.q[k] = q[i];
        a.cdf[k] = run;
        if (q[i] > 0) {
            double* c = a.cols + (size_t)col * 9;
            const double* up = a.u_prev + (size_t)k * kNP;
#pragma unroll
            for (int dd = 0; dd < kNP; ++dd) c[dd] = up[dd];
            c[8] = (double)q[i];
            ++col;
        }
    }
    if (blockIdx.x == (unsigned)(G - 1) && threadIdx.x == 0) {
        a.ctr->survivors = tc;
        a.ctr->fallback = strict ? 0ull : 1ull;
    }
}

// Block sums, maxima and scans of kOneThreads threads: wave by wave in
// registers, then the waves' values in LDS.
constexpr int kOneWaves = kOneThreads / kWave;

template <class T, class Op>
__device__ __forceinline__ T one_reduce(T v, T* sh, Op op)
{
#pragma unroll
    for (int off = kWave / 2; off > 0; off >>= 1) v = op(v, __shfl_xor(v, off, kWave));
    __syncthreads();
    if ((threadIdx.x & (kWave - 1)) == 0) sh[threadIdx.x / kWave] = v;
    __syncthreads();
    v = sh[0];
#pragma unroll
    for (int w = 1; w < kOneWaves; ++w) v = op(v, sh[w]);
    return v;
}

__device__ __forceinline__ unsigned long long one_excl_scan(unsigned long long v, unsigned long long* sh,
                                                            unsigned long long* total)
{
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    unsigned long long incl = v;
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        const unsigned long long o = __shfl_up(incl, off, kWave);
        if (lane >= off) incl += o;
    }
    __syncthreads();
    if (lane == kWave - 1) sh[w] = incl;
    __syncthreads();
    unsigned long long before = 0, all = 0;
#pragma unroll
    for (int i = 0; i < kOneWaves; ++i) {
        if (i < w) before += sh[i];
        all += sh[i];
    }
    *total = all;
    return before + incl - v;
}

// The three passes in one workgroup (N <= kOneResample), which also clears the
// stage's counters.
__global__ __launch_bounds__(kOneThreads) void resample_one_kernel(ResampleArgs a)
{
    __shared__ unsigned long long shu[kOneWaves];
    __shared__ double shd[kOneWaves];
    __shared__ uint16_t place[kOneResample];  // column of a survivor
    constexpr int kMost = kOneResample / kOneThreads;
    constexpr uint16_t kNone = 0xFFFF;
    const int t = threadIdx.x;
    if (t < (int)(sizeof(StageCounters) / 8)) {
        unsigned long long* c = (unsigned long long*)a.ctr;
        c[t] = c + t == &a.ctr->ts[kTsBegin] ? wall_clock64() : 0ull;
    }
    const int per = (a.N + kOneThreads - 1) / kOneThreads, k0 = t * per;
    double d[kMost];
    unsigned long long ns = 0;
    double wmx = 0.0;
#pragma unroll
    for (int i = 0; i < kMost; ++i) {
        const int k = k0 + i;
        d[i] = i < per && k < a.N ? a.d_prev[k] : __builtin_inf();
        if (d[i] < a.eps) {
            ++ns;
            const double w = a.eps - d[i];
            wmx = w > wmx ? w : wmx;
        }
    }
    ns = one_reduce(ns, shu, [](unsigned long long x, unsigned long long y) { return x + y; });
    wmx = one_reduce(wmx, shd, [](double x, double y) { return x > y ? x : y; });
    const bool strict = ns > 0;
    const double wmax = strict ? wmx : 0.0;
    unsigned long long sq = 0, sc = 0, tot, survivors;
#pragma unroll
    for (int i = 0; i < kMost; ++i) {
        if (i < per && k0 + i < a.N) {
            const unsigned long long q = quantise(d[i], a.eps, strict, wmax);
            sq += q;
            sc += q > 0;
        }
    }
    unsigned long long run = one_excl_scan(sq, shu, &tot);
    unsigned long long col = one_excl_scan(sc, shu, &survivors);
#pragma unroll
    for (int i = 0; i < kMost; ++i) {
        const int k = k0 + i;
        if (i < per && k < a.N) {
            const unsigned long long q = quantise(d[i], a.eps, strict, wmax);
            run += q;
            a.q[k] = q;
            a.cdf[k] = run;
            place[k] = q > 0 ? (uint16_t)col : kNone;
            if (q > 0) a.cols[(size_t)col++ * 9 + 8] = (double)q;
        }
    }
    __syncthreads();
#pragma unroll 4
    for (int e = t; e < a.N * kNP; e += kOneThreads) {
        const uint16_t c = place[e / kNP];
        if (c != kNone) a.cols[(size_t)c * 9 + e % kNP] = a.u_prev[e];
    }
    if (t == 0) {
        a.ctr->survivors = survivors;
        a.ctr->fallback = strict ? 0ull : 1ull;
    }
}

// ---------------------------------------------------------------------------
// Importance weights.  Row j (an accepted particle with step sigma_j) gets
//   L_j = sum_k q_k exp(-|u_j - u_k|^2 / (2 sigma_j^2))
// over the previous particles with q_k > 0, and log-weight
//   l_j = 8 log sigma_j - log L_j,
// the log of 1 / (proposal density at u_j given sigma_j) up to a constant
// (prior density 1 on the cube).  One lane per row; the columns are split in
// `chunks` contiguous ranges (grid y) so the launch fills the chip; every lane
// of a wave evaluates the same column, from scalar loads.  Per-chunk partial
// sums are added in a fixed order.
//
// The exponential here is table driven (1024 entries of 2^(i/1024) in LDS and
// a cubic in the remainder).  Its relative error (a few 1e-16) is far inside
// the 1e-12 the weights are held to; the trajectories never use it.
// ---------------------------------------------------------------------------
using wterm::sigma_half_octave;
using wterm::wave_sum_u64;

// ---- windowed evaluation -------------------------------------------------
// Row j only needs the columns within its radius R_j = W_j sigma_j: every
// other column has a term at most q_k e^{-W_j^2/2}, and W_j is chosen from the
// row's own parent term so that all of them together stay below 2^-53 of the
// row sum (at most 37.7, where every omitted exponential is below e^-710).
// Per stage: statistics of the columns choose the sort code (wterm.h), columns
// are sorted by it, rows by (half-octave of sigma descending, code), both are
// gathered into sorted arrays with what the pair test needs, and every wave
// (64 consecutive sorted rows) evaluates the columns one of its rows needs.

// Column statistics: sum, sum of squares, minimum and maximum per coordinate.
// Thread t takes coordinate t % 8 of every 32nd column.
__global__ __launch_bounds__(kBlock) void wdim_partial_kernel(WeightArgs a)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) a.ctr->ts[kTsWeights] = wall_clock64();
    __shared__ double sh[4][kBlock];
    const int M = (int)*a.M, t = threadIdx.x, d = t & 7;
    double s1 = 0.0, s2 = 0.0, mn = __builtin_inf(), mx = -__builtin_inf();
    for (int k = blockIdx.x * (kBlock / 8) + t / 8; k < M; k += gridDim.x * (kBlock / 8)) {
        const double v = a.cols[(size_t)k * 9 + d];
        s1 += v;
        s2 += v * v;
        mn = v < mn ? v : mn;
        mx = v > mx ? v : mx;
    }
    sh[0][t] = s1;
    sh[1][t] = s2;
    sh[2][t] = mn;
    sh[3][t] = mx;
    __syncthreads();
    for (int off = kBlock / 2; off >= 8; off >>= 1) {
        if (t < off) {
            sh[0][t] += sh[0][t + off];
            sh[1][t] += sh[1][t + off];
            sh[2][t] = sh[2][t] < sh[2][t + off] ? sh[2][t] : sh[2][t + off];
            sh[3][t] = sh[3][t] > sh[3][t + off] ? sh[3][t] : sh[3][t + off];
        }
        __syncthreads();
    }
    if (t < 32) a.dimpart[blockIdx.x * 32 + t] = sh[t >> 3][t & 7];
}

__global__ __launch_bounds__(kBlock) void wgeom_kernel(WeightArgs a)
{
    __shared__ double sh[kBlock];
    const int t = threadIdx.x, which = (t & 31) >> 3;
    double v = which < 2 ? 0.0 : (which == 2 ? __builtin_inf() : -__builtin_inf());
    for (int b = t >> 5; b < kDimBlocks; b += kBlock / 32) {
        const double p = a.dimpart[b * 32 + (t & 31)];
        v = which < 2 ? v + p : (which == 2 ? (p < v ? p : v) : (p > v ? p : v));
    }
    sh[t] = v;
    __syncthreads();
    for (int off = kBlock / 2; off >= 32; off >>= 1) {
        if (t < off) {
            const double p = sh[t + off];
            sh[t] = which < 2 ? sh[t] + p : (which == 2 ? (p < sh[t] ? p : sh[t]) : (p > sh[t] ? p : sh[t]));
        }
        __syncthreads();
    }
    wterm::make_geom(sh, sh + 8, sh + 16, sh + 24, (double)*a.M, a.geom);
}

// Sort key of column i, or of row i, whose window radius it stores; cells: this
// thread's column of an LDS array, `stride` threads apart.
__device__ __forceinline__ unsigned long long sort_key(const WeightArgs& a, const WeightGeom& g, size_t i, bool row,
                                                       uint32_t* cells, int stride)
{
    double u[kNP];
#pragma unroll
    for (int d = 0; d < kNP; ++d) {
        u[d] = row ? a.u[i * kNP + d] : a.cols[i * 9 + d];
        cells[d * stride] = wterm::cell20(u[d], g.lo[d], g.inv[d]);
    }
    uint32_t key = wterm::morton32(g, cells, stride);
    if (row) {
        const double sj = a.sigma[i];
        // half-octaves in descending order: the widest windows are dispatched first
        key = ((127u - (uint32_t)sigma_half_octave(sj)) << 25) | (key >> 7);
        const int32_t par = a.parent[i];
        const bool ok = par >= 0 && par < a.n_prev;
        a.rwin[i] = wterm::window_radius(u, sj, ok ? a.u_prev + (size_t)par * kNP : u, ok ? (double)a.q_prev[par] : 0.0,
                                         (double)a.cdf[a.n_prev - 1]);
    }
    return ((unsigned long long)key << 32) | (unsigned long long)i;
}

// Keys of the columns (grid.y 0) and of the rows (grid.y 1), padded for the
// bitonic sort unless they go to the counting sort.
__global__ __launch_bounds__(kBlock) void wkeys_kernel(WeightArgs a)
{
    __shared__ uint32_t cells[kNP * kBlock];
    const size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x;
    const bool row = blockIdx.y != 0, rank = a.N <= kRankSort;
    const size_t n = (size_t)(row ? a.N : (int)*a.M);
    unsigned long long* keys = rank ? a.unsorted[row] : (row ? a.rowkeys : a.colkeys);
    if (i < n) keys[i] = sort_key(a, *a.geom, i, row, cells + threadIdx.x, kBlock);
    else if (!rank && i < a.npad) keys[i] = ~0ull;
}

// Statistics, sort code and keys in one workgroup (N <= kOnePrep).
__global__ __launch_bounds__(kOneThreads) void wprep_one_kernel(WeightArgs a)
{
    __shared__ union {
        double stat[4][kOneThreads];
        uint32_t cells[kNP * kOneThreads];
    } sh;
    __shared__ double fin[32];
    __shared__ WeightGeom g;
    const int M = (int)*a.M, t = threadIdx.x, d = t & 7;
    if (t == 0) a.ctr->ts[kTsWeights] = wall_clock64();
    double v[4] = {0.0, 0.0, __builtin_inf(), -__builtin_inf()};
    for (int k = t / 8; k < M; k += kOneThreads / 8) {
        const double x = a.cols[(size_t)k * 9 + d];
        v[0] += x;
        v[1] += x * x;
        v[2] = x < v[2] ? x : v[2];
        v[3] = x > v[3] ? x : v[3];
    }
    // the eight threads of a wave that share a coordinate, then the waves
#pragma unroll
    for (int off = 8; off < kWave; off <<= 1) {
        v[0] += __shfl_xor(v[0], off, kWave);
        v[1] += __shfl_xor(v[1], off, kWave);
        const double lo = __shfl_xor(v[2], off, kWave), hi = __shfl_xor(v[3], off, kWave);
        v[2] = lo < v[2] ? lo : v[2];
        v[3] = hi > v[3] ? hi : v[3];
    }
    if ((t & (kWave - 1)) < 8)
        for (int q = 0; q < 4; ++q) sh.stat[q][(t / kWave) * 8 + d] = v[q];
    __syncthreads();
    if (t < 32) {
        const int q = t >> 3;
        double r = sh.stat[q][t & 7];
        for (int w = 1; w < kOneWaves; ++w) {
            const double o = sh.stat[q][w * 8 + (t & 7)];
            r = q < 2 ? r + o : (q == 2 ? (o < r ? o : r) : (o > r ? o : r));
        }
        fin[t] = r;
    }
    __syncthreads();
    wterm::make_geom(fin, fin + 8, fin + 16, fin + 24, (double)M, &g);
    __syncthreads();
    if (t == 0) *a.geom = g;
    for (int i = t; i < M; i += kOneThreads) a.unsorted[0][i] = sort_key(a, g, i, false, sh.cells + t, kOneThreads);
    for (int i = t; i < a.N; i += kOneThreads) a.unsorted[1][i] = sort_key(a, g, i, true, sh.cells + t, kOneThreads);
}

// Counting sort of unique keys: a key's place is the number of smaller ones.
// 64 keys a workgroup; its sixteen waves count among a share each of every
// LDS tile of all keys (scalar loads instead left each wave waiting for the
// next eight keys, 48 us at 5003).  n^2 comparisons on the whole chip: 4.6 us
// up to 1024, 11 us at 5003 and 34 us at 16384, rows and columns together,
// where the bitonic sort's first launch alone takes 24.
constexpr int kRankTile = 2048;

__global__ __launch_bounds__(kOneThreads) void wrank_kernel(WeightArgs a)
{
    __shared__ unsigned long long tile[kRankTile];
    __shared__ unsigned int part[kOneWaves][kWave];
    const bool row = blockIdx.y != 0;
    const int n = row ? a.N : (int)*a.M;
    if ((int)blockIdx.x * kWave >= n) return;
    const unsigned long long* keys = a.unsorted[row];
    const int t = threadIdx.x, w = t / kWave, lane = t & (kWave - 1);
    const int i = blockIdx.x * kWave + lane;
    const unsigned long long mine = i < n ? keys[i] : 0ull;
    constexpr int share = kRankTile / kOneWaves;
    unsigned int less = 0;
    for (int base = 0; base < n; base += kRankTile) {
        __syncthreads();
#pragma unroll
        for (int k = t; k < kRankTile; k += kOneThreads) tile[k] = base + k < n ? keys[base + k] : ~0ull;
        __syncthreads();
        if (base + w * share < n) {
#pragma unroll 16
            for (int j = 0; j < share; ++j) less += tile[w * share + j] < mine ? 1u : 0u;
        }
    }
    part[w][lane] = less;
    __syncthreads();
    if (w == 0 && i < n) {
        for (int k = 1; k < kOneWaves; ++k) less += part[k][lane];
        (row ? a.rowkeys : a.colkeys)[less] = mine;
    }
}

// Sorted columns (a wave per tile) and sorted rows (a wave per group).
__global__ __launch_bounds__(kBlock) void wgather_kernel(WeightArgs a)
{
    const size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (blockIdx.y == 0) {
        const int M = (int)*a.M;
        if (i < a.sc.pad && i < weight_col_pad((size_t)M))
            wterm::gather_column(a.sc, *a.geom, i, i < (size_t)M,
                                 a.cols + (i < (size_t)M ? (size_t)(a.colkeys[i] & 0xFFFFFFFFull) : 0) * 9);
    } else if (i < a.sr.pad) {
        const bool real = i < (size_t)a.N;
        const size_t j = real ? (size_t)(a.rowkeys[i] & 0xFFFFFFFFull) : 0;
        wterm::gather_row(a.sr, *a.geom, i, real, a.u + j * kNP, a.sigma[j], a.rwin[j], a.ex);
    }
}

// grid (row blocks, chunks): kGroups groups of 64 rows against the tiles of the
// chunk, a group's near tiles dealt in turn to kSplit waves.
// Five waves a SIMD (96 VGPRs) hide the columns' scalar loads best: 262 ms in
// stage 1 of N = 2^20 against 295 at six; 128 rows a workgroup balance better
// than 256 (16.2 against 18.0 ms in a run of N = 131072).  In later stages a
// few groups of wide rows hold most of the work and the launch lasts as long
// as their longest wave: dealt to four waves, 8 stages of N = 20011 take 0.60
// ms for 0.67, the last four of 10 at N = 131072 2.2 for 2.5 (weight_split).
// A run's launches against a window on one sorted coordinate: N = 20011 (8
// stages) 1.81 -> 0.60 ms, 131072 (10) 27.7 -> 14.8 ms, 2^20 (4) 876 -> 559 ms;
// the early stages are at 90-95% of the vector issue rate.
template <int kGroups, int kSplit>
__global__ __launch_bounds__(kGroups * kSplit * kWave) __attribute__((amdgpu_waves_per_eu(5))) void weights_kernel(
    WeightArgs a)
{
    __shared__ double T[wterm::kTab];
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0 && a.first_chunk == 0) a.ctr->ts[kTsSum] = wall_clock64();
    const int M = (int)*a.M;
    const int chunk = a.first_chunk + (int)blockIdx.y;
    const int t0 = chunk * a.chunk_tiles;
    const int t1 = min((M + kColTile - 1) / kColTile, t0 + a.chunk_tiles);
    if (t0 >= t1) return;  // past the columns: the finalize pass does not read this chunk
    const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x / kWave), lane = threadIdx.x & (kWave - 1);
    const int g = w / kSplit, split = w % kSplit;
    const int group = (int)blockIdx.x * kGroups + g, r = group * kWave + lane;
    // most workgroups of the late stages have no tile near: they leave before
    // the table and the rows are loaded
    const unsigned long long first = wterm::near_tiles(a.sr, a.sc, group, lane, t0, t1);
    double total = 0.0;
    uint2 c = make_uint2(0, 0);
    if (__syncthreads_or(first != 0 || t1 - t0 > kWave)) {
        wterm::load_table(T, a.tab);
        __syncthreads();
        total = wterm::row_sum(a.sr, a.sc, group, lane, t0, t1, M, first, T, a.ex, c.x, c.y, split, kSplit);
        if constexpr (kSplit > 1) {  // (a barrier here cost 1% where a wave has its group to itself)
            __shared__ double part[kGroups][kSplit][kWave];
            __shared__ uint2 count[kGroups][kSplit];
            part[g][split][lane] = total;
            if (lane == 0) count[g][split] = c;
            __syncthreads();
            total = 0.0;
            c = make_uint2(0, 0);
#pragma unroll
            for (int i = 0; i < kSplit; ++i) {
                total += part[g][i][lane];
                c.x += count[g][i].x;
                c.y += count[g][i].y;
            }
        }
    }
    if (split != 0) return;
    if (r < a.N) a.partial[(size_t)(a.first_slot + (int)blockIdx.y) * a.N + r] = total;
    // (counted per group and added up by the finalize pass: 130000 atomics on one
    // line took longer than the smaller stages' sums)
    if (lane == 0) a.counts[(size_t)chunk * (a.sr.pad / kWave) + group] = c;
}

__global__ __launch_bounds__(kBlock) void wtable_kernel(double* tab)
{
    const int i = blockIdx.x * kBlock + threadIdx.x;
    if (i < wterm::kTab) tab[i] = wterm::table_entry(i);
}

// Test hook: one importance-weight term per record {u_j[8], sigma_j, u_k[8],
// q_k}, by the weight kernels' own term code (table exponential from LDS,
// scaled by the row's c_j), accumulated as the first term of a row sum.
__global__ __launch_bounds__(kBlock) void wterm_debug_kernel(int64_t n, const double* in, double* out, WeightArgs a)
{
    __shared__ double T[wterm::kTab];
    for (int i = threadIdx.x; i < wterm::kTab; i += kBlock) T[i] = wterm::table_entry(i);
    __syncthreads();
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const double* r = in + (size_t)i * 18;
    double uj[kNP];
    wterm::Col c;
#pragma unroll
    for (int d = 0; d < kNP; ++d) {
        uj[d] = r[d];
        c.u[d] = r[9 + d];
    }
    c.q = r[17];
    const double cj = wterm::row_scale(r[8], a.ex);
    const double D = wterm::dist2(uj, c), R = wterm::kWindow * r[8];
    out[i] = D <= R * R ? __builtin_fma(c.q, wterm::term_exp(D, cj, T, a.ex, a.ex[1]), 0.0) * wterm::kSumScale : 0.0;
}

// Chunks that hold columns.
__device__ __forceinline__ int used_chunks(const WeightArgs& a)
{
    const int tiles = ((int)*a.M + kColTile - 1) / kColTile;
    return min(a.chunks, (tiles + a.chunk_tiles - 1) / a.chunk_tiles);
}

// Sum of row r over the chunks before `end`, in order.
__device__ __forceinline__ double row_total(const WeightArgs& a, int r, int end)
{
    const int n = a.first_slot + max(end - a.first_chunk, 0);
    double L = 0.0;
#pragma unroll 8
    for (int c = 0; c < n; ++c) L += a.partial[(size_t)c * a.N + r];
    return L;
}

// The sums so far to slot 0, for another pass (fewer slots than chunks).
__global__ __launch_bounds__(kBlock) void weights_fold_kernel(WeightArgs a)
{
    const int r = blockIdx.x * kBlock + threadIdx.x;
    if (r < a.N) a.partial[r] = row_total(a, r, min(used_chunks(a), a.first_chunk + a.slots - a.first_slot));
}

__global__ __launch_bounds__(kBlock) void weights_finalize_kernel(WeightArgs a)
{
    const int r = blockIdx.x * kBlock + threadIdx.x;
    if (r == 0) a.ctr->ts[kTsSummed] = wall_clock64();
    const int nch = used_chunks(a);
    // a wave's group: its terms and window pairs
    const int group = r / kWave, lane = threadIdx.x & (kWave - 1);
    if (group * kWave < a.N) {
        unsigned long long listed = 0, window = 0;
        for (int c = lane; c < nch; c += kWave) {
            const uint2 n = a.counts[(size_t)c * (a.sr.pad / kWave) + group];
            listed += n.x;
            window += n.y;
        }
        listed = wave_sum_u64(listed);
        window = wave_sum_u64(window);
        if (lane == 0 && listed) {
            atomicAdd(a.terms, listed * (unsigned long long)min(kWave, a.N - group * kWave));
            atomicAdd(a.window_terms, window);
        }
    }
    if (r >= a.N) return;
    const double L = row_total(a, r, nch);
    const size_t j = (size_t)(a.rowkeys[r] & 0xFFFFFFFFull);
    a.logw[j] = 8.0 * dm::log(a.sigma[j]) - dm::log(L);
}

// ---------------------------------------------------------------------------
// W_j = exp(l_j - max l) / sum; ESS = 1 / sum W^2.  Per-block partials
// combined in block order.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void norm_max_kernel(NormArgs a)
{
    __shared__ double sh[kBlock];
    double mx = -__builtin_inf();
    for (int i = 0; i < kPer; ++i) {
        const int j = blockIdx.x * kChunk + i * kBlock + threadIdx.x;
        if (j < a.N) mx = a.logw[j] > mx ? a.logw[j] : mx;
    }
    mx = block_max_f64(mx, sh);
    if (threadIdx.x == 0) a.sc.d0[blockIdx.x] = mx;
}

__global__ __launch_bounds__(kBlock) void norm_exp_kernel(NormArgs a)
{
    __shared__ double sh[kBlock];
    double mx = -__builtin_inf();
    for (int b = threadIdx.x; b < (int)gridDim.x; b += kBlock) mx = a.sc.d0[b] > mx ? a.sc.d0[b] : mx;
    mx = block_max_f64(mx, sh);
    double s = 0.0;
    for (int i = 0; i < kPer; ++i) {
        const int j = blockIdx.x * kChunk + i * kBlock + threadIdx.x;
        if (j < a.N) {
            const double e = dm::exp(a.logw[j] - mx);
            a.W[j] = e;
            s += e;
        }
    }
    s = block_sum_f64(s, sh);
    if (threadIdx.x == 0) a.sc.d1[blockIdx.x] = s;
}

__device__ __forceinline__ double ordered_total(const double* part, int G, double* sh)
{
    // each thread sums a contiguous run of block partials, then a fixed tree
    const int per = (G + kBlock - 1) / kBlock;
    double s = 0.0;
    const int b0 = threadIdx.x * per, b1 = min(G, b0 + per);
    for (int b = b0; b < b1; ++b) s += part[b];
    return block_sum_f64(s, sh);
}

__global__ __launch_bounds__(kBlock) void norm_scale_kernel(NormArgs a)
{
    __shared__ double sh[kBlock];
    const double total = ordered_total(a.sc.d1, gridDim.x, sh);
    double s2 = 0.0;
    for (int i = 0; i < kPer; ++i) {
        const int j = blockIdx.x * kChunk + i * kBlock + threadIdx.x;
        if (j < a.N) {
            const double w = a.W[j] / total;
            a.W[j] = w;
            s2 += w * w;
        }
    }
    s2 = block_sum_f64(s2, sh);
    if (threadIdx.x == 0) a.sc.d0[blockIdx.x] = s2;
}

__global__ __launch_bounds__(kBlock) void norm_ess_kernel(NormArgs a, int G)
{
    __shared__ double sh[kBlock];
    const double s2 = ordered_total(a.sc.d0, G, sh);
    if (threadIdx.x == 0) *a.ess = 1.0 / s2;
}

__global__ __launch_bounds__(kBlock) void uniform_weights_kernel(NormArgs a)
{
    const int j = blockIdx.x * kBlock + threadIdx.x;
    if (j < a.N) {
        a.W[j] = 1.0 / (double)a.N;
        a.logw[j] = 0.0;
    }
}

// The same in one workgroup (N <= kOneEnd).
__device__ __forceinline__ void normalise_one(const NormArgs& a, double* sh)
{
    const int t = threadIdx.x;
    if (a.uniform) {
        for (int j = t; j < a.N; j += kOneThreads) {
            a.W[j] = 1.0 / (double)a.N;
            a.logw[j] = 0.0;
        }
        return;
    }
    constexpr int kMost = kOneEnd / kOneThreads;
    double e[kMost];
    double mx = -__builtin_inf();
#pragma unroll
    for (int i = 0; i < kMost; ++i) {
        const int j = t + i * kOneThreads;
        e[i] = j < a.N ? a.logw[j] : -__builtin_inf();
        mx = e[i] > mx ? e[i] : mx;
    }
    mx = one_reduce(mx, sh, [](double x, double y) { return x > y ? x : y; });
    const auto add = [](double x, double y) { return x + y; };
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < kMost; ++i) {
        if (t + i * kOneThreads < a.N) {
            e[i] = dm::exp(e[i] - mx);
            s += e[i];
        }
    }
    s = one_reduce(s, sh, add);
    double s2 = 0.0;
#pragma unroll
    for (int i = 0; i < kMost; ++i) {
        const int j = t + i * kOneThreads;
        if (j < a.N) {
            const double w = e[i] / s;
            a.W[j] = w;
            s2 += w * w;
        }
    }
    s2 = one_reduce(s2, sh, add);
    if (t == 0) *a.ess = 1.0 / s2;
}

// ---------------------------------------------------------------------------
// eq. 8 tolerance: type-7 percentile with numpy's "linear" arithmetic.  Up to
// kSelectOne values one workgroup selects (blockselect.h: three passes at one
// compute unit's L2 rate, 25 us at 20011 values).  More take four launches of the same
// method: the range of the values, a histogram of the 11 bits from the highest
// one they differ in, the values of the rank's bin collected beside the
// smallest value above it, and one workgroup that finishes among those (more than
// its list holds: crowd_hist_kernel).
// 38-50 us at 2^17 and 54-78 at 2^18 (one workgroup: 88 and 165), where six
// fixed digits in thirteen launches took 76 at 2^17.
// ---------------------------------------------------------------------------
constexpr int kSelectOne = 1 << 15;
constexpr int kBins = bsel::kBins;

__device__ __forceinline__ void note_select(const SelectArgs& a)
{
    if (a.ctr && blockIdx.x == 0 && threadIdx.x == 0) a.ctr->ts[kTsSelect] = wall_clock64();
}

__global__ __launch_bounds__(bsel::kThreads) void select_one_kernel(SelectArgs a)
{
    __shared__ bsel::Shared sh;
    note_select(a);
    const double r = bsel::quantile7(bsel::FromMemory{a.x, a.N}, a.N, a.alpha, sh);
    if (threadIdx.x == 0) *a.out = r;
}

// The end of a small stage: workgroup 0 selects, workgroup 1 normalises.
__global__ __launch_bounds__(kOneThreads) void stage_end_one_kernel(NormArgs n, SelectArgs q)
{
    __shared__ union {
        bsel::Shared sel;
        double red[kOneWaves];
    } sh;
    if (blockIdx.x == 0) {
        note_select(q);
        const double r = bsel::quantile7(bsel::FromMemory{q.x, q.N}, q.N, q.alpha, sh.sel);
        if (threadIdx.x == 0) *q.out = r;
    } else {
        normalise_one(n, sh.red);
    }
}

// Counters and results of the stage to host memory, a thread a word.
__global__ __launch_bounds__(kWave) void publish_kernel(StageCounters* ctr, StageCounters* host)
{
    constexpr int words = sizeof(StageCounters) / 8;
    static_assert(words <= kWave, "a thread a word");
    if (threadIdx.x == 0) ctr->ts[kTsEnd] = wall_clock64();
    __syncthreads();
    if (threadIdx.x < words) ((unsigned long long*)host)[threadIdx.x] = ((unsigned long long*)ctr)[threadIdx.x];
    __threadfence_system();
}

// Per-block minimum and maximum (u0, u1); block 0 clears the histogram and the
// collected count.
__global__ __launch_bounds__(kBlock) void select_range_kernel(SelectArgs a)
{
    __shared__ unsigned long long slo[kBlock / kWave], shi[kBlock / kWave];
    note_select(a);
    unsigned long long lo = ~0ull, hi = 0ull;
#pragma unroll 4
    for (int k = blockIdx.x * kBlock + threadIdx.x; k < a.N; k += gridDim.x * kBlock) {
        const unsigned long long b = bsel::bits_of(a.x[k]);
        lo = b < lo ? b : lo;
        hi = b > hi ? b : hi;
    }
    lo = bsel::wave_min64(lo);
    hi = bsel::wave_max64(hi);
    if ((threadIdx.x & (kWave - 1)) == 0) {
        slo[threadIdx.x / kWave] = lo;
        shi[threadIdx.x / kWave] = hi;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / kWave; ++w) {
            lo = slo[w] < lo ? slo[w] : lo;
            hi = shi[w] > hi ? shi[w] : hi;
        }
        a.sc.u0[blockIdx.x] = lo;
        a.sc.u1[blockIdx.x] = hi;
    }
    if (blockIdx.x == 0) {
        for (int b = threadIdx.x; b < kBins; b += kBlock) a.sc.hist[b] = 0u;
        if (threadIdx.x == 0) a.sc.sel[0] = 0ull;
    }
}

// The range of all values from the blocks' (every thread gets it), the digit's
// shift and the first bin's prefix.
struct Digit {
    unsigned long long lo, hi, base;
    int sh;
};

__device__ __forceinline__ Digit select_digit(const SelectArgs& a, int G, unsigned long long* shu)
{
    Digit g{~0ull, 0ull, 0ull, 0};
    for (int b = threadIdx.x; b < G; b += kBlock) {
        g.lo = a.sc.u0[b] < g.lo ? a.sc.u0[b] : g.lo;
        g.hi = a.sc.u1[b] > g.hi ? a.sc.u1[b] : g.hi;
    }
    g.lo = bsel::wave_min64(g.lo);
    g.hi = bsel::wave_max64(g.hi);
    constexpr int nw = kBlock / kWave;
    if ((threadIdx.x & (kWave - 1)) == 0) {
        shu[threadIdx.x / kWave] = g.lo;
        shu[nw + threadIdx.x / kWave] = g.hi;
    }
    __syncthreads();
    for (int w = 0; w < nw; ++w) {
        g.lo = shu[w] < g.lo ? shu[w] : g.lo;
        g.hi = shu[nw + w] > g.hi ? shu[nw + w] : g.hi;
    }
    const int top = g.lo == g.hi ? 0 : 63 - __builtin_clzll(g.lo ^ g.hi);
    g.sh = top > 10 ? top - 10 : 0;
    g.base = g.lo >> g.sh;
    __syncthreads();
    return g;
}

__global__ __launch_bounds__(kBlock) void select_hist_kernel(SelectArgs a)
{
    __shared__ unsigned int h[kBins];
    __shared__ unsigned long long shu[2 * kBlock / kWave];
    for (int b = threadIdx.x; b < kBins; b += kBlock) h[b] = 0u;
    const Digit g = select_digit(a, gridDim.x, shu);
#pragma unroll 4
    for (int k = blockIdx.x * kBlock + threadIdx.x; k < a.N; k += gridDim.x * kBlock)
        atomicAdd(&h[(unsigned)((bsel::bits_of(a.x[k]) >> g.sh) - g.base)], 1u);
    __syncthreads();
    for (int b = threadIdx.x; b < kBins; b += kBlock)
        if (h[b]) atomicAdd(&a.sc.hist[b], h[b]);
}

// Bin of the rank (every block finds it), its values collected into the list
// (unless they are more than it holds), the block's smallest value above.
__global__ __launch_bounds__(kBlock) void select_collect_kernel(SelectArgs a)
{
    __shared__ unsigned long long shu[kBlock];
    __shared__ unsigned int s_bin, s_below, s_count;
    const Digit g = select_digit(a, gridDim.x, shu);
    int r0, r1;
    bsel::ranks7(a.N, a.alpha, r0, r1);
    constexpr int per = kBins / kBlock;
    unsigned int h[per];
    unsigned long long s = 0, tot;
#pragma unroll
    for (int i = 0; i < per; ++i) {
        h[i] = a.sc.hist[threadIdx.x * per + i];
        s += h[i];
    }
    unsigned long long run = block_excl_scan_u64(s, shu, &tot);
#pragma unroll
    for (int i = 0; i < per; ++i) {
        if (run <= (unsigned)r0 && (unsigned)r0 < run + h[i]) {
            s_bin = threadIdx.x * per + i;
            s_below = (unsigned int)run;
            s_count = h[i];
        }
        run += h[i];
    }
    __syncthreads();
    const unsigned long long want = g.base + s_bin;
    unsigned long long above = ~0ull;
    if (s_count <= a.sc.list_cap) {
#pragma unroll 4
        for (int k = blockIdx.x * kBlock + threadIdx.x; k < a.N; k += gridDim.x * kBlock) {
            const double x = a.x[k];
            const unsigned long long b = bsel::bits_of(x), d = b >> g.sh;
            if (d == want) a.sc.list[atomicAdd(&a.sc.sel[0], 1ull)] = x;
            else if (d > want && b < above) above = b;
        }
    }
    above = bsel::wave_min64(above);
    if ((threadIdx.x & (kWave - 1)) == 0) shu[threadIdx.x / kWave] = above;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / kWave; ++w) above = shu[w] < above ? shu[w] : above;
        a.sc.u2[blockIdx.x] = above;
        if (blockIdx.x == 0) {
            a.sc.sel[1] = s_below;
            a.sc.sel[2] = s_count;
            a.sc.sel[3] = want << g.sh;
            a.sc.sel[4] = (unsigned long long)g.sh;
            a.sc.sel[5] = (unsigned)r0 - s_below;
        }
    }
}

__global__ __launch_bounds__(bsel::kThreads) void select_finish_kernel(SelectArgs a, int G)
{
    __shared__ bsel::Shared sh;
    int r0, r1;
    bsel::ranks7(a.N, a.alpha, r0, r1);
    const unsigned int count = (unsigned int)a.sc.sel[2], rank = (unsigned int)r0 - (unsigned int)a.sc.sel[1];
    unsigned long long xa, xb;
    const bool crowded = count > a.sc.list_cap;  // into one of 2048 bins
    if (threadIdx.x == 0) {
        a.sc.sel[6] = crowded ? 1ull : 0ull;
        if (a.ctr) a.ctr->crowded = a.sc.sel[6];
    }
    if (crowded) {  // launch_select_crowded
        for (int b = threadIdx.x; b < kBins; b += bsel::kThreads) a.sc.hist[b] = 0u;
        return;
    }
    bsel::order_pair(bsel::FromMemory{a.sc.list, (int)count}, (int)count, rank, sh);
    xa = sh.xa;
    xb = sh.xb;
    if (rank + 1 >= count) {
        xb = ~0ull;
        for (int b = 0; b < G; ++b) xb = a.sc.u2[b] < xb ? a.sc.u2[b] : xb;
    }
    if (threadIdx.x == 0) *a.out = bsel::interpolate7(a.N, a.alpha, xa, xb);
}

// Crowded values (few distinct ones, or a range stretched by outliers): digits
// of 11 bits from the rank's bin down, by all of the chip, until the prefix is
// the value.  The first launches of select have the 11 bits above; at most five
// digits are left.  Few distinct values: 0.06 ms at 40000, 0.11 at 2^20 and 0.19 at
// 2^22, where one workgroup over all of them took 0.19, 5.4 and 21.6; a third stage
// of 2^22 particles x 20 days 0.18 for 5.2.  Where values are not crowded these
// launches do nothing.
constexpr int kCrowdDigits = 5;

__global__ __launch_bounds__(kBlock) void crowd_hist_kernel(SelectArgs a)
{
    __shared__ unsigned int h[kBins];
    const int left = (int)a.sc.sel[4];
    if (!a.sc.sel[6] || left == 0) return;
    const int sh = left > 11 ? left - 11 : 0;
    const unsigned long long prefix = a.sc.sel[3] >> left, digits = (1ull << (left - sh)) - 1ull;
    for (int b = threadIdx.x; b < kBins; b += kBlock) h[b] = 0u;
    __syncthreads();
    const int lane = threadIdx.x & (kWave - 1);
    for (int k0 = blockIdx.x * kBlock; k0 < a.N; k0 += gridDim.x * kBlock) {
        const int k = k0 + (int)threadIdx.x;
        const unsigned long long b = k < a.N ? bsel::bits_of(a.x[k]) : 0ull;
        bool mine = k < a.N && b >> left == prefix;
        const unsigned int d = (unsigned int)((b >> sh) & digits);
        // a few rounds of one addition for all lanes of a digit (the same LDS word
        // takes one lane after the other)
        for (int i = 0; i < 4; ++i) {
            const unsigned long long todo = __ballot(mine);
            if (!todo) break;
            const unsigned int one = __shfl(d, __builtin_ctzll(todo), kWave);
            const unsigned long long same = __ballot(mine && d == one);
            if (lane == __builtin_ctzll(todo)) atomicAdd(&h[one], (unsigned int)__popcll(same));
            if (d == one) mine = false;
        }
        if (mine) atomicAdd(&h[d], 1u);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < kBins; b += kBlock)
        if (h[b]) atomicAdd(&a.sc.hist[b], h[b]);
}

// The rank's digit; the histogram is cleared for the next one.
__global__ __launch_bounds__(kBlock) void crowd_pick_kernel(SelectArgs a)
{
    __shared__ unsigned long long shu[kBlock];
    const int left = (int)a.sc.sel[4];
    const unsigned long long rank = a.sc.sel[5], prefix = a.sc.sel[3];
    if (!a.sc.sel[6] || left == 0) return;
    const int sh = left > 11 ? left - 11 : 0;
    constexpr int per = kBins / kBlock;
    unsigned int h[per];
    unsigned long long s = 0, tot;
#pragma unroll
    for (int i = 0; i < per; ++i) {
        h[i] = a.sc.hist[threadIdx.x * per + i];
        a.sc.hist[threadIdx.x * per + i] = 0u;
        s += h[i];
    }
    unsigned long long run = block_excl_scan_u64(s, shu, &tot);  // (all threads have read the state)
#pragma unroll
    for (int i = 0; i < per; ++i) {
        if (run <= rank && rank < run + h[i]) {
            a.sc.sel[2] = h[i];
            a.sc.sel[3] = prefix | (unsigned long long)(threadIdx.x * per + i) << sh;
            a.sc.sel[4] = (unsigned long long)sh;
            a.sc.sel[5] = rank - run;
        }
        run += h[i];
    }
}

// Per-block smallest value above the one found.
__global__ __launch_bounds__(kBlock) void crowd_above_kernel(SelectArgs a)
{
    __shared__ unsigned long long sh[kBlock / kWave];
    if (!a.sc.sel[6]) return;
    const unsigned long long xa = a.sc.sel[3];
    unsigned long long above = ~0ull;
#pragma unroll 4
    for (int k = blockIdx.x * kBlock + threadIdx.x; k < a.N; k += gridDim.x * kBlock) {
        const unsigned long long b = bsel::bits_of(a.x[k]);
        if (b > xa && b < above) above = b;
    }
    above = bsel::wave_min64(above);
    if ((threadIdx.x & (kWave - 1)) == 0) sh[threadIdx.x / kWave] = above;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < kBlock / kWave; ++w) above = sh[w] < above ? sh[w] : above;
        a.sc.u2[blockIdx.x] = above;
    }
}

__global__ __launch_bounds__(kWave) void crowd_finish_kernel(SelectArgs a, int G)
{
    if (!a.sc.sel[6]) return;
    const unsigned long long count = a.sc.sel[2], xa = a.sc.sel[3], rank = a.sc.sel[5];
    unsigned long long above = ~0ull;
    for (int b = threadIdx.x; b < G; b += kWave) above = a.sc.u2[b] < above ? a.sc.u2[b] : above;
    above = bsel::wave_min64(above);
    if (threadIdx.x == 0) *a.out = bsel::interpolate7(a.N, a.alpha, xa, rank + 1 < count ? xa : above);
}

// theta_d = lo_d + u_d (hi_d - lo_d) for the copy-out of a population.
__global__ __launch_bounds__(kBlock) void to_theta_kernel(const double* u, Model m, double* theta, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n * kNP) return;
    const int d = (int)(i % kNP);
    theta[i] = m.lo[d] + u[i] * m.width[d];
}

inline unsigned blocks_of(int64_t n, int per) { return (unsigned)((n + per - 1) / per); }

}  // namespace

void weight_exp_constants(double ex[7])
{
    const double L = 0.6931471805599453 / 1024.0;  // ln2 / 1024 (exact scaling of the double ln 2)
    ex[0] = L;
    ex[1] = (L * L) / 2.0;
    ex[2] = (L * L * L) / 6.0;
    ex[3] = 1477.3197218702985;           // 1024 / ln 2
    ex[4] = ex[5] = ex[6] = 0.0;
}

void launch_to_theta(const double* u, const Model& m, double* theta, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(to_theta_kernel, dim3(blocks_of(n * kNP, kBlock)), dim3(kBlock), 0, s, u, m, theta, n);
}

void launch_resample(const ResampleArgs& a, hipStream_t s)
{
    if (a.N <= kOneResample) {
        hipLaunchKernelGGL(resample_one_kernel, dim3(1), dim3(kOneThreads), 0, s, a);
        return;
    }
    const dim3 g(blocks_of(a.N, kChunk)), b(kBlock);
    hipLaunchKernelGGL(resample_stats_kernel, g, b, 0, s, a);
    hipLaunchKernelGGL(resample_count_kernel, g, b, 0, s, a);
    hipLaunchKernelGGL(resample_write_kernel, g, b, 0, s, a);
}

void launch_weights_window(const WeightArgs& a, hipStream_t s)
{
    const dim3 b(kBlock);
    if (a.N <= kOnePrep) {
        hipLaunchKernelGGL(wprep_one_kernel, dim3(1), dim3(kOneThreads), 0, s, a);
    } else {
        const size_t n = a.N <= kRankSort ? (size_t)a.N : a.npad;
        hipLaunchKernelGGL(wdim_partial_kernel, dim3(kDimBlocks), b, 0, s, a);
        hipLaunchKernelGGL(wgeom_kernel, dim3(1), b, 0, s, a);
        hipLaunchKernelGGL(wkeys_kernel, dim3(blocks_of((int64_t)n, kBlock), 2), b, 0, s, a);
    }
    if (a.N <= kRankSort) hipLaunchKernelGGL(wrank_kernel, dim3(blocks_of(a.N, kWave), 2), dim3(kOneThreads), 0, s, a);
    else launch_sort_u64_pair(a.colkeys, a.rowkeys, a.npad, s);
    hipLaunchKernelGGL(wgather_kernel, dim3(blocks_of((int64_t)a.sr.pad, kBlock), 2), b, 0, s, a);
}

void launch_wterm_debug(int64_t n, const double* in, double* out, hipStream_t s)
{
    WeightArgs a{};
    weight_exp_constants(a.ex);
    hipLaunchKernelGGL(wterm_debug_kernel, dim3(blocks_of(n, kBlock)), dim3(kBlock), 0, s, n, in, out, a);
}

void launch_weight_table(double* tab, hipStream_t s)
{
    hipLaunchKernelGGL(wtable_kernel, dim3((wterm::kTab + kBlock - 1) / kBlock), dim3(kBlock), 0, s, tab);
}

constexpr int kWeightSplit = 4;

// Whether a group's tiles are dealt to four waves.  Below 2048 rows a launch is
// a few waves' latency (13 us for 14 dealt), from 2^18 on no wave's share
// stands out, and two groups at the same columns use the scalar cache better
// (559 ms for 565 in 4 stages of 2^20); 300000: 56.0 and 56.3.
static bool weight_split(int64_t N) { return N >= 2048 && N < ((int64_t)1 << 18); }

void launch_weights_sum(WeightArgs& a, hipStream_t s)
{
    a.first_chunk = a.first_slot = 0;
    for (;;) {
        const int n = std::min(a.slots - a.first_slot, a.chunks - a.first_chunk);
        if (weight_split(a.N))
            hipLaunchKernelGGL((weights_kernel<1, kWeightSplit>), dim3(blocks_of(a.N, kWave), n), dim3(kWeightSplit * kWave), 0,
                               s, a);
        else
            hipLaunchKernelGGL((weights_kernel<kWeightRows / kWave, 1>), dim3(blocks_of(a.N, kWeightRows), n),
                               dim3(kWeightRows), 0, s, a);
        if (a.first_chunk + n == a.chunks) return;
        hipLaunchKernelGGL(weights_fold_kernel, dim3(blocks_of(a.N, kBlock)), dim3(kBlock), 0, s, a);
        a.first_chunk += n;
        a.first_slot = 1;
    }
}

void launch_weights_finalize(const WeightArgs& a, hipStream_t s)
{
    hipLaunchKernelGGL(weights_finalize_kernel, dim3(blocks_of(a.N, kBlock)), dim3(kBlock), 0, s, a);
}

// Tiles per chunk.  Below 2048 rows: as many as leave 12000 workgroups of work
// (about half of N survives).  Dealt to four waves: 6000 workgroups (0.60 ms at
// N = 20011; 0.62 at 12000 and 0.65 at 3000), at least a tile a wave, at most 64
// tiles (14.7 ms at N = 131072; 15.0 with 32, 15.7 with 16) and 64 chunks.  From
// 2^18 on: 32 tiles doubled until 128 chunks are enough, and at most 112 chunks:
// the partial sums are most of the workspace there, and it has to fit in what
// earlier versions asked for (128 chunks at every size: 4 stages of 300000 26.7
// ms for 27.4, of 600000 97.2 for 97.8, of 2^18 and 2^20 the same).
int weight_chunk_tiles(int64_t N)
{
    const int64_t tiles = (N + kColTile - 1) / kColTile;
    if (weight_split(N)) {
        const int64_t groups = (N + kWave - 1) / kWave;
        const int64_t t = std::min<int64_t>(64, std::max<int64_t>(kWeightSplit, groups * tiles / 2 / 6000));
        return (int)std::max<int64_t>(t, (tiles + 63) / 64);
    }
    const int64_t rb = (N + kWeightRows - 1) / kWeightRows;
    int64_t t = std::min<int64_t>(16, std::max<int64_t>(1, rb * tiles / 2 / 12000));
    while ((tiles + t - 1) / t > 128) t *= 2;
    return (int)std::max<int64_t>(t, (tiles + 111) / 112);
}

int weight_chunks(int64_t N)
{
    const int64_t tiles = (N + kColTile - 1) / kColTile, t = weight_chunk_tiles(N);
    return (int)((tiles + t - 1) / t);
}

size_t weight_first_bytes(int64_t N)
{
    // partial sums of 1024 columns a chunk, doubled until 128 are enough, or of
    // 2048 workgroups and 64 chunks; keys; columns, their keys, radii; parameters
    int64_t cols = 1024;
    while ((N + cols - 1) / cols > 128) cols *= 2;
    const int64_t rows = (N + kBlock - 1) / kBlock;
    const int64_t chunks = std::max<int64_t>((N + cols - 1) / cols, std::min<int64_t>(64, 2048 / rows));
    return (size_t)N * 8 * (size_t)(chunks + 9 + 1 + 1 + kNP) + 2 * sort_padded_size((size_t)N) * 8;
}

void launch_stage_end(const NormArgs& a, const SelectArgs& q, hipStream_t s)
{
    if (a.N <= kOneEnd) {
        hipLaunchKernelGGL(stage_end_one_kernel, dim3(2), dim3(kOneThreads), 0, s, a, q);
        return;
    }
    if (a.uniform) {
        hipLaunchKernelGGL(uniform_weights_kernel, dim3(blocks_of(a.N, kBlock)), dim3(kBlock), 0, s, a);
    } else {
        const unsigned G = blocks_of(a.N, kChunk);
        hipLaunchKernelGGL(norm_max_kernel, dim3(G), dim3(kBlock), 0, s, a);
        hipLaunchKernelGGL(norm_exp_kernel, dim3(G), dim3(kBlock), 0, s, a);
        hipLaunchKernelGGL(norm_scale_kernel, dim3(G), dim3(kBlock), 0, s, a);
        hipLaunchKernelGGL(norm_ess_kernel, dim3(1), dim3(kBlock), 0, s, a, (int)G);
    }
    launch_select(q, s);
}

void launch_publish(StageCounters* ctr, StageCounters* host, hipStream_t s)
{
    hipLaunchKernelGGL(publish_kernel, dim3(1), dim3(kWave), 0, s, ctr, host);
}

static unsigned select_blocks(int64_t N) { return std::min(blocks_of(N, 4 * kBlock), 512u); }

void launch_select(const SelectArgs& a, hipStream_t s)
{
    if (a.N <= kSelectOne) {
        hipLaunchKernelGGL(select_one_kernel, dim3(1), dim3(bsel::kThreads), 0, s, a);
        return;
    }
    const unsigned G = select_blocks(a.N);
    hipLaunchKernelGGL(select_range_kernel, dim3(G), dim3(kBlock), 0, s, a);
    hipLaunchKernelGGL(select_hist_kernel, dim3(G), dim3(kBlock), 0, s, a);
    hipLaunchKernelGGL(select_collect_kernel, dim3(G), dim3(kBlock), 0, s, a);
    hipLaunchKernelGGL(select_finish_kernel, dim3(1), dim3(bsel::kThreads), 0, s, a, (int)G);
    if (!a.ctr) launch_select_crowded(a, s);  // nobody reads whether they are
}

void launch_select_crowded(const SelectArgs& a, hipStream_t s)
{
    const unsigned G = select_blocks(a.N);
    for (int i = 0; i < kCrowdDigits; ++i) {
        hipLaunchKernelGGL(crowd_hist_kernel, dim3(G), dim3(kBlock), 0, s, a);
        hipLaunchKernelGGL(crowd_pick_kernel, dim3(1), dim3(kBlock), 0, s, a);
    }
    hipLaunchKernelGGL(crowd_above_kernel, dim3(G), dim3(kBlock), 0, s, a);
    hipLaunchKernelGGL(crowd_finish_kernel, dim3(1), dim3(kWave), 0, s, a, (int)G);
}

}  // namespace abcsmc
