// batch.hip -- kernels of the batched mode.  One stage of every run is the
// fixed sequence
//   begin -> [resample x3] -> propose (persistent) -> compact scan -> scatter
//         -> [weights -> finalize -> normalise | uniform] -> select -> end
// reading the stage index and per-run state from device memory, so the host
// captures it once in a graph and replays it per stage.  Per run the
// arithmetic is exactly the single-run path's (same per-lane proposal code,
// same first-N-in-index-order cut, same integer CDF and percentile), so a run
// gives the same bits batched or alone; only the weights' summation order
// differs (1e-12).
#include "batch.h"
#include "blockselect.h"
#include "dmath.h"
#include "propose.h"
#include "wterm.h"

namespace abcsmc {

namespace {

__device__ __forceinline__ unsigned long long ld_relaxed(const unsigned long long* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ int ld_relaxed_i(const int* p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <int kThreads = kBlock, typename T>
__device__ __forceinline__ T bsum(T v, T* sh)
{
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int off = kThreads / 2; off > 0; off >>= 1) {
        if (t < off) sh[t] += sh[t + off];
        __syncthreads();
    }
    const T r = sh[0];
    __syncthreads();
    return r;
}

template <int kThreads = kBlock>
__device__ __forceinline__ double bmax(double v, double* sh)
{
    const int t = threadIdx.x;
    sh[t] = v;
    __syncthreads();
    for (int off = kThreads / 2; off > 0; off >>= 1) {
        if (t < off) sh[t] = sh[t] > sh[t + off] ? sh[t] : sh[t + off];
        __syncthreads();
    }
    const double r = sh[0];
    __syncthreads();
    return r;
}

// Exclusive scan of one value per thread (Hillis-Steele in LDS).
__device__ __forceinline__ unsigned long long bscan_excl(unsigned long long v, unsigned long long* sh)
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
    const unsigned long long r = sh[t] - v;
    __syncthreads();
    return r;
}

// ------------------------------------------------------------------ begin/end

// Stage set-up of every run: tolerance (eps^0 = +inf; eps^i = eq. 8 result of
// stage i-1), eq. 16 Beta shape, counters, and the chunk budget the
// persistent kernel aims for (N / (rate C) x margin).
__global__ __launch_bounds__(kBlock) void begin_kernel(BatchArgs a)
{
    const int stage = a.g->stage;
    for (int r = threadIdx.x; r < a.n_runs; r += kBlock) {
        const BRun& R = a.runs[r];
        BState& S = a.st[r];
        if (S.failed) continue;
        S.eps = stage == 0 ? __builtin_inf() : S.eps_next;
        if (stage == 1) S.eps1 = S.eps;
        if (stage == 0) {
            S.beta_a = 0.0;
            S.beta_b = 0;
        } else if (R.step_schedule == 1) {
            S.beta_a = R.beta_a_fixed;
            S.beta_b = R.beta_b_fixed;
        } else {
            S.beta_a = S.eps / S.eps1;
            S.beta_b = 2 * stage;
        }
        S.nxt = stage == 0 ? 0 : 1 - S.cur;
        S.issued = S.completed = S.done_acc = S.accepted = S.proposals = 0;
        S.invalid = S.attempts = S.days = S.survivors = S.fallback = S.terms = S.window_terms = 0;
        const double rate = S.rate > 0.01 ? S.rate : 0.01;
        unsigned long long lim = stage == 0
                                     ? (unsigned long long)((R.N + a.chunk - 1) / a.chunk)
                                     : (unsigned long long)__builtin_ceil((double)R.N / (rate * a.chunk) * a.g->margin);
        if (lim < 1) lim = 1;
        S.limit = lim;
    }
}

__global__ __launch_bounds__(kBlock) void end_kernel(BatchArgs a)
{
    const int stage = a.g->stage;
    for (int r = threadIdx.x; r < a.n_runs; r += kBlock) {
        const BRun& R = a.runs[r];
        BState& S = a.st[r];
        if (S.failed) continue;
        S.cur = S.nxt;
        if (stage > 0) S.rate = (double)R.N / (double)S.proposals;
        S.stages_done = (unsigned long long)stage + 1;
    }
    __syncthreads();
    if (threadIdx.x == 0) a.g->stage = stage + 1;
}

// ------------------------------------------------------------------ resample

// Same three passes as the single-run resample, over each run's block range.
__device__ __forceinline__ void res_mode(const BRun& R, bool& strict, double& wmax, unsigned long long* shu,
                                         double* shd)
{
    unsigned long long ns = 0;
    double wmx = 0.0;
    for (int b = threadIdx.x; b < R.res_nblk; b += kBlock) {
        ns += R.red_u[b];
        wmx = R.red_d[b] > wmx ? R.red_d[b] : wmx;
    }
    ns = bsum(ns, shu);
    wmx = bmax(wmx, shd);
    strict = ns > 0;
    wmax = strict ? wmx : 0.0;
}

__device__ __forceinline__ unsigned long long quantise(double d, double eps, bool strict, double wmax)
{
    const bool in = strict ? (d < eps) : (d <= eps);
    if (!in) return 0ull;
    return wmax > 0.0 ? (unsigned long long)__builtin_floor(((eps - d) / wmax) * 0x1p40) : 1ull;
}

constexpr int kRChunk = 1024, kRPer = kRChunk / kBlock;

__global__ __launch_bounds__(kBlock) void res_stats_kernel(BatchArgs a)
{
    __shared__ unsigned long long shu[kBlock];
    __shared__ double shd[kBlock];
    const int2 rb = a.res_tab[blockIdx.x];
    const BRun& R = a.runs[rb.x];
    const BState& S = a.st[rb.x];
    if (S.failed) return;
    const double* d = R.d[S.cur];
    unsigned long long ns = 0;
    double wmx = 0.0;
    for (int i = 0; i < kRPer; ++i) {
        const int k = rb.y * kRChunk + i * kBlock + threadIdx.x;
        if (k < R.N && d[k] < S.eps) {
            ++ns;
            const double w = S.eps - d[k];
            wmx = w > wmx ? w : wmx;
        }
    }
    ns = bsum(ns, shu);
    wmx = bmax(wmx, shd);
    if (threadIdx.x == 0) {
        R.red_u[rb.y] = ns;
        R.red_d[rb.y] = wmx;
    }
}

__global__ __launch_bounds__(kBlock) void res_count_kernel(BatchArgs a)
{
    __shared__ unsigned long long shu[kBlock];
    __shared__ double shd[kBlock];
    const int2 rb = a.res_tab[blockIdx.x];
    const BRun& R = a.runs[rb.x];
    const BState& S = a.st[rb.x];
    if (S.failed) return;
    bool strict;
    double wmax;
    res_mode(R, strict, wmax, shu, shd);
    const double* d = R.d[S.cur];
    const int k0 = rb.y * kRChunk + threadIdx.x * kRPer;
    unsigned long long sq = 0, sc = 0;
    for (int i = 0; i < kRPer; ++i) {
        const int k = k0 + i;
        if (k < R.N) {
            const unsigned long long q = quantise(d[k], S.eps, strict, wmax);
            sq += q;
            sc += q > 0;
        }
    }
    sq = bsum(sq, shu);
    sc = bsum(sc, shu);
    if (threadIdx.x == 0) {
        R.red_u[R.res_nblk + rb.y] = sq;
        R.red_u[2 * R.res_nblk + rb.y] = sc;
    }
}

__global__ __launch_bounds__(kBlock) void res_write_kernel(BatchArgs a)
{
    __shared__ unsigned long long shu[kBlock];
    __shared__ double shd[kBlock];
    const int2 rb = a.res_tab[blockIdx.x];
    const BRun& R = a.runs[rb.x];
    BState& S = a.st[rb.x];
    if (S.failed) return;
    bool strict;
    double wmax;
    res_mode(R, strict, wmax, shu, shd);
    const int G = R.res_nblk;
    const unsigned long long* bq = R.red_u + G;
    const unsigned long long* bc = R.red_u + 2 * G;
    unsigned long long oq = 0, oc = 0, tc = 0;
    for (int b = threadIdx.x; b < G; b += kBlock) {
        if (b < rb.y) {
            oq += bq[b];
            oc += bc[b];
        }
        tc += bc[b];
    }
    oq = bsum(oq, shu);
    oc = bsum(oc, shu);
    tc = bsum(tc, shu);
    const double* d = R.d[S.cur];
    const double* up = R.u[S.cur];
    const int k0 = rb.y * kRChunk + threadIdx.x * kRPer;
    unsigned long long q[kRPer];
    unsigned long long sq = 0, sc = 0;
    for (int i = 0; i < kRPer; ++i) {
        const int k = k0 + i;
        q[i] = k < R.N ? quantise(d[k], S.eps, strict, wmax) : 0ull;
        sq += q[i];
        sc += q[i] > 0;
    }
    unsigned long long run = oq + bscan_excl(sq, shu);
    unsigned long long col = oc + bscan_excl(sc, shu);
    for (int i = 0; i < kRPer; ++i) {
        const int k = k0 + i;
        if (k >= R.N) break;
        run += q[i];
        R.q[k] = q[i];
        R.cdf[k] = run;
        if (q[i] > 0) {
            double* c = R.cols + (size_t)col * 9;
#pragma unroll
            for (int dd = 0; dd < kNP; ++dd) c[dd] = up[(size_t)k * kNP + dd];
            c[8] = (double)q[i];
            ++col;
        }
    }
    if (rb.y == G - 1 && threadIdx.x == 0) {
        S.survivors = tc;
        S.fallback = strict ? 0ull : 1ull;
    }
}

// ------------------------------------------------------------------ propose

// Work-item scheduler of the persistent kernel (thread 0 of a workgroup).
// Pass 0 issues chunks of runs below their budget; pass 1 over-issues for
// runs still short of N acceptances, with a bound on chunks in flight (stage 0,
// where every proposal is accepted, issues exactly ceil(N / chunk) chunks).
// Every call either returns a chunk index below the run's capacity or -1, and
// a workgroup that completes a chunk always calls again, so a run short of N
// is re-examined after its last chunk in flight and every workgroup reaches
// its exit.
__device__ int pick(const BatchArgs& a, int start, bool exact, int* chunk)
{
    const int R = a.n_runs;
    for (int pass = 0; pass < (exact ? 1 : 2); ++pass) {
        for (int i = 0; i < R; ++i) {
            const int r = a.order[(start + i) % R];
            const BRun& Rr = a.runs[r];
            BState& S = a.st[r];
            if (ld_relaxed_i(&S.failed)) continue;
            const unsigned long long done = ld_relaxed(&S.done_acc);
            if (done >= (unsigned long long)Rr.N) continue;
            const unsigned long long cap = (unsigned long long)Rr.cap_chunks;
            const unsigned long long issued = ld_relaxed(&S.issued);
            if (issued >= cap) continue;
            if (pass == 0) {
                if (issued >= S.limit) continue;
            } else {
                const unsigned long long inflight = issued - ld_relaxed(&S.completed);
                const double rate = S.rate > 0.01 ? S.rate : 0.01;
                const double need = __builtin_ceil((double)(Rr.N - done) / (rate * a.chunk)) * a.g->margin;
                const unsigned long long bound = need > 1.0 ? (unsigned long long)need : 1ull;
                if (inflight >= bound) continue;
            }
            const unsigned long long k = atomicAdd(&S.issued, 1ull);
            if (k < cap) {
                *chunk = (int)k;
                return r;
            }
        }
    }
    return -1;
}

// kQuad: four lanes per proposal, kChunkQuad proposals per work item.  Three
// waves a SIMD, at the price of some spills outside the day loop, and three
// workgroups a compute unit for it: 48 runs of 2048 to 65536 particles, 6
// stages, 87.2 ms at two, 84.0 at three, 92 at four.  The quads have few items
// to hide latency with and run best without spills (12 small runs: 3.65 ms at
// two, 4.0 at three).
template <bool kRound0, bool kQuad>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kQuad ? 2 : 3))) void propose_persistent_kernel(BatchArgs a)
{
    __shared__ int s_run, s_chunk;
    __shared__ unsigned long long s_cnt[kBlock / kWave][4];
    const int stage = a.g->stage;
    int iter = 0;
    for (;;) {
        if (threadIdx.x == 0) {
            int ch = 0;
            const int r = pick(a, (int)((blockIdx.x + (unsigned)iter * gridDim.x) % (unsigned)a.n_runs), kRound0, &ch);
            s_run = r;
            s_chunk = ch;
        }
        __syncthreads();
        const int r = s_run, k = s_chunk;
        __syncthreads();
        if (r < 0) break;
        ++iter;
        const BRun& R = a.runs[r];
        const BState& S = a.st[r];
        // proposal index within the stage
        const uint32_t p = kQuad ? (uint32_t)k * kChunkQuad + threadIdx.x / 4 : (uint32_t)k * kChunkP + threadIdx.x;
        const bool lead = !kQuad || (threadIdx.x & 3u) == 0;
        const int cur = S.cur;
        const lane::ProposalIn in{R.obs,
                                  (uint32_t)stage,
                                  R.max_attempts,
                                  S.eps,
                                  (R.early_exit && !kRound0) ? (S.eps * S.eps) * (1.0 + 0x1p-48) : __builtin_inf(),
                                  R.u[cur],
                                  R.cdf,
                                  R.N,
                                  S.beta_a,
                                  S.beta_b,
                                  R.step_is_variance,
                                  -1.0,
                                  0.0};
        lane::ProposalOut o;
        if (R.m.sampler == 0) lane::propose_one<kRound0, 0, kQuad>(R.m, in, p, o);
        else lane::propose_one<kRound0, 1, kQuad>(R.m, in, p, o);
        if (lead) {
            double* su = R.st_u + (size_t)p * kNP;
#pragma unroll
            for (int q = 0; q < kNP; ++q) su[q] = o.u[q];
            R.st_d[p] = o.d;
            R.st_sigma[p] = o.sigma;
            R.st_parent[p] = o.parent;
            R.st_att[p] = o.att;
        }
        unsigned long long mask = __ballot(o.acc && lead);
        if (kQuad) mask = lane::quad_ballot(mask);
        const unsigned long long inv = lane::wave_sum_u64(lead && !o.valid ? 1ull : 0ull);
        const unsigned long long natt = lane::wave_sum_u64(lead ? (unsigned long long)(o.att < 0 ? -o.att : o.att) : 0ull);
        const unsigned long long ndays = lane::wave_sum_u64(lead ? (unsigned long long)o.days : 0ull);
        const int w = threadIdx.x / kWave;
        if ((threadIdx.x & (kWave - 1)) == 0) {
            if (kQuad) reinterpret_cast<unsigned short*>(R.wave_mask)[p / 16] = (unsigned short)mask;
            else R.wave_mask[p / kWave] = mask;
            s_cnt[w][0] = (unsigned long long)__popcll(mask);
            s_cnt[w][1] = inv;
            s_cnt[w][2] = natt;
            s_cnt[w][3] = ndays;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            unsigned long long c[4] = {0, 0, 0, 0};
            for (int ww = 0; ww < kBlock / kWave; ++ww)
                for (int f = 0; f < 4; ++f) c[f] += s_cnt[ww][f];
            BState& Sw = a.st[r];
            if (c[1]) atomicAdd(&Sw.invalid, c[1]);
            atomicAdd(&Sw.attempts, c[2]);
            atomicAdd(&Sw.days, c[3]);
            __threadfence();
            atomicAdd(&Sw.done_acc, c[0]);
            atomicAdd(&Sw.completed, 1ull);
        }
    }
}

// ------------------------------------------------------------------ compaction

// One block per run: exclusive prefix of per-wave acceptance counts over the
// issued chunks (index order) and the stage's acceptance total.
__global__ __launch_bounds__(kBlock) void bcompact_scan_kernel(BatchArgs a)
{
    __shared__ unsigned long long sh[kBlock];
    const int r = blockIdx.x;
    const BRun& R = a.runs[r];
    BState& S = a.st[r];
    if (S.failed) return;
    const unsigned long long issued = S.issued < (unsigned long long)R.cap_chunks ? S.issued : (unsigned long long)R.cap_chunks;
    const int nW = (int)issued * (a.chunk / kWave);
    const int per = (nW + kBlock - 1) / kBlock;
    const int w0 = threadIdx.x * per, w1 = min(nW, w0 + per);
    unsigned long long s = 0;
    for (int w = w0; w < w1; ++w) s += __popcll(R.wave_mask[w]);
    unsigned long long run = bscan_excl(s, sh);
    for (int w = w0; w < w1; ++w) {
        R.wave_off[w] = (uint32_t)run;
        run += __popcll(R.wave_mask[w]);
    }
    const unsigned long long tot = bsum(s, sh);
    if (threadIdx.x == 0) {
        S.accepted = tot;
        if (tot < (unsigned long long)R.N) S.failed = 1;  // out of proposals: the run keeps its last stage
    }
}

__global__ __launch_bounds__(kBlock) void bcompact_scatter_kernel(BatchArgs a)
{
    const int r = blockIdx.y, k = blockIdx.x;
    const BRun& R = a.runs[r];
    BState& S = a.st[r];
    if (S.failed) return;
    const unsigned long long issued = S.issued < (unsigned long long)R.cap_chunks ? S.issued : (unsigned long long)R.cap_chunks;
    const uint32_t p = (uint32_t)k * kBlock + threadIdx.x;
    if ((unsigned long long)p >= issued * (unsigned)a.chunk) return;
    const unsigned long long mask = R.wave_mask[p / kWave];
    const uint32_t lane = p % kWave;
    if (!((mask >> lane) & 1ull)) return;
    const unsigned long long below = lane ? (mask & ((1ull << lane) - 1ull)) : 0ull;
    const unsigned long long gr = R.wave_off[p / kWave] + (unsigned long long)__popcll(below);
    if (gr >= (unsigned long long)R.N) return;
    const int nx = S.nxt;
    const double* su = R.st_u + (size_t)p * kNP;
    double* du = R.u[nx] + (size_t)gr * kNP;
#pragma unroll
    for (int q = 0; q < kNP; ++q) du[q] = su[q];
    R.d[nx][gr] = R.st_d[p];
    R.sigma[nx][gr] = R.st_sigma[p];
    R.parent[nx][gr] = R.st_parent[p];
    R.index[nx][gr] = p;
    R.att[nx][gr] = R.st_att[p];
    if (gr == (unsigned long long)(R.N - 1)) S.proposals = (unsigned long long)p + 1ull;
}

// ------------------------------------------------------------------ weights

// Weight pass, per run as the single-run one (smc.hip, wterm.h): column
// statistics choose the run's sort code; columns sorted by code, rows by
// (sigma half-octave descending, code); gathered with what the pair test
// needs; every wave evaluates the columns one of its rows needs.  Every
// run has a region of the key arrays of its own, a power of two long, and all
// regions are sorted by the same launches (one sort of all runs' keys took 580
// us of a stage for 1.2 million particles in 48 runs, 200 us so; 72 and
// 24 at 21500 in 12).
using wterm::sigma_half_octave;

constexpr int kDimThreads = 1024;

// One block per run: sum, sum of squares, minimum and maximum of each
// coordinate over the run's columns (thread t: coordinate t % 8).
__global__ __launch_bounds__(kDimThreads) void bwgeom_kernel(BatchArgs a)
{
    __shared__ double sh[4][kDimThreads];
    const BRun& R = a.runs[blockIdx.x];
    BState& S = a.st[blockIdx.x];
    if (S.failed) return;
    const int M = (int)S.survivors, t = threadIdx.x, d = t & 7;
    double s1 = 0.0, s2 = 0.0, mn = __builtin_inf(), mx = -__builtin_inf();
#pragma unroll 4
    for (int k = t / 8; k < M; k += kDimThreads / 8) {
        const double v = R.cols[(size_t)k * 9 + d];
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
    for (int off = kDimThreads / 2; off >= 8; off >>= 1) {
        if (t < off) {
            sh[0][t] += sh[0][t + off];
            sh[1][t] += sh[1][t + off];
            sh[2][t] = sh[2][t] < sh[2][t + off] ? sh[2][t] : sh[2][t + off];
            sh[3][t] = sh[3][t] > sh[3][t + off] ? sh[3][t] : sh[3][t + off];
        }
        __syncthreads();
    }
    wterm::make_geom(sh[0], sh[1], sh[2], sh[3], (double)M, &S.geom);
}

// grid.y 0: columns, 1: rows.
__global__ __launch_bounds__(kBlock) void bkeys_kernel(BatchArgs a)
{
    __shared__ uint32_t cells[kNP * kBlock];
    const size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= a.spans.n[0]) return;  // each thread uses its own LDS column only
    const bool row = blockIdx.y != 0;
    unsigned long long* keys = row ? a.rowkeys : a.colkeys;
    const int r = a.key_run[i / kKeyUnit];
    const BRun& R = a.runs[r];
    const BState& S = a.st[r];
    const unsigned long long k = (unsigned long long)((int)i - R.koff);
    if (k >= (unsigned long long)R.N) {
        keys[i] = ~0ull;
        return;
    }
    if (S.failed || (!row && k >= (unsigned long long)S.survivors)) {
        keys[i] = (0xFFFFFFFFull << 20) | k;
        return;
    }
    const WeightGeom& g = S.geom;
    const int nx = S.nxt;
    double u[kNP];
#pragma unroll
    for (int d = 0; d < kNP; ++d) {
        u[d] = row ? R.u[nx][k * kNP + d] : R.cols[k * 9 + d];
        cells[d * kBlock + threadIdx.x] = wterm::cell20(u[d], g.lo[d], g.inv[d]);
    }
    uint32_t key = wterm::morton32(g, cells + threadIdx.x, kBlock);
    if (row) {
        const double sj = R.sigma[nx][k];
        // half-octaves in descending order: the widest windows are dispatched first
        key = ((127u - (uint32_t)sigma_half_octave(sj)) << 25) | (key >> 7);
        const int32_t par = R.parent[nx][k];
        const bool ok = par >= 0 && par < R.N;
        a.rwin[R.off + k] = wterm::window_radius(u, sj, ok ? R.u[1 - nx] + (size_t)par * kNP : u, ok ? (double)R.q[par] : 0.0,
                                         (double)R.cdf[R.N - 1]);
    }
    keys[i] = ((unsigned long long)key << 20) | k;
}

// grid = finalize table (run, row block): the block's slots of the run's
// sorted columns and rows.
__global__ __launch_bounds__(kWeightRows) void bgather_kernel(BatchArgs a)
{
    const int2 fb = a.fin_tab[blockIdx.x];
    const BRun& R = a.runs[fb.x];
    const BState& S = a.st[fb.x];
    if (S.failed) return;
    const size_t i = (size_t)fb.y * kWeightRows + threadIdx.x;
    if (blockIdx.y == 0) {
        const size_t M = (size_t)S.survivors;
        if (i < weight_col_pad(M))
            wterm::gather_column(R.sc, S.geom, i, i < M, R.cols + (i < M ? (size_t)(a.colkeys[R.koff + i] & 0xFFFFFull) : 0) * 9);
    } else {
        const bool real = i < (size_t)R.N;
        const size_t j = real ? (size_t)(a.rowkeys[R.koff + i] & 0xFFFFFull) : 0;
        wterm::gather_row(R.sr, S.geom, i, real, R.u[S.nxt] + j * kNP, R.sigma[S.nxt][j], a.rwin[R.off + j], a.ex);
    }
}

// grid = weight table (run, row block, chunk): chunk c of the run's column
// tiles, sorted rows.  (Five waves a SIMD as in the single run: 10% of the
// launch against four; with 28 instructions a term for 31 a run of 48 fits with
// 2048 to 65536 particles went from 94.6 to 90.7 ms.)
__global__ __launch_bounds__(kWeightRows) __attribute__((amdgpu_waves_per_eu(5))) void bweights_kernel(BatchArgs a, int entry0)
{
    __shared__ double T[wterm::kTab];
    const int4 wb = a.w_tab[entry0 + blockIdx.x];
    const BRun& R = a.runs[wb.x];
    const BState& S = a.st[wb.x];
    if (S.failed) return;  // uniform across the block
    const int M = (int)S.survivors, tiles = (M + kColTile - 1) / kColTile;
    const int t0 = (int)(((long long)tiles * wb.z) / R.wchunks), t1 = (int)(((long long)tiles * (wb.z + 1)) / R.wchunks);
    const int rr = wb.y * kWeightRows + threadIdx.x;
    double* out = R.wpart + (size_t)wb.w * R.N;
    const int w = threadIdx.x / kWave, lane = threadIdx.x & (kWave - 1);
    const int group = __builtin_amdgcn_readfirstlane(wb.y * (kWeightRows / kWave) + w);
    if (t0 >= t1) {
        if (rr < R.N) out[rr] = 0.0;
        if (lane == 0) R.wcounts[(size_t)wb.z * (R.sr.pad / kWave) + group] = make_uint2(0, 0);
        return;
    }
    uint32_t listed = 0, window = 0;
    double total = 0.0;
    const unsigned long long first = wterm::near_tiles(R.sr, R.sc, group, lane, t0, t1);
    if (__syncthreads_or(first != 0 || t1 - t0 > kWave)) {
        wterm::load_table(T, a.wtab);
        __syncthreads();
        total = wterm::row_sum(R.sr, R.sc, group, lane, t0, t1, M, first, T, a.ex, listed, window);
    }
    if (rr < R.N) out[rr] = total;
    if (lane == 0) R.wcounts[(size_t)wb.z * (R.sr.pad / kWave) + group] = make_uint2(listed, window);
}

// Sum of row rr over the first `slots` slots, in the chunks' order.
__device__ __forceinline__ double slot_total(const BRun& R, int rr, int slots)
{
    double L = 0.0;
    for (int c = 0; c < slots; ++c) L += R.wpart[(size_t)c * R.N + rr];
    return L;
}

// After pass `pass`, the sums of the runs that need another one to slot 0.
__global__ __launch_bounds__(kWeightRows) void bfold_kernel(BatchArgs a, int pass)
{
    const int2 fb = a.fin_tab[blockIdx.x];
    const BRun& R = a.runs[fb.x];
    if (a.st[fb.x].failed || weight_pass(R.wchunks - 1, R.wslots) <= pass) return;
    const int rr = fb.y * kWeightRows + threadIdx.x;
    if (rr < R.N) R.wpart[rr] = slot_total(R, rr, R.wslots);
}

__global__ __launch_bounds__(kWeightRows) void bfinalize_kernel(BatchArgs a)
{
    const int2 fb = a.fin_tab[blockIdx.x];
    const BRun& R = a.runs[fb.x];
    const BState& S = a.st[fb.x];
    if (S.failed) return;
    const int rr = fb.y * kWeightRows + threadIdx.x;
    const int group = rr / kWave, lane = threadIdx.x & (kWave - 1);
    if (group * kWave < R.N) {
        unsigned long long listed = 0, window = 0;
        for (int c = lane; c < R.wchunks; c += kWave) {
            const uint2 n = R.wcounts[(size_t)c * (R.sr.pad / kWave) + group];
            listed += n.x;
            window += n.y;
        }
        listed = wterm::wave_sum_u64(listed);
        window = wterm::wave_sum_u64(window);
        if (lane == 0 && listed) {
            atomicAdd(&a.st[fb.x].terms, listed * (unsigned long long)min(kWave, R.N - group * kWave));
            atomicAdd(&a.st[fb.x].window_terms, window);
        }
    }
    if (rr >= R.N) return;
    const double L = slot_total(R, rr, weight_slot(R.wchunks - 1, R.wslots) + 1);
    const size_t j = (size_t)(a.rowkeys[R.koff + rr] & 0xFFFFFull);
    R.logw[S.nxt][j] = 8.0 * dm::log(R.sigma[S.nxt][j]) - dm::log(L);
}

constexpr int kNormThreads = 1024;

// One block per run: W = softmax(l), ESS.  Bound by the longest run's passes
// through one block: 214 us with 256 threads, 54 with 1024 (N = 65536).
__global__ __launch_bounds__(kNormThreads) void bnormalise_kernel(BatchArgs a, int uniform)
{
    __shared__ double sh[kNormThreads];
    const BRun& R = a.runs[blockIdx.x];
    BState& S = a.st[blockIdx.x];
    if (S.failed) return;
    const int nx = S.nxt, N = R.N;
    double* l = R.logw[nx];
    double* W = R.W[nx];
    if (uniform) {
        for (int j = threadIdx.x; j < N; j += kNormThreads) {
            W[j] = 1.0 / (double)N;
            l[j] = 0.0;
        }
        if (threadIdx.x == 0) S.ess = (double)N;
        return;
    }
    double mx = -__builtin_inf();
#pragma unroll 4
    for (int j = threadIdx.x; j < N; j += kNormThreads) mx = l[j] > mx ? l[j] : mx;
    mx = bmax<kNormThreads>(mx, sh);
    double s = 0.0;
#pragma unroll 4
    for (int j = threadIdx.x; j < N; j += kNormThreads) {
        const double e = dm::exp(l[j] - mx);
        W[j] = e;
        s += e;
    }
    s = bsum<kNormThreads>(s, sh);
    double s2 = 0.0;
#pragma unroll 4
    for (int j = threadIdx.x; j < N; j += kNormThreads) {
        const double w = W[j] / s;
        W[j] = w;
        s2 += w * w;
    }
    s2 = bsum<kNormThreads>(s2, sh);
    if (threadIdx.x == 0) S.ess = 1.0 / s2;
}

// ------------------------------------------------------------------ select

// One block per run: eq. 8 type-7 percentile.
__global__ __launch_bounds__(bsel::kThreads) void bselect_kernel(BatchArgs a)
{
    __shared__ bsel::Shared sh;
    const BRun& R = a.runs[blockIdx.x];
    BState& S = a.st[blockIdx.x];
    if (S.failed) return;  // uniform across the block
    const double res = bsel::quantile7(bsel::FromMemory{R.d[S.nxt], R.N}, R.N, R.surv_ratio, sh);
    if (threadIdx.x == 0) S.eps_next = res;
}

}  // namespace

void batch_launch_stage(const BatchArgs& a, bool stage0, hipStream_t s)
{
    const dim3 b(kBlock);
    hipLaunchKernelGGL(begin_kernel, dim3(1), b, 0, s, a);
    if (!stage0) {
        hipLaunchKernelGGL(res_stats_kernel, dim3(a.n_res_blocks), b, 0, s, a);
        hipLaunchKernelGGL(res_count_kernel, dim3(a.n_res_blocks), b, 0, s, a);
        hipLaunchKernelGGL(res_write_kernel, dim3(a.n_res_blocks), b, 0, s, a);
        if (a.chunk == kChunkQuad)
            hipLaunchKernelGGL((propose_persistent_kernel<false, true>), dim3(a.propose_blocks), b, 0, s, a);
        else
            hipLaunchKernelGGL((propose_persistent_kernel<false, false>), dim3(a.propose_blocks), b, 0, s, a);
    } else {
        if (a.chunk == kChunkQuad)
            hipLaunchKernelGGL((propose_persistent_kernel<true, true>), dim3(a.propose_blocks), b, 0, s, a);
        else
            hipLaunchKernelGGL((propose_persistent_kernel<true, false>), dim3(a.propose_blocks), b, 0, s, a);
    }
    hipLaunchKernelGGL(bcompact_scan_kernel, dim3(a.n_runs), b, 0, s, a);
    hipLaunchKernelGGL(bcompact_scatter_kernel, dim3(a.max_cap_blocks, a.n_runs), b, 0, s, a);
    if (!stage0) {
        hipLaunchKernelGGL(bwgeom_kernel, dim3(a.n_runs), dim3(kDimThreads), 0, s, a);
        hipLaunchKernelGGL(bkeys_kernel, dim3((unsigned)((a.spans.n[0] + kBlock - 1) / kBlock), 2), b, 0, s, a);
        launch_sort_spans(a.colkeys, a.rowkeys, a.spans, s);
        const dim3 bw(kWeightRows);
        hipLaunchKernelGGL(bgather_kernel, dim3(a.n_fin_blocks, 2), bw, 0, s, a);
        for (int p = 0; p < kMaxWPasses && a.w_pass[p + 1] > a.w_pass[p]; ++p) {
            if (p > 0) hipLaunchKernelGGL(bfold_kernel, dim3(a.n_fin_blocks), bw, 0, s, a, p - 1);
            hipLaunchKernelGGL(bweights_kernel, dim3(a.w_pass[p + 1] - a.w_pass[p]), bw, 0, s, a, a.w_pass[p]);
        }
        hipLaunchKernelGGL(bfinalize_kernel, dim3(a.n_fin_blocks), bw, 0, s, a);
    }
    hipLaunchKernelGGL(bnormalise_kernel, dim3(a.n_runs), dim3(kNormThreads), 0, s, a, stage0 ? 1 : 0);
    hipLaunchKernelGGL(bselect_kernel, dim3(a.n_runs), dim3(bsel::kThreads), 0, s, a);
    hipLaunchKernelGGL(end_kernel, dim3(1), b, 0, s, a);
}

}  // namespace abcsmc
