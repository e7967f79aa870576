// sim.hip -- proposal kernel (perturb + simulate + distance + accept, one
// wave64 lane per proposal), ordered compaction of acceptances, trajectory
// kernel and the primitive test hook.
#include "dmath.h"
#include "kernels.h"
#include "propose.h"

namespace abcsmc {

namespace {

// ---------------------------------------------------------------------------
// Proposal kernel of one batch: lane p makes proposal j = base + p and
// publishes the wave's acceptance ballot for the ordered compaction.
// ---------------------------------------------------------------------------
// Waves per SIMD the register allocation aims for.  The binomial kernels take
// 161 and 167 VGPRs, so three waves per SIMD are resident whether two or three
// are asked for; two gave a slightly different schedule (10 stages of 131072
// particles x 120 days 7.92 ms, three 7.97, four, with spills, 8.30; 2^20 x 60
// without early exit 8.77, 8.76 and 8.62).
#ifndef ABCSMC_PROPOSE_WAVES
#define ABCSMC_PROPOSE_WAVES 2
#endif

template <bool kRound0, int kSampler>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(ABCSMC_PROPOSE_WAVES)))
void propose_kernel(ProposeArgs a)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) a.ctr->ts[kTsPropose] = wall_clock64();
    const uint32_t p = blockIdx.x * kBlock + threadIdx.x;
    const bool active = p < a.count;
    const uint32_t j = a.base + p;
    const lane::ProposalIn in{a.obs,    a.round,  a.max_attempts, a.eps,   a.exit_thr,          a.u_prev,
                              a.cdf,    a.n_prev, a.beta_a,       a.beta_b, a.step_is_variance, a.s_fixed, a.beta_b_real};
    lane::ProposalOut o;
    o.valid = false;
    o.acc = false;
    o.days = 0;
    o.att = 0;
    if (active) lane::propose_one<kRound0, kSampler>(a.m, in, j, o);
    if (active) {
        double* su = a.st_u + (size_t)p * kNP;
#pragma unroll
        for (int q = 0; q < kNP; ++q) su[q] = o.u[q];
        a.st_d[p] = o.d;
        a.st_sigma[p] = o.sigma;
        a.st_parent[p] = o.parent;
        a.st_att[p] = o.att;
    }
    const unsigned long long mask = __ballot(o.acc);
    const unsigned long long inv = lane::wave_sum_u64((active && !o.valid) ? 1ull : 0ull);
    const unsigned long long natt = lane::wave_sum_u64(active ? (unsigned long long)(o.att < 0 ? -o.att : o.att) : 0ull);
    const unsigned long long ndays = lane::wave_sum_u64((unsigned long long)o.days);
    if ((threadIdx.x & (kWave - 1)) == 0) {
        a.wave_mask[p / kWave] = mask;
        if (inv) atomicAdd(&a.ctr->invalid, inv);
        if (natt) atomicAdd(&a.ctr->attempts, natt);
        if (ndays) atomicAdd(&a.ctr->days, ndays);
    }
}

// The same with four lanes per proposal (64 proposals per workgroup).
template <bool kRound0, int kSampler>
__global__ __launch_bounds__(kBlock) void propose_quad_kernel(ProposeArgs a)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) a.ctr->ts[kTsPropose] = wall_clock64();
    const uint32_t p = blockIdx.x * (kBlock / 4) + threadIdx.x / 4;
    const bool active = p < a.count, lead = (threadIdx.x & 3u) == 0;
    const uint32_t j = a.base + p;
    const lane::ProposalIn in{a.obs,    a.round,  a.max_attempts, a.eps,   a.exit_thr,          a.u_prev,
                              a.cdf,    a.n_prev, a.beta_a,       a.beta_b, a.step_is_variance, a.s_fixed, a.beta_b_real};
    lane::ProposalOut o;
    o.valid = false;
    o.acc = false;
    o.days = 0;
    o.att = 0;
    if (active) {
        lane::propose_one<kRound0, kSampler, true>(a.m, in, j, o);
        if (lead) {
            double* su = a.st_u + (size_t)p * kNP;
#pragma unroll
            for (int q = 0; q < kNP; ++q) su[q] = o.u[q];
            a.st_d[p] = o.d;
            a.st_sigma[p] = o.sigma;
            a.st_parent[p] = o.parent;
            a.st_att[p] = o.att;
        }
    }
    const unsigned long long mask = lane::quad_ballot(__ballot(o.acc && lead));
    const bool count = active && lead;
    const unsigned long long inv = lane::wave_sum_u64((count && !o.valid) ? 1ull : 0ull);
    const unsigned long long natt = lane::wave_sum_u64(count ? (unsigned long long)(o.att < 0 ? -o.att : o.att) : 0ull);
    const unsigned long long ndays = lane::wave_sum_u64(count ? (unsigned long long)o.days : 0ull);
    if ((threadIdx.x & (kWave - 1)) == 0) {
        reinterpret_cast<unsigned short*>(a.wave_mask)[p / 16] = (unsigned short)mask;
        if (inv) atomicAdd(&a.ctr->invalid, inv);
        if (natt) atomicAdd(&a.ctr->attempts, natt);
        if (ndays) atomicAdd(&a.ctr->days, ndays);
    }
}

// Exclusive prefix of the per-wave acceptance counts (one workgroup).
constexpr int kScanThreads = 1024;

__global__ __launch_bounds__(kScanThreads) void compact_scan_kernel(CompactArgs a)
{
    if (threadIdx.x == 0) a.ctr->ts[kTsProposed] = wall_clock64();
    __shared__ unsigned long long part[kScanThreads];
    const uint32_t nW = (a.count + kWave - 1) / kWave;
    const uint32_t per = (nW + kScanThreads - 1) / kScanThreads;
    const uint32_t t = threadIdx.x;
    const uint32_t b0 = t * per, b1 = min(nW, b0 + per);
    unsigned long long s = 0;
    for (uint32_t w = b0; w < b1; ++w) s += __popcll(a.wave_mask[w]);
    part[t] = s;
    __syncthreads();
    // Hillis-Steele inclusive scan over 1024 partial sums
    for (int off = 1; off < kScanThreads; off <<= 1) {
        const unsigned long long v = (t >= (uint32_t)off) ? part[t - off] : 0ull;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    unsigned long long run = part[t] - s;
    for (uint32_t w = b0; w < b1; ++w) {
        a.wave_off[w] = (uint32_t)run;
        run += __popcll(a.wave_mask[w]);
    }
    if (t == kScanThreads - 1) a.ctr->accepted = a.before + part[t];
}

// Scatter the acceptances of the batch into population slots in proposal
// order; slots >= N are dropped (the stage keeps its first N acceptances).
// kScan: every workgroup adds up the ballots before its own (up to kCompactOne
// proposals 16 words a thread) instead of a scan in a launch of its own.
constexpr uint32_t kCompactOne = 1u << 18;

template <bool kScan>
__global__ __launch_bounds__(kBlock) void compact_scatter_kernel(CompactArgs a)
{
    __shared__ unsigned int part[kBlock / kWave];
    const uint32_t p = blockIdx.x * kBlock + threadIdx.x;
    const uint32_t w = p / kWave, lane = p % kWave, nW = (a.count + kWave - 1) / kWave;
    unsigned long long offset = 0;  // acceptances of the batch before wave w
    if (kScan) {
        const uint32_t first = blockIdx.x * (kBlock / kWave);
        unsigned int s = 0;
        for (uint32_t i = threadIdx.x; i < first; i += kBlock) s += (unsigned int)__popcll(a.wave_mask[i]);
#pragma unroll
        for (int off = kWave / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, kWave);
        if (lane == 0) part[threadIdx.x / kWave] = s;
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kBlock / kWave; ++i) offset += part[i];
        for (uint32_t i = first; i < w && i < nW; ++i) offset += __popcll(a.wave_mask[i]);
        if (w == nW - 1 && lane == 0) {
            a.ctr->accepted = a.before + offset + __popcll(a.wave_mask[w]);
        }
        if (p == 0) a.ctr->ts[kTsProposed] = wall_clock64();
    } else if (p < a.count) {
        offset = a.wave_off[w];
    }
    if (p >= a.count) return;
    const unsigned long long mask = a.wave_mask[w];
    if (!((mask >> lane) & 1ull)) return;
    const unsigned long long below = lane ? (mask & ((1ull << lane) - 1ull)) : 0ull;
    const unsigned long long gr = a.before + offset + (unsigned long long)__popcll(below);
    if (gr >= (unsigned long long)a.N) return;
    const double* su = a.st_u + (size_t)p * kNP;
    double* du = a.pop.u + (size_t)gr * kNP;
#pragma unroll
    for (int q = 0; q < kNP; ++q) du[q] = su[q];
    a.pop.d[gr] = a.st_d[p];
    a.pop.sigma[gr] = a.st_sigma[p];
    a.pop.parent[gr] = a.st_parent[p];
    a.pop.index[gr] = a.base + p;
    a.pop.att[gr] = a.st_att[p];
    if (gr == (unsigned long long)(a.N - 1)) a.ctr->proposals = (unsigned long long)a.base + p + 1ull;
}

template <int kSampler, bool kQuad>
__global__ __launch_bounds__(kBlock) void simulate_traj_kernel(TrajArgs a)
{
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t k = kQuad ? t / 4 : t;
    if (k >= a.n) return;
    double th[kNP];
#pragma unroll
    for (int q = 0; q < kNP; ++q) th[q] = a.theta[k * kNP + q];
    int64_t* traj = a.traj + (size_t)k * (size_t)(a.m.T + 1) * 6;
    // a bare trajectory: no observations, no distance
    int32_t days = 0;
    const uint32_t index = a.index0 + (uint32_t)k;
    if (kQuad)
        lane::simulate_distance_quad<kSampler, true>(a.m, th, nullptr, a.round, index, __builtin_inf(), traj, days);
    else
        lane::simulate_distance<kSampler, true>(a.m, th, nullptr, a.round, index, __builtin_inf(), traj, days);
}

// log1p(x) and (cos 2 pi t, sin 2 pi t) over all the arguments that the test
// hook takes: the kernels' own functions where those are defined (x in
// [-1/2, 0), t = (h + 1/2) 2^-32), the same formulas elsewhere.
__device__ __forceinline__ double hook_log1p(double x)
{
    if (x < 0.0 && x >= -0.5) return dm::log1p_neg(-x);
    if (x != x) return x;
    if (x == -1.0) return -__builtin_inf();
    if (x < -1.0) return __builtin_nan("");
    if (x >= 0.0 && x <= 0.41421356237309515) {
        const double s = x / (2.0 + x);
        const double R = dm::atanh_tail(s * s);
        return 2.0 * (s + s * R);
    }
    const double u = 1.0 + x;
    return dm::log(u) + (x - (u - 1.0)) / u;
}

__device__ __forceinline__ void hook_sincos2pi(double t, double& c, double& s)
{
    const double h = t * 0x1p32 - 0.5;
    if (h >= 0.0 && h < 0x1p32 && __builtin_floor(h) == h) {
        dm::sincos_half((uint32_t)h, c, s);
        return;
    }
    const double t4 = t * 4.0;
    const double q = __builtin_floor(t4);
    const double f = t4 - q;
    const bool fold = f > 0.5;
    double sy, pc;
    dm::sincos_octant((fold ? 1.0 - f : f) * dm::kHalfPi, sy, pc);
    const unsigned iq = (unsigned)(int)q;
    const bool swap = fold != ((iq & 1u) != 0);
    const double cc = swap ? sy : pc;
    const double ss = swap ? pc : sy;
    c = (iq + 1u) & 2u ? -cc : cc;
    s = iq & 2u ? -ss : ss;
}

__global__ __launch_bounds__(kBlock) void debug_eval_kernel(int32_t fn, int64_t n, const void* in,
                                                            void* out, double pa, int32_t pb)
{
    const int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    const double* x = (const double*)in;
    double* y = (double*)out;
    switch (fn) {
    case 0: y[i] = dm::exp(x[i]); break;
    case 1: y[i] = dm::expm1_select(x[i]); break;
    case 2: y[i] = dm::log(x[i]); break;
    case 3: y[i] = hook_log1p(x[i]); break;
    case 4: { double c, s; hook_sincos2pi(x[i], c, s); y[i] = c; } break;
    case 5: { double c, s; hook_sincos2pi(x[i], c, s); y[i] = s; } break;
    case 6: y[i] = __builtin_sqrt(x[i]); break;
    case 7: y[i] = x[2 * i] / x[2 * i + 1]; break;
    case 8: {
        const uint32_t* c = (const uint32_t*)in + 6 * i;
        dm::u4 o = dm::philox10(dm::u4{c[0], c[1], c[2], c[3]}, c[4], c[5]);
        uint32_t* r = (uint32_t*)out + 4 * i;
        r[0] = o.x; r[1] = o.y; r[2] = o.z; r[3] = o.w;
    } break;
    case 9: {
        const uint64_t w = ((const uint64_t*)in)[i];
        dm::normal_pair(w, y[2 * i], y[2 * i + 1]);
    } break;
    case 10:
    case 12: {
        const int64_t nn = ((const int64_t*)in)[3 * i];
        const double pp = ((const double*)in)[3 * i + 1];
        const uint64_t w = ((const uint64_t*)in)[3 * i + 2];
        const double r = fn == 10 ? dm::binomial((double)nn, pp, w) : dm::normal_floor((double)nn, pp, w);
        ((int64_t*)out)[i] = (int64_t)r;
    } break;
    case 13: {
        const double* ab = (const double*)in;
        y[i] = dm::beta_general(ab[0], ab[1], (uint64_t)pa, (uint32_t)i, (uint32_t)pb, 0);
    } break;
    case 11: {
        const uint64_t* w = (const uint64_t*)in + (size_t)i * pb;
        double L = 0.0;
        for (int32_t mm = 0; mm < pb; ++mm) L = L + dm::log(dm::u01(w[mm])) / (pa + (double)mm);
        y[i] = dm::exp(L);
    } break;
    case 15: y[i] = dm::exp_select(x[i]); break;
    case 16: y[i] = dm::log1p_neg(x[i]); break;
    case 17: y[i] = dm::odds(x[i]); break;
    case 18: y[i] = dm::sqrt_n(x[i]); break;
    case 19: y[i] = dm::div_n(x[2 * i], x[2 * i + 1]); break;
    default: break;
    }
}

inline unsigned grid_for(int64_t n) { return (unsigned)((n + kBlock - 1) / kBlock); }

}  // namespace

int64_t propose_first_batch_lanes()
{
    int dev = 0, cus = 0, blocks = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
        return 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&blocks, propose_kernel<false, 0>, kBlock, 0) != hipSuccess ||
        blocks < 1) {
        (void)hipGetLastError();
        return 0;
    }
    return (int64_t)cus * blocks * kBlock;
}

// Four lanes a trajectory cut its time from 455 to 220 us (120 days) as long
// as the quads' waves have a SIMD each, to 315-325 us at two waves a SIMD and
// to 430 us at three, while one lane a trajectory takes 455 us up to 65536 of
// them; at four (550 us) the quads' extra instructions show.  The floor-normal
// day has no searches to share out: 145, 220-250 and 325-335 us at one, two
// and three waves against 245-310 us.
// Rates that may be undefined go to the one-lane form.
bool propose_by_quads(int64_t n, int sampler, bool any_rates)
{
    if (any_rates && sampler == 0) return false;
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    const int64_t per_wave_round = (int64_t)cus * 4 * (kWave / 4);  // trajectories at one quad wave per SIMD
    return n <= per_wave_round * (sampler == 0 ? 3 : 2);
}

void launch_propose(const ProposeArgs& a, bool round0, hipStream_t s)
{
    const dim3 g(grid_for(a.count)), b(kBlock);
    if (propose_by_quads(a.count, a.m.sampler, a.m.any_rates)) {
        const dim3 gq(grid_for((int64_t)a.count * 4));
        if (round0) {
            if (a.m.sampler == 0) hipLaunchKernelGGL((propose_quad_kernel<true, 0>), gq, b, 0, s, a);
            else hipLaunchKernelGGL((propose_quad_kernel<true, 1>), gq, b, 0, s, a);
        } else {
            if (a.m.sampler == 0) hipLaunchKernelGGL((propose_quad_kernel<false, 0>), gq, b, 0, s, a);
            else hipLaunchKernelGGL((propose_quad_kernel<false, 1>), gq, b, 0, s, a);
        }
        return;
    }
    if (round0) {
        if (a.m.sampler == 0) hipLaunchKernelGGL((propose_kernel<true, 0>), g, b, 0, s, a);
        else hipLaunchKernelGGL((propose_kernel<true, 1>), g, b, 0, s, a);
    } else {
        if (a.m.sampler == 0) hipLaunchKernelGGL((propose_kernel<false, 0>), g, b, 0, s, a);
        else hipLaunchKernelGGL((propose_kernel<false, 1>), g, b, 0, s, a);
    }
}

void launch_compact(const CompactArgs& a, hipStream_t s)
{
    if (a.count <= kCompactOne) {
        hipLaunchKernelGGL(compact_scatter_kernel<true>, dim3(grid_for(a.count)), dim3(kBlock), 0, s, a);
        return;
    }
    hipLaunchKernelGGL(compact_scan_kernel, dim3(1), dim3(kScanThreads), 0, s, a);
    hipLaunchKernelGGL(compact_scatter_kernel<false>, dim3(grid_for(a.count)), dim3(kBlock), 0, s, a);
}

void launch_simulate_traj(const TrajArgs& a, hipStream_t s)
{
    const bool quad = propose_by_quads(a.n, a.m.sampler, a.m.any_rates);
    const dim3 g(grid_for(quad ? 4 * a.n : a.n)), b(kBlock);
    if (a.m.sampler == 0) {
        if (quad) hipLaunchKernelGGL((simulate_traj_kernel<0, true>), g, b, 0, s, a);
        else hipLaunchKernelGGL((simulate_traj_kernel<0, false>), g, b, 0, s, a);
    } else {
        if (quad) hipLaunchKernelGGL((simulate_traj_kernel<1, true>), g, b, 0, s, a);
        else hipLaunchKernelGGL((simulate_traj_kernel<1, false>), g, b, 0, s, a);
    }
}

void launch_debug_eval(int32_t fn, int64_t n, const void* in, void* out, double pa, int32_t pb,
                       hipStream_t s)
{
    if (fn == 14) {
        launch_wterm_debug(n, (const double*)in, (double*)out, s);
        return;
    }
    hipLaunchKernelGGL(debug_eval_kernel, dim3(grid_for(n)), dim3(kBlock), 0, s, fn, n, in, out, pa, pb);
}

}  // namespace abcsmc
