// propose.h -- per-lane device code of one proposal: perturbation (or prior
// draw), forward simulation, distance and acceptance.  Shared by the plain
// batch kernel and the persistent batched-runs kernel.
#pragma once

#include "dmath.h"
#include "kernels.h"

namespace abcsmc {
namespace lane {

// ---------------------------------------------------------------------------
// One trajectory of the epidemic model (§II-B, eqs. 3-5) with the running
// Euclidean distance to the observed (A, R, D) (§II-C).
//   init   Ru = 0, I = floor(kappa A0) (capped so S >= 0), S = P - (A0+R0+D0+I)
//   day t  g = alpha0 + alpha / (1 + (A+R+D)^n)          (eq. 4)
//          transitions in the order of h (eq. 5): S->I, I->A, A->R, A->D, I->Ru,
//          each drawn from what is left of its source compartment
//   dist   sum over days 1..T of dA^2, dR^2, dD^2 in that order; sqrt at the end
// Returns +inf as soon as the partial sum exceeds exit_thr (the final
// distance would exceed eps).  Stream (index, round, SIM, t) of day t: draw k
// takes its inversion uniform from word k and its normal deviate from the
// Box-Muller pairs of words 5 (draws 0, 1), 6 (draws 2, 3) and 7 (draw 4);
// the floor-normal sampler uses the cosine deviate of word k.
// ---------------------------------------------------------------------------
// A wave's lanes disagree in nearly every day about some range test or about
// which draws search and which round a normal, so the day is written without
// branches except the searches: all three Box-Muller pairs are formed (on
// average some lane of a wave needs each of them on 99% of the days), range
// tests select, and a search counts instead of masking lanes off.  Bound by
// instruction issue; against the branching form the proposal kernel went from
// 636 to 377 us a batch at 25000-30000 proposals x 97 days (one wave a SIMD)
// and from 1171 to 872 us at 170000 x 120.
// With kSplit the three series' sums of squares also go to split[0..2]
// (no early exit; the surrogate's training targets); the returned distance
// is the same as without.
// With kTraj and series != null the trajectory's (A, R, D) go to
// series[(3 t + c) * sstride] (day t = 0..T) instead of traj.
// kAnyRates: rates may be undefined (Model::any_rates, a loop of its own: the
// draws' tests for it in the one loop cost 1-4% of the launches).
template <int kSampler, bool kTraj, bool kSplit, bool kAnyRates>
__device__ __forceinline__ double simulate_days(const Model& m, const double* th, const double* __restrict__ obs,
                                                uint32_t round, uint32_t index, double exit_thr, int64_t* traj,
                                                int32_t& days, double* split, double* series, int64_t sstride)
{
    const double alpha0 = th[0], alpha_c = th[1], n_exp = th[2], beta = th[3];
    const double gamma = th[4], delta = th[5], eta = th[6], kappa = th[7];
    double A = m.A0, R = m.R0, D = m.D0;
    double I = __builtin_floor(kappa * A);
    const double room = m.P - (A + R + D);
    if (I > room) I = room;
    if (I < 0.0) I = 0.0;
    double S = m.P - (A + R + D + I);
    double Ru = 0.0;
    // the four fixed transition probabilities and what their inversions need
    dm::Prob pr[4];
    double l1[4], od[4];
    if (kSampler == 0) {
        const double x[4] = {-gamma, -beta, -delta, -(beta * eta)};  // I->A, A->R, A->D, I->Ru
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            pr[k] = dm::make_prob(-dm::expm1_select(x[k]));
            l1[k] = dm::log1p_neg(pr[k].q);
            od[k] = dm::odds(pr[k].q);
        }
    }
    if (kTraj) {
        if (series) {
            series[0] = A;
            series[sstride] = R;
            series[2 * sstride] = D;
        } else {
            traj[0] = (int64_t)S; traj[1] = (int64_t)I; traj[2] = (int64_t)A;
            traj[3] = (int64_t)R; traj[4] = (int64_t)D; traj[5] = (int64_t)Ru;
        }
    }
    double acc = 0.0;
    for (int32_t t = 0; t < m.T; ++t) {
        const dm::w2 b0 = dm::block_words(m.seed, index, round, dm::kSim, (uint32_t)t, 0);
        const dm::w2 b1 = dm::block_words(m.seed, index, round, dm::kSim, (uint32_t)t, 1);
        const dm::w2 b2 = dm::block_words(m.seed, index, round, dm::kSim, (uint32_t)t, 2);
        const double C = A + R + D;
        double pw = dm::exp_select(n_exp * dm::log_pos(C));
        pw = C == 0.0 ? (n_exp == 0.0 ? 1.0 : 0.0) : pw;
        const double g = alpha0 + alpha_c / (1.0 + pw);
        const double rate = (g * I) * m.invP;
        double n1, n2, n3, n4, n5;
        if (kSampler == 0) {
            const dm::w2 b3 = dm::block_words(m.seed, index, round, dm::kSim, (uint32_t)t, 3);
            double z0, z1, z2, z3, z4, z5;
            dm::normal_pair(b2.b, z0, z1);
            dm::normal_pair(b3.a, z2, z3);
            dm::normal_pair(b3.b, z4, z5);
            const dm::Prob pSI = dm::make_prob(-dm::expm1_select(-rate));
            auto fixed = [&](int k) {
                return [&, k](double& a, double& r) {
                    a = l1[k];
                    r = od[k];
                };
            };
            n1 = dm::binomial_draw<kAnyRates>(S, pSI, z0, b0.a, [&](double& a, double& r) {
                a = dm::log1p_neg(pSI.q);
                r = dm::odds(pSI.q);
            });
            n2 = dm::binomial_draw<kAnyRates>(I, pr[0], z1, b0.b, fixed(0));
            n3 = dm::binomial_draw<kAnyRates>(A, pr[1], z2, b1.a, fixed(1));
            n4 = dm::binomial_draw<kAnyRates>(A - n3, pr[2], z3, b1.b, fixed(2));
            n5 = dm::binomial_draw<kAnyRates>(I - n2, pr[3], z4, b2.a, fixed(3));
        } else {
            n1 = dm::normal_floor(S, rate * S, b0.a);
            n2 = dm::normal_floor(I, gamma * I, b0.b);
            n3 = dm::normal_floor(A, beta * A, b1.a);
            n4 = dm::normal_floor(A - n3, delta * A, b1.b);
            n5 = dm::normal_floor(I - n2, (beta * eta) * I, b2.a);
        }
        S = S - n1;
        I = I + n1 - n2 - n5;
        A = A + n2 - n3 - n4;
        R = R + n3;
        D = D + n4;
        Ru = Ru + n5;
        if (kTraj) {
            if (series) {
                double* col = series + (size_t)(3 * (t + 1)) * sstride;
                col[0] = A;
                col[sstride] = R;
                col[2 * sstride] = D;
            } else {
                int64_t* row = traj + (size_t)(t + 1) * 6;
                row[0] = (int64_t)S; row[1] = (int64_t)I; row[2] = (int64_t)A;
                row[3] = (int64_t)R; row[4] = (int64_t)D; row[5] = (int64_t)Ru;
            }
        }
        if (kSplit) {
            const double* o = obs + (size_t)(t + 1) * 3;
            const double dA = A - o[0];
            const double dR = R - o[1];
            const double dD = D - o[2];
            split[0] = split[0] + dA * dA;
            split[1] = split[1] + dR * dR;
            split[2] = split[2] + dD * dD;
            acc = acc + dA * dA;
            acc = acc + dR * dR;
            acc = acc + dD * dD;
        } else if (!kTraj) {
            const double* o = obs + (size_t)(t + 1) * 3;
            const double dA = A - o[0];
            const double dR = R - o[1];
            const double dD = D - o[2];
            acc = acc + dA * dA;
            acc = acc + dR * dR;
            acc = acc + dD * dD;
            if (acc > exit_thr) {
                days = t + 1;
                return __builtin_inf();
            }
        }
    }
    days = m.T;
    return __builtin_sqrt(acc);
}

template <int kSampler, bool kTraj, bool kSplit = false>
__device__ __forceinline__ double simulate_distance(const Model& m, const double* th,
                                                    const double* __restrict__ obs, uint32_t round,
                                                    uint32_t index, double exit_thr, int64_t* traj,
                                                    int32_t& days, double* split = nullptr,
                                                    double* series = nullptr, int64_t sstride = 0)
{
    if (kSampler == 0 && m.any_rates)
        return simulate_days<kSampler, kTraj, kSplit, true>(m, th, obs, round, index, exit_thr, traj, days, split,
                                                            series, sstride);
    return simulate_days<kSampler, kTraj, kSplit, false>(m, th, obs, round, index, exit_thr, traj, days, split,
                                                         series, sstride);
}

// ---------------------------------------------------------------------------
// Four lanes per trajectory.  A small batch leaves most of the chip idle and
// takes as long as one wave's instruction stream, so its parallelism is spent
// inside the trajectory: lane q of a quad makes Philox block q of the day,
// lanes 1-3 one Box-Muller pair each while lane 0 takes log C, lanes 0-2 draw
// S->I, I->A and A->R at once, then lanes 3 and 0 draw A->D and I->Ru.  The
// state is kept by all four lanes; values change hands by quad permutes.
// Every value is the one-lane form's, bit for bit.  (Ordinary rates only.)
// ---------------------------------------------------------------------------
template <int kCtrl>
__device__ __forceinline__ uint32_t quad_perm(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, kCtrl, 0xF, 0xF, true);
}
template <int kCtrl>
__device__ __forceinline__ uint64_t quad_perm(uint64_t v)
{
    return ((uint64_t)quad_perm<kCtrl>((uint32_t)(v >> 32)) << 32) | quad_perm<kCtrl>((uint32_t)v);
}
template <int kCtrl>
__device__ __forceinline__ double quad_perm(double v)
{
    return __longlong_as_double((long long)quad_perm<kCtrl>((uint64_t)__double_as_longlong(v)));
}
// the value lane k of the quad holds, in all four lanes
template <int k, class T>
__device__ __forceinline__ T quad_lane(T v)
{
    return quad_perm<k * 0x55>(v);
}

// every fourth bit of a wave's ballot, closed up to the wave's 16 quads
__device__ __forceinline__ unsigned long long quad_ballot(unsigned long long m)
{
    m &= 0x1111111111111111ull;
    m = (m | (m >> 3)) & 0x0303030303030303ull;
    m = (m | (m >> 6)) & 0x000F000F000F000Full;
    m = (m | (m >> 12)) & 0x000000FF000000FFull;
    return (m | (m >> 24)) & 0xFFFFull;
}

template <int kSampler, bool kTraj, bool kSplit = false>
__device__ __forceinline__ double simulate_distance_quad(const Model& m, const double* th,
                                                         const double* __restrict__ obs, uint32_t round,
                                                         uint32_t index, double exit_thr, int64_t* traj,
                                                         int32_t& days, double* split = nullptr,
                                                         double* series = nullptr, int64_t sstride = 0)
{
    const uint32_t q = threadIdx.x & 3u;
    const double alpha0 = th[0], alpha_c = th[1], n_exp = th[2], beta = th[3];
    const double gamma = th[4], delta = th[5], eta = th[6], kappa = th[7];
    double A = m.A0, R = m.R0, D = m.D0;
    double I = __builtin_floor(kappa * A);
    const double room = m.P - (A + R + D);
    if (I > room) I = room;
    if (I < 0.0) I = 0.0;
    double S = m.P - (A + R + D + I);
    double Ru = 0.0;
    // the lane's fixed transition probability: I->Ru, I->A, A->R, A->D
    dm::Prob own{};
    double l1 = 0.0, od = 0.0;
    if (kSampler == 0) {
        own = dm::make_prob(-dm::expm1_select(q == 0 ? -(beta * eta) : q == 1 ? -gamma : q == 2 ? -beta : -delta));
        l1 = dm::log1p_neg(own.q);
        od = dm::odds(own.q);
    }
    auto record = [&](int32_t t) {
        if (!kTraj || q != 0) return;
        if (series) {
            double* col = series + (size_t)(3 * t) * sstride;
            col[0] = A;
            col[sstride] = R;
            col[2 * sstride] = D;
        } else {
            int64_t* row = traj + (size_t)t * 6;
            row[0] = (int64_t)S; row[1] = (int64_t)I; row[2] = (int64_t)A;
            row[3] = (int64_t)R; row[4] = (int64_t)D; row[5] = (int64_t)Ru;
        }
    };
    record(0);
    double acc = 0.0;
    for (int32_t t = 0; t < m.T; ++t) {
        const dm::w2 b = dm::block_words(m.seed, index, round, dm::kSim, (uint32_t)t, q);
        const double C = A + R + D;
        // the lane's Box-Muller word and, in lane 0 (binomial: words 5, 6, 7 in lanes
        // 2, 3, 1) or 1 (floor-normal: words 0-3 in lanes 0-3), the logarithm of C
        // (permutes stand outside every selection: all four lanes take part)
        uint64_t wn;
        if (kSampler == 0) {
            const uint64_t w7 = quad_lane<3>(b.b);
            wn = q == 1 ? w7 : q == 2 ? b.b : b.a;
        } else {
            const uint64_t w1 = quad_lane<0>(b.b), w2 = quad_lane<1>(b.a), w3 = quad_lane<1>(b.b);
            wn = q == 0 ? b.a : q == 1 ? w1 : q == 2 ? w2 : w3;
        }
        double u1 = dm::u1_of(wn);
        if (kSampler == 0) u1 = q == 0 ? C : u1;
        const double lg = dm::log_pos(u1);
        double zc, zs, logC;
        dm::normal_from_log(lg, wn, zc, zs);
        double z4 = 0.0;
        if (kSampler == 0) {
            logC = quad_lane<0>(lg);
        } else {
            const uint64_t w4 = quad_lane<2>(b.a);
            const double l4 = dm::log_pos(q == 1 ? C : dm::u1_of(w4));
            double unused;
            dm::normal_from_log(quad_lane<0>(l4), w4, z4, unused);
            logC = quad_lane<1>(l4);
        }
        double pw = dm::exp_select(n_exp * logC);
        pw = C == 0.0 ? (n_exp == 0.0 ? 1.0 : 0.0) : pw;
        const double g = alpha0 + alpha_c / (1.0 + pw);
        const double rate = (g * I) * m.invP;
        double n1, n2, n3, n4, n5;
        if (kSampler == 0) {
            const dm::Prob pSI = dm::make_prob(-dm::expm1_select(-rate));
            // S->I, I->A, A->R in lanes 0, 1, 2 (lane 3: a draw from nothing)
            const dm::Prob pa{q == 0 ? pSI.q : own.q, q == 0 ? pSI.flip : own.flip};
            const double na = q == 0 ? S : q == 1 ? I : q == 2 ? A : 0.0;
            const double zs2 = quad_lane<2>(zs), zc23 = quad_perm<0x32>(zc);  // lane 0 <- 2, lane 2 <- 3
            const uint64_t ub = quad_lane<0>(b.b), ua = quad_lane<1>(b.a);
            const double x = dm::binomial_draw<false>(na, pa, q == 1 ? zs2 : zc23, q == 0 ? b.a : q == 1 ? ub : ua,
                                               [&](double& a, double& r) {
                                                   a = l1;
                                                   r = od;
                                                   if (q == 0) {
                                                       a = dm::log1p_neg(pSI.q);
                                                       r = dm::odds(pSI.q);
                                                   }
                                               });
            n1 = quad_lane<0>(x);
            n2 = quad_lane<1>(x);
            n3 = quad_lane<2>(x);
            // A->D in lane 3, I->Ru in lane 0
            const double nb = q == 3 ? A - n3 : q == 0 ? I - n2 : 0.0;
            const double zc1 = quad_lane<1>(zc);
            const uint64_t u3 = quad_lane<1>(b.b), u4 = quad_lane<2>(b.a);
            const double y = dm::binomial_draw<false>(nb, own, q == 0 ? zc1 : zs, q == 0 ? u4 : u3,
                                               [&](double& a, double& r) {
                                                   a = l1;
                                                   r = od;
                                               });
            n4 = quad_lane<3>(y);
            n5 = quad_lane<0>(y);
        } else {
            const double x = dm::normal_floor_z(q == 0 ? S : q == 1 ? I : A, q == 0 ? rate * S : q == 1 ? gamma * I : beta * A,
                                                zc);
            n1 = quad_lane<0>(x);
            n2 = quad_lane<1>(x);
            n3 = quad_lane<2>(x);
            const double y = dm::normal_floor_z(q == 3 ? A - n3 : I - n2, q == 3 ? delta * A : (beta * eta) * I,
                                                q == 3 ? zc : z4);
            n4 = quad_lane<3>(y);
            n5 = quad_lane<0>(y);
        }
        S = S - n1;
        I = I + n1 - n2 - n5;
        A = A + n2 - n3 - n4;
        R = R + n3;
        D = D + n4;
        Ru = Ru + n5;
        record(t + 1);
        if (kSplit || !kTraj) {
            const double* o = obs + (size_t)(t + 1) * 3;
            const double dA = A - o[0];
            const double dR = R - o[1];
            const double dD = D - o[2];
            if (kSplit) {
                split[0] = split[0] + dA * dA;
                split[1] = split[1] + dR * dR;
                split[2] = split[2] + dD * dD;
            }
            acc = acc + dA * dA;
            acc = acc + dR * dR;
            acc = acc + dD * dD;
            if (!kSplit && acc > exit_thr) {
                days = t + 1;
                return __builtin_inf();
            }
        }
    }
    days = m.T;
    return __builtin_sqrt(acc);
}

// First k with cdf[k] > r (cdf non-decreasing, cdf[n-1] > r).
__device__ __forceinline__ int32_t upper_bound_u64(const uint64_t* __restrict__ cdf, int32_t n, uint64_t r)
{
    int32_t lo = 0, hi = n - 1;
    while (lo < hi) {
        const int32_t mid = lo + ((hi - lo) >> 1);
        if (cdf[mid] > r) hi = mid;
        else lo = mid + 1;
    }
    return lo;
}

__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}


// Inputs of one proposal beyond the model.
struct ProposalIn {
    const double* obs;       // (T+1) x 3
    uint32_t round;
    int32_t max_attempts;
    double eps;              // accept iff d <= eps
    double exit_thr;         // early-exit threshold on the partial sum of squares
    const double* u_prev;    // previous population, n_prev x 8
    const uint64_t* cdf;     // its integer CDF
    int32_t n_prev;
    double beta_a;
    int32_t beta_b;
    int32_t step_is_variance;
    double s_fixed;          // >= 0: step size of every proposal (MCMC variant); < 0: Beta draw
    double beta_b_real;      // > 0: real Beta shape b (general sampler; beta_b unused)
};

struct ProposalOut {
    double u[kNP];
    double sigma;
    int32_t parent;
    int32_t att;             // attempts used; -max_attempts for a void proposal
    double d;
    bool valid;
    bool acc;
    int32_t days;            // days simulated
};

// ---------------------------------------------------------------------------
// One proposal j.  Stage 0: u ~ U(0,1)^8 (prior of eq. 2 in the unit cube).
// Stage i >= 1, attempt a = 1, 2, ...: parent k ~ Categorical(q) (eq. 11) from
// word 0; s ~ Beta(a_i, b_i) (eq. 16) from words 5..5+b-1; z ~ N(0, I_8) from
// the Box-Muller pairs of words 1..4; u = u_k + sigma z (eq. 17); stop at the
// first u inside [0,1]^8.  Then simulate, distance, accept iff d <= eps.
// ---------------------------------------------------------------------------
// Attempt att (1, 2, ...) of proposal j in stage >= 1: true when u lies in the cube.
__device__ __forceinline__ bool attempt(const Model& m, const ProposalIn& a, uint32_t j, int32_t att, uint64_t Q,
                                        double* u, double& sigma, int32_t& parent)
{
    const uint32_t sub = (uint32_t)(att - 1);
    const dm::w2 b0 = dm::block_words(m.seed, j, a.round, dm::kPerturb, sub, 0);
    const dm::w2 b1 = dm::block_words(m.seed, j, a.round, dm::kPerturb, sub, 1);
    const dm::w2 b2 = dm::block_words(m.seed, j, a.round, dm::kPerturb, sub, 2);
    const uint64_t r = __umul64hi(b0.a, Q);
    const int32_t k = upper_bound_u64(a.cdf, a.n_prev, r);
    // Beta(a, b), b integer: exp( sum_m log U_m / (a + m) )
    double L = 0.0;
    uint64_t hold = 0;
    const int32_t nb = (a.s_fixed >= 0.0 || a.beta_b_real > 0.0) ? 0 : a.beta_b;
    for (int32_t mm = 0; mm < nb; ++mm) {
        uint64_t w;
        if (mm == 0) {
            w = b2.b;
        } else if (mm & 1) {
            const dm::w2 nb = dm::block_words(m.seed, j, a.round, dm::kPerturb, sub, 2u + (uint32_t)((mm + 1) >> 1));
            w = nb.a;
            hold = nb.b;
        } else {
            w = hold;
        }
        L = L + dm::log_pos(dm::u01(w)) / (a.beta_a + (double)mm);
    }
    const double s = a.s_fixed >= 0.0       ? a.s_fixed
                     : a.beta_b_real > 0.0 ? dm::beta_general(a.beta_a, a.beta_b_real, m.seed, j, a.round, sub)
                                           : dm::exp(L);
    double sg = a.step_is_variance ? __builtin_sqrt(s) : s;
    if (sg < 1e-8) sg = 1e-8;
    double z[kNP];
    dm::normal_pair(b0.b, z[0], z[1]);
    dm::normal_pair(b1.a, z[2], z[3]);
    dm::normal_pair(b1.b, z[4], z[5]);
    dm::normal_pair(b2.a, z[6], z[7]);
    const double* up = a.u_prev + (size_t)k * kNP;
    bool inside = true;
#pragma unroll
    for (int d = 0; d < kNP; ++d) {
        const double v = up[d] + sg * z[d];
        u[d] = v;
        inside = inside && (v >= 0.0 && v <= 1.0);
    }
    sigma = sg;
    parent = k;
    return inside;
}

// Stage-0 prior draw (kRound0) or the perturbation attempts of stage >= 1:
// fills o.u, o.sigma, o.parent, o.att and o.valid.
template <bool kRound0>
__device__ __forceinline__ void perturb_one(const Model& m, const ProposalIn& a, uint32_t j, ProposalOut& o)
{
    double* u = o.u;
    double sigma = 0.0;
    int32_t parent = -1;
    int32_t att = 1;
    bool valid = true;
    {
        if (kRound0) {
#pragma unroll
            for (uint32_t blk = 0; blk < 4; ++blk) {
                const dm::w2 w = dm::block_words(m.seed, j, 0, dm::kPrior, 0, blk);
                u[2 * blk] = dm::u01(w.a);
                u[2 * blk + 1] = dm::u01(w.b);
            }
        } else {
            const uint64_t Q = a.cdf[a.n_prev - 1];
            valid = false;
            for (att = 1; att <= a.max_attempts; ++att) {
                if (attempt(m, a, j, att, Q, u, sigma, parent)) {
                    valid = true;
                    break;
                }
            }
            if (!valid) att = -a.max_attempts;
        }
    }
    o.sigma = sigma;
    o.parent = parent;
    o.att = att;
    o.valid = valid;
}

// perturb_one by a quad: its lanes try four attempts at a time and the first
// one inside the cube is kept (none: the last of max_attempts, as one lane
// after another would leave it).
template <bool kRound0>
__device__ __forceinline__ void perturb_quad(const Model& m, const ProposalIn& a, uint32_t j, ProposalOut& o)
{
    if (kRound0) {
        perturb_one<true>(m, a, j, o);
        return;
    }
    const uint32_t q = threadIdx.x & 3u, quad0 = threadIdx.x & (kWave - 4);
    const uint64_t Q = a.cdf[a.n_prev - 1];
    o.valid = false;
    int32_t base = 0;
    for (;; base += 4) {
        const int32_t att = base + 1 + (int32_t)q;
        const bool in = att <= a.max_attempts && attempt(m, a, j, att, Q, o.u, o.sigma, o.parent);
        const uint32_t hit = (uint32_t)(__ballot(in) >> quad0) & 15u;
        uint32_t src;
        if (hit) {
            src = (uint32_t)__builtin_ctz(hit);
            o.valid = true;
            o.att = base + 1 + (int32_t)src;
        } else if (base + 4 >= a.max_attempts) {
            src = (uint32_t)(a.max_attempts - 1 - base);
            o.att = -a.max_attempts;
        } else {
            continue;
        }
        const int from = (int)(quad0 + src);
#pragma unroll
        for (int d = 0; d < kNP; ++d) o.u[d] = __shfl(o.u[d], from, kWave);
        o.sigma = __shfl(o.sigma, from, kWave);
        o.parent = __shfl(o.parent, from, kWave);
        return;
    }
}

// kQuad: the four lanes of a quad make the proposal together (and all hold
// the result).
template <bool kRound0, int kSampler, bool kQuad = false>
__device__ __forceinline__ void propose_one(const Model& m, const ProposalIn& a, uint32_t j, ProposalOut& o)
{
    if (kQuad) perturb_quad<kRound0>(m, a, j, o);
    else perturb_one<kRound0>(m, a, j, o);
    double d = __builtin_inf();
    bool acc = false;
    int32_t days = 0;
    if (o.valid) {
        double th[kNP];
#pragma unroll
        for (int q = 0; q < kNP; ++q) th[q] = m.lo[q] + o.u[q] * m.width[q];
        d = kQuad ? simulate_distance_quad<kSampler, false>(m, th, a.obs, a.round, j, a.exit_thr, nullptr, days)
                  : simulate_distance<kSampler, false>(m, th, a.obs, a.round, j, a.exit_thr, nullptr, days);
        acc = d <= a.eps;
    }
    o.d = d;
    o.acc = acc;
    o.days = days;
}

}  // namespace lane
}  // namespace abcsmc
