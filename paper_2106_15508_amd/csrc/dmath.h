// dmath.h -- device-side numerics of the ABC-SMC hot path (gfx950, wave64).
//
// Every random quantity of the method is a transformed uniform (the
// reparameterisation of §III-A).  The transforms below are written so that
// each result is a fixed sequence of IEEE-754 binary64 operations
// (+ - * / sqrt fma floor rint ldexp frexp, all exact or correctly rounded on
// CDNA4 and built with -ffp-contract=off), which makes the draws, and hence
// the trajectories, reproducible bit for bit on any conforming machine:
//
//   u01(w)        ((w >> 12) + 1/2) * 2^-52                      in (0,1), exact
//   exp(x)        k = rint(x log2 e), r = (x - k ln2_hi) - k ln2_lo (fma),
//                 2^k * sum_{i<=13} r^i / i!   (Horner, fma); 0 below e^-708
//   log(x)        x = f 2^e, f in [1/sqrt2, sqrt2), s = (f-1)/(f+1),
//                 2 atanh(s) by its series to s^23, plus e ln2
//   log1p(x)      atanh series of x/(2+x) near 0, else log(1+x) + rounding error
//   expm1(x)      Taylor to x^14 for |x| <= ln2/2, else exp(x) - 1
//   cos/sin 2pi t quadrant and octant folding, Taylor to y^18 / y^17
//   normal pair   Box-Muller on the two 32-bit halves of one word
//   Bin(n,p)      sequential-search inversion when n min(p,1-p) < 10,
//                 else floor(m + 1/2 + sqrt(m(1-q)) z), clamped
//   Beta(a,b)     b integer: exp( sum_{m<b} log(U_m) / (a+m) )
//
// Counts are carried as doubles holding exact integers (< 2^53).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace abcsmc {
namespace dm {

// ---------------------------------------------------------------- Philox

struct u4 {
    uint32_t x, y, z, w;
};

// x ^ y ^ z in one instruction
__device__ __forceinline__ uint32_t xor3(uint32_t x, uint32_t y, uint32_t z)
{
    return (uint32_t)__builtin_amdgcn_bitop3_b32((int)x, (int)y, (int)z, 0x96);
}

__device__ __forceinline__ u4 philox10(u4 c, uint32_t k0, uint32_t k1)
{
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        const uint64_t m0 = (uint64_t)0xD2511F53u * c.x;
        const uint64_t m1 = (uint64_t)0xCD9E8D57u * c.z;
        u4 n;
        n.x = xor3((uint32_t)(m1 >> 32), c.y, k0);
        n.y = (uint32_t)m1;
        n.z = xor3((uint32_t)(m0 >> 32), c.w, k1);
        n.w = (uint32_t)m0;
        c = n;
        k0 += 0x9E3779B9u;
        k1 += 0xBB67AE85u;
    }
    return c;
}

enum : uint32_t { kPrior = 1, kPerturb = 2, kSim = 3 };

// The two 64-bit words of block `blk` of stream (index, round, purpose, sub).
struct w2 {
    uint64_t a, b;
};

__device__ __forceinline__ w2 block_words(uint64_t seed, uint32_t index, uint32_t round,
                                          uint32_t purpose, uint32_t sub, uint32_t blk)
{
    u4 c{index, round, (purpose << 24) | (sub & 0xFFFFFFu), blk};
    u4 o = philox10(c, (uint32_t)seed, (uint32_t)(seed >> 32));
    return w2{((uint64_t)o.y << 32) | o.x, ((uint64_t)o.w << 32) | o.z};
}

// ((w >> 12) + 1/2) 2^-52: the 52 bits as the mantissa of a number in [1, 2),
// less 1 - 2^-53 (exact: the result has 53 bits)
__device__ __forceinline__ double u01(uint64_t w)
{
    return __longlong_as_double((long long)((w >> 12) | 0x3FF0000000000000ull)) - 0x1.fffffffffffffp-1;
}

// ---------------------------------------------------------------- constants

constexpr double kLn2Hi = 0x1.62e42feep-1;           // ln 2 to 32 significant bits
constexpr double kLn2Lo = 0x1.a39ef35793c76p-33;     // ln 2 - kLn2Hi, rounded
constexpr double kLog2e = 1.4426950408889634;        // 1 / ln 2
constexpr double kSqrt1_2 = 0.70710678118654757;     // 1 / sqrt 2
constexpr double kHalfPi = 1.5707963267948966;       // pi / 2
constexpr double kExpHi = 709.782712893384;          // above: +inf
constexpr double kExpLo = -708.0;                    // below: 0

// 1/i! (i = 0..18), each the double nearest the exact value.
constexpr double kF0 = 1.0, kF1 = 1.0, kF2 = 1.0 / 2.0, kF3 = 1.0 / 6.0, kF4 = 1.0 / 24.0,
                 kF5 = 1.0 / 120.0, kF6 = 1.0 / 720.0, kF7 = 1.0 / 5040.0, kF8 = 1.0 / 40320.0,
                 kF9 = 1.0 / 362880.0, kF10 = 1.0 / 3628800.0, kF11 = 1.0 / 39916800.0,
                 kF12 = 1.0 / 479001600.0, kF13 = 1.0 / 6227020800.0,
                 kF14 = 1.0 / 87178291200.0, kF15 = 1.0 / 1307674368000.0,
                 kF16 = 1.0 / 20922789888000.0, kF17 = 1.0 / 355687428096000.0,
                 kF18 = 1.0 / 6402373705728000.0;

// ---------------------------------------------------------------- division, square root

// a / b and sqrt(x), correctly rounded, for operands and results that stay
// well inside the normal range (x > 0): Newton-Raphson steps on the hardware's
// reciprocal and Markstein's correction of the quotient by its residual;
// Goldschmidt's coupled iteration for x^(1/2) and x^(-1/2) / 2 and two residual
// corrections.  Without the scaling, range tests and fix-up that any operand
// needs they take a third of the instructions.  Callers name the range.
__device__ __forceinline__ double div_n(double a, double b)
{
    double y = __builtin_amdgcn_rcp(b);
    y = __builtin_fma(y, __builtin_fma(-b, y, 1.0), y);
    y = __builtin_fma(y, __builtin_fma(-b, y, 1.0), y);
    const double q = a * y;
    return __builtin_fma(__builtin_fma(-b, q, a), y, q);
}

__device__ __forceinline__ double sqrt_n(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    double g = x * y;
    double h = 0.5 * y;
    const double r = __builtin_fma(-h, g, 0.5);
    g = __builtin_fma(g, r, g);
    h = __builtin_fma(h, r, h);
    g = __builtin_fma(__builtin_fma(-g, g, x), h, g);
    return __builtin_fma(__builtin_fma(-g, g, x), h, g);
}

// ---------------------------------------------------------------- exp family

// e^r for |r| <= ln2/2 + tiny: degree-13 Taylor polynomial.
__device__ __forceinline__ double exp_poly(double r)
{
    double p = kF13;
    p = __builtin_fma(p, r, kF12);
    p = __builtin_fma(p, r, kF11);
    p = __builtin_fma(p, r, kF10);
    p = __builtin_fma(p, r, kF9);
    p = __builtin_fma(p, r, kF8);
    p = __builtin_fma(p, r, kF7);
    p = __builtin_fma(p, r, kF6);
    p = __builtin_fma(p, r, kF5);
    p = __builtin_fma(p, r, kF4);
    p = __builtin_fma(p, r, kF3);
    p = __builtin_fma(p, r, kF2);
    p = __builtin_fma(p, r, kF1);
    p = __builtin_fma(p, r, kF0);
    return p;
}

// k as an int32, saturating: v_cvt_i32_f64 clamps an input outside the int32
// range (NaN: 0) by its definition, where a C++ conversion would be
// undefined.  One instruction, as the plain conversion compiles to.
__device__ __forceinline__ int cvt_i32_sat(double x)
{
    int r;
    asm("v_cvt_i32_f64 %0, %1" : "=v"(r) : "v"(x));
    return r;
}

// exp(x) for x already known to lie in [kExpLo, kExpHi].
__device__ __forceinline__ double exp_core(double x)
{
    const double k = __builtin_rint(x * kLog2e);
    const double t = x - k * kLn2Hi;
    const double r = __builtin_fma(-k, kLn2Lo, t);
    return __builtin_ldexp(exp_poly(r), (int)k);
}

__device__ __forceinline__ double exp(double x)
{
    if (x != x) return x;
    if (x > kExpHi) return __builtin_inf();
    if (x < kExpLo) return 0.0;
    return exp_core(x);
}

// exp(x) for any x, the range tests by selection (no branch).
__device__ __forceinline__ double exp_select(double x)
{
    const double k = __builtin_rint(x * kLog2e);
    const double t = x - k * kLn2Hi;
    const double r = __builtin_fma(-k, kLn2Lo, t);
    double e = __builtin_ldexp(exp_poly(r), cvt_i32_sat(k));
    e = x > kExpHi ? __builtin_inf() : e;
    return x < kExpLo ? 0.0 : e;
}

// expm1(x) for any x without a branch: the Taylor polynomial of the small
// arguments and the exponential's polynomial share their coefficients
// 1/13! .. 1/2!, so one Horner chain runs on x or on the reduced argument
// (its first step adds 0 or 1/14!), the same operations as the two branches.
__device__ __forceinline__ double expm1_select(double x)
{
    const bool small = __builtin_fabs(x) <= 0.34657359027997264;
    const double k = __builtin_rint(x * kLog2e);
    const double t = x - k * kLn2Hi;
    const double r = __builtin_fma(-k, kLn2Lo, t);
    const double v = small ? x : r;
    double p = __builtin_fma(small ? kF14 : 0.0, v, kF13);
    p = __builtin_fma(p, v, kF12);
    p = __builtin_fma(p, v, kF11);
    p = __builtin_fma(p, v, kF10);
    p = __builtin_fma(p, v, kF9);
    p = __builtin_fma(p, v, kF8);
    p = __builtin_fma(p, v, kF7);
    p = __builtin_fma(p, v, kF6);
    p = __builtin_fma(p, v, kF5);
    p = __builtin_fma(p, v, kF4);
    p = __builtin_fma(p, v, kF3);
    p = __builtin_fma(p, v, kF2);
    double e = __builtin_fma(__builtin_fma(p, v, kF1), v, kF0);
    e = __builtin_ldexp(e, cvt_i32_sat(k));
    e = x > kExpHi ? __builtin_inf() : e;
    e = x < kExpLo ? 0.0 : e;
    return small ? __builtin_fma(x * x, p, x) : e - 1.0;
}

// ---------------------------------------------------------------- log family

// s^2/3 + s^4/5 + ... + s^22/23 evaluated at z = s^2 (times z).
__device__ __forceinline__ double atanh_tail(double z)
{
    double q = 1.0 / 23.0;
    q = __builtin_fma(q, z, 1.0 / 21.0);
    q = __builtin_fma(q, z, 1.0 / 19.0);
    q = __builtin_fma(q, z, 1.0 / 17.0);
    q = __builtin_fma(q, z, 1.0 / 15.0);
    q = __builtin_fma(q, z, 1.0 / 13.0);
    q = __builtin_fma(q, z, 1.0 / 11.0);
    q = __builtin_fma(q, z, 1.0 / 9.0);
    q = __builtin_fma(q, z, 1.0 / 7.0);
    q = __builtin_fma(q, z, 1.0 / 5.0);
    q = __builtin_fma(q, z, 1.0 / 3.0);
    return z * q;
}

// log(x) for finite x > 0 (NaN stays NaN); the division's operands lie in
// [-0.3, 0.42] and [1.7, 2.42], exact zero included.
__device__ __forceinline__ double log_pos(double x)
{
    int e;
    double f = __builtin_frexp(x, &e);
    if (f < kSqrt1_2) {
        f = f * 2.0;
        e = e - 1;
    }
    const double a = f - 1.0;
    const double s = div_n(a, 2.0 + a);
    const double R = atanh_tail(s * s);
    const double lf = 2.0 * (s + s * R);
    const double de = (double)e;
    return de * kLn2Hi + (de * kLn2Lo + lf);
}

__device__ __forceinline__ double log(double x)
{
    if (x != x) return x;
    if (x < 0.0) return __builtin_nan("");
    if (x == 0.0) return -__builtin_inf();
    if (x == __builtin_inf()) return x;
    return log_pos(x);
}

// ---------------------------------------------------------------- trig / normals

// sin y and cos y for 0 <= y <= pi/4 (Taylor).
__device__ __forceinline__ void sincos_octant(double y, double& sy, double& pc)
{
    const double ny2 = -(y * y);
    double ps = kF17;
    ps = __builtin_fma(ps, ny2, kF15);
    ps = __builtin_fma(ps, ny2, kF13);
    ps = __builtin_fma(ps, ny2, kF11);
    ps = __builtin_fma(ps, ny2, kF9);
    ps = __builtin_fma(ps, ny2, kF7);
    ps = __builtin_fma(ps, ny2, kF5);
    ps = __builtin_fma(ps, ny2, kF3);
    ps = __builtin_fma(ps, ny2, kF1);
    sy = y * ps;
    pc = kF18;
    pc = __builtin_fma(pc, ny2, kF16);
    pc = __builtin_fma(pc, ny2, kF14);
    pc = __builtin_fma(pc, ny2, kF12);
    pc = __builtin_fma(pc, ny2, kF10);
    pc = __builtin_fma(pc, ny2, kF8);
    pc = __builtin_fma(pc, ny2, kF6);
    pc = __builtin_fma(pc, ny2, kF4);
    pc = __builtin_fma(pc, ny2, kF2);
    pc = __builtin_fma(pc, ny2, kF0);
}

__device__ __forceinline__ double flip_sign(double v, uint32_t bit31)
{
    return __longlong_as_double(__double_as_longlong(v) ^ (long long)((uint64_t)bit31 << 32));
}

// (cos 2 pi t, sin 2 pi t) for t = (h + 1/2) 2^-32.  The quadrant q and the
// octant fold are taken from h's bits: f = 4 t - q is (r + 1/2) 2^-30 for the low
// 30 bits r, above 1/2 where bit 29 is set, and 1 - f there has the complement
// of r; all of these are exact.
__device__ __forceinline__ void sincos_half(uint32_t h, double& c, double& s)
{
    const uint32_t fold = (uint32_t)((int32_t)(h << 2) >> 31);  // all ones where bit 29 is set
    const double g = ((double)((h ^ fold) & 0x1FFFFFFFu) + 0.5) * 0x1p-30;
    double sy, pc;
    sincos_octant(g * kHalfPi, sy, pc);
    const bool swap = ((h ^ (h >> 1)) & 0x20000000u) != 0;  // fold, or an odd quadrant
    const double cc = swap ? sy : pc;
    const double ss = swap ? pc : sy;
    c = flip_sign(cc, (h ^ (h << 1)) & 0x80000000u);  // quadrants 1 and 2
    s = flip_sign(ss, h & 0x80000000u);               // quadrants 2 and 3
}

// Box-Muller pair from one word: u1 = low half, u2 = high half; lu = log u1.
__device__ __forceinline__ double u1_of(uint64_t w) { return ((double)(uint32_t)w + 0.5) * 0x1p-32; }

__device__ __forceinline__ void normal_from_log(double lu, uint64_t w, double& z0, double& z1)
{
    const double rho = sqrt_n(-2.0 * lu);  // of [2^-32, 45]
    double c, s;
    sincos_half((uint32_t)(w >> 32), c, s);
    z0 = rho * c;
    z1 = rho * s;
}

__device__ __forceinline__ void normal_pair(uint64_t w, double& z0, double& z1)
{
    normal_from_log(log_pos(u1_of(w)), w, z0, z1);
}

// Cosine half of the pair only (the floor-normal and gamma samplers).
__device__ __forceinline__ double normal_one(uint64_t w)
{
    double z0, z1;
    normal_pair(w, z0, z1);
    return z0;
}

// ---------------------------------------------------------------- samplers

// Word w of stream (index, round, purpose, sub): half w % 2 of block w / 2.
__device__ __forceinline__ uint64_t word_at(uint64_t seed, uint32_t index, uint32_t round, uint32_t purpose,
                                            uint32_t sub, uint32_t w)
{
    const w2 b = block_words(seed, index, round, purpose, sub, w >> 1);
    return (w & 1u) ? b.b : b.a;
}

// Gamma(k) by Marsaglia & Tsang (ACM TOMS 2000): k' = k (k + 1 if k < 1),
// d = k' - 1/3, c = 1/sqrt(9 d); iteration m: z = first Box-Muller normal of
// word w0 + 2m, U from word w0 + 2m + 1, v = (1 + c z)^3, accept d v when
// v > 0 and log U < z^2/2 + d - d v + d log v; d after 32 rejections.  For
// k < 1 the result is scaled by U^(1/k), U from word w0 + 64.
__device__ __forceinline__ double gamma_mt(double k, uint64_t seed, uint32_t index, uint32_t round, uint32_t sub,
                                           uint32_t w0)
{
    const double kk = k < 1.0 ? k + 1.0 : k;
    const double d = kk - 1.0 / 3.0;
    const double c = 1.0 / __builtin_sqrt(9.0 * d);
    double g = d;
    for (uint32_t m = 0; m < 32; ++m) {
        const double z = normal_one(word_at(seed, index, round, kPerturb, sub, w0 + 2 * m));
        const double t = 1.0 + c * z;
        if (!(t > 0.0)) continue;
        const double v = t * t * t;
        const double U = u01(word_at(seed, index, round, kPerturb, sub, w0 + 2 * m + 1));
        if (log(U) < 0.5 * (z * z) + d - d * v + d * log(v)) {
            g = d * v;
            break;
        }
    }
    if (k < 1.0) g = g * exp(log(u01(word_at(seed, index, round, kPerturb, sub, w0 + 64))) / k);
    return g;
}

// Beta(a, b), real shapes: X / (X + Y), X ~ Gamma(a) from words 5.., Y ~
// Gamma(b) from words 70.. of the attempt's PERTURB stream; 0 if both vanish.
__device__ __forceinline__ double beta_general(double a, double b, uint64_t seed, uint32_t index, uint32_t round,
                                               uint32_t sub)
{
    const double X = gamma_mt(a, seed, index, round, sub, 5);
    const double Y = gamma_mt(b, seed, index, round, sub, 70);
    const double s = X + Y;
    return s > 0.0 ? X / s : 0.0;
}

constexpr double kTSwitch = 10.0;
constexpr int kBinvCap = 128;
constexpr int kBinvStep = 4;  // search steps between two looks at the wave

// 1/j, j = 1..kBinvCap, rounded to nearest at compile time.  The search's
// step counter is wave-uniform, so an entry is a scalar load; kBinvStep more
// entries let the loop request the next group while it works on this one.
struct RecipTab {
    double v[kBinvCap + kBinvStep];
    constexpr RecipTab() : v{}
    {
        for (int j = 0; j < kBinvCap + kBinvStep; ++j) v[j] = 1.0 / (double)(j + 1);
    }
};
__device__ constexpr RecipTab kRecip{};

// A success probability as the samplers use it: q = min(p, 1 - p) (0 for
// p <= 0 or p = 1; NaN stays NaN) and whether the draw counts failures.
struct Prob {
    double q;
    bool flip;
};

__device__ __forceinline__ Prob make_prob(double p)
{
    Prob r;
    r.flip = p > 0.5;
    r.q = r.flip ? 1.0 - p : p;
    r.q = p <= 0.0 ? 0.0 : r.q;
    return r;
}

// log1p(-q) and q / (1 - q) for 0 < q <= 1/2: what the inversion of Bin(n, q)
// needs of q.  (Quotients of a subnormal q may round differently from IEEE
// division; there n log1p(-q) vanishes against 1 and the draw is 0.)
__device__ __forceinline__ double log1p_neg(double q)
{
    if (-q >= kSqrt1_2 - 1.0) {
        const double s = div_n(-q, 2.0 - q);
        const double R = atanh_tail(s * s);
        return 2.0 * (s + s * R);
    }
    const double u = 1.0 - q;
    return log_pos(u) + div_n(-q - (u - 1.0), u);
}

__device__ __forceinline__ double odds(double q) { return div_n(q, 1.0 - q); }

// Bin(n, q) by sequential search, 0 < n q < kTSwitch, l1 = log1p(-q),
// r = q / (1 - q): the number of k with u > F(k), k < min(n, kBinvCap), where
// f(0) = exp(n l1), f(k + 1) = f(k) ((n - k) r) (1/(k + 1)) and F sums f.  F
// never falls, so the draw is a count and lanes that are done need no mask:
// the wave takes kBinvStep steps, then looks whether any lane still searches.
// (Past k = n the terms are zeros: F stays.)  The factors of f(k + 1) do not
// depend on f, and the next reciprocals are requested a group ahead: what is
// left of a step's latency is one product and one sum, where a loop that
// stopped lane by lane waited for its scalar load in every step.
__device__ __forceinline__ double binomial_search(double n, double l1, double r, uint64_t wu)
{
    const double u = u01(wu);
    double f = exp_core(n * l1);  // n l1 in [-14, 0]
    double F = f;
    double nk = n;
    unsigned count = 0;
    double c[kBinvStep];
#pragma unroll
    for (int s = 0; s < kBinvStep; ++s) c[s] = kRecip.v[s];
    for (int it = 0; it < kBinvCap; it += kBinvStep) {
        double d[kBinvStep];
#pragma unroll
        for (int s = 0; s < kBinvStep; ++s) d[s] = kRecip.v[it + kBinvStep + s];
#pragma unroll
        for (int s = 0; s < kBinvStep; ++s) {
            count += u > F ? 1u : 0u;
            f = f * ((nk * r) * c[s]);
            F = F + f;
            nk = nk - 1.0;
        }
        if (__ballot(u > F) == 0ull) break;
#pragma unroll
        for (int s = 0; s < kBinvStep; ++s) c[s] = d[s];
    }
    const double x = (double)count;
    return x < n ? x : n;
}

// Bin(n, p) with p as q (Prob) from a uniform word and a standard normal; n
// is an exact integer >= 0 held in a double.  n q < kTSwitch searches, the
// rest rounds the normal.  The normal branch is taken by nearly every wave
// and runs unmasked; inv() supplies (l1, r) where a lane searches.
// kAnyRates: n or p may be NaN.  An empty compartment and a probability of 0
// then draw 0 whatever the other one is, and the rest stays NaN.
template <bool kAnyRates, class Inv>
__device__ __forceinline__ double binomial_draw(double n, const Prob& p, double z, uint64_t wu, Inv inv)
{
    const double m = n * p.q;
    const bool small = m < kTSwitch;           // false for NaN
    const double sd = sqrt_n(m * (1.0 - p.q));  // used for m >= kTSwitch: in [2, 2^27]
    const double y = (m + 0.5) + sd * z;        // finite, or NaN where m is
    // clamped to [0, n]; the product of y and 0 keeps the NaN that max drops
    double x = __builtin_fma(y, 0.0, __builtin_fmax(__builtin_fmin(__builtin_floor(y), n), 0.0));
    x = small ? 0.0 : x;
    if (small && m > 0.0) {
        double l1, r;
        inv(l1, r);
        x = binomial_search(n, l1, r, wu);
    }
    if (kAnyRates && m != m && (n <= 0.0 || p.q <= 0.0)) x = 0.0;
    return p.flip ? n - x : x;
}

// Bin(n, p) from one word: its uniform and its cosine deviate.
__device__ __forceinline__ double binomial(double n, double p, uint64_t w)
{
    const Prob P = make_prob(p);
    return binomial_draw<true>(n, P, normal_one(w), w, [&](double& l1, double& r) {
        l1 = log1p_neg(P.q);
        r = odds(P.q);
    });
}

// floor(N(h, sqrt h)) clamped to [0, n] (the paper's own transition sampler).
__device__ __forceinline__ double normal_floor_z(double n, double h, double z)
{
    double x = __builtin_floor(h + __builtin_sqrt(h) * z);
    x = x < 0.0 ? 0.0 : x;
    x = x > n ? n : x;
    return (n <= 0.0 || !(h > 0.0)) ? 0.0 : x;
}

__device__ __forceinline__ double normal_floor(double n, double h, uint64_t w)
{
    return normal_floor_z(n, h, normal_one(w));
}

}  // namespace dm
}  // namespace abcsmc
