// wterm.h -- one importance-weight term q_k exp(-|u_j - u_k|^2 / (2 sigma_j^2))
// with a table-driven exponential, the sort code, the pair test and the
// per-wave column loop (device code shared by the single-run and batched weight kernels).
#pragma once

#include "dmath.h"
#include "kernels.h"

namespace abcsmc {
namespace wterm {

// Scalar-column form used by the weight kernels.  Columns (u_k[8] and q_k, in
// two arrays: a 64-byte line holds one column's u) are the same for every
// lane of a wave, so they are read through wave-uniform pointers in the
// constant address space (scalar loads into SGPRs, no LDS staging).  The
// exponential uses a 1024-entry table of 2^(i/1024):
//   t = D c_j with c_j = -1024 / (2 sigma_j^2 ln 2)  (the exponent in units
//   of ln2/1024), k = rint(t), r = (t - k) ln2/1024, |r| <= 3.4e-4,
//   exp = 2^(k >> 10) 2^((k & 1023)/1024) (1 + r + r^2/2 + r^3/6)
// (truncation r^4/24 < 6e-16 relative); the weight q_k enters by one fma
// into the running sum.  A term is added where the column lies in the row's
// window (D <= R_j^2), which bounds t: k is the low word of t + 1.5 2^52, and
// the power of two enters by one integer addition to the high word of the
// table entry (whose own i << 10 is taken off beforehand; entries carry 2^64,
// the sum's scale, so that exponents down to the widest window's -710 stay
// normal).  Far columns of a wave's list may give anything and are left out
// by the execution mask.  28 vector instructions (25 FP64) where rint,
// conversion, ldexp and the column's number from LDS took 31.
constexpr int kTabBits = 10;
constexpr int kTab = 1 << kTabBits;

typedef const __attribute__((address_space(4))) double* const_col_ptr;  // constant address space

struct Col {
    double u[kNP];
    double q;
};

__device__ __forceinline__ Col load_col(const_col_ptr cu, const_col_ptr cq, uint32_t k)
{
    typedef const __attribute__((address_space(4))) char* const_byte_ptr;
    Col c;
    const_col_ptr p = (const_col_ptr)((const_byte_ptr)cu + k * (uint32_t)(kNP * sizeof(double)));
#pragma unroll
    for (int d = 0; d < kNP; ++d) c.u[d] = p[d];
    c.q = *(const_col_ptr)((const_byte_ptr)cq + k * (uint32_t)sizeof(double));
    return c;
}

// |u_j - u_k|^2
__device__ __forceinline__ double dist2(const double* uj, const Col& c)
{
    double D = 0.0;
#pragma unroll
    for (int d = 0; d < kNP; ++d) {
        const double df = uj[d] - c.u[d];
        D = __builtin_fma(df, df, D);
    }
    return D;
}

// exp of the term (without q) times 2^64: with f = t - k in [-1/2, 1/2] and
// L = ln2/1024, e^(f L) = 1 + f (L + f (L^2/2 + f L^3/6)); ex[0..2] = L, L^2/2,
// L^3/6 (kernel arguments: SGPRs).  For |D c_j| < 1086 * 1024, where the scaled
// result is still a normal number (the widest window reaches 1.0499e6).
__device__ __forceinline__ double term_exp(double D, double cj, const double* T, const double* ex, double ex1)
{
    constexpr double kMagic = 0x1.8p52;
    const double v = __builtin_fma(D, cj, kMagic);
    const double f = __builtin_fma(D, cj, -(v - kMagic));
    const uint32_t k = (uint32_t)__double_as_longlong(v);
    double p = __builtin_fma(f, ex[2], ex1);
    p = __builtin_fma(p, f, ex[0]);
    p = __builtin_fma(p, f, 1.0);
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    u32x2 e = __builtin_bit_cast(u32x2, T[k & (kTab - 1)]);
    e.y += k << (20 - kTabBits);
    return __builtin_bit_cast(double, e) * p;
}

// sum += q x in the lanes of mask.
__device__ __forceinline__ void add_where(unsigned long long mask, double q, double x, double& sum)
{
    unsigned long long all;
    asm("s_and_saveexec_b64 %1, %2\n\tv_fma_f64 %0, %3, %4, %0\n\ts_mov_b64 exec, %1"
        : "+v"(sum), "=&s"(all)
        : "s"(mask), "s"(q), "v"(x)
        : "scc");
}

constexpr double kSumScale = 0x1p-64;  // of the sums of term_exp

// Per-lane scale c_j of the row's exponent (ex[3] = 1024 / ln 2).
__device__ __forceinline__ double row_scale(double sigma, const double* ex)
{
    return -ex[3] / (2.0 * (sigma * sigma));
}

static_assert(kTab == kWeightTab, "table length");
static_assert(kColTile == kWave, "a lane per column of a tile");

// Table entry i: 2^(i/1024 + 64) with i << 10 taken off its high word.
__device__ __forceinline__ double table_entry(int i)
{
    const long long e = __double_as_longlong(dm::exp((double)i * (0.6931471805599453 / kTab)));
    return __longlong_as_double(e + ((64ll << 52) - ((long long)i << (52 - kTabBits))));
}

// Copy of the table (written once per context by launch_weight_table) into
// LDS; all threads of the block take part.
__device__ __forceinline__ void load_table(double* T, const double* g)
{
    for (int i = threadIdx.x; i < kTab; i += blockDim.x) T[i] = g[i];
}

// Widest window of a row (the cap of window_radius): a column more than
// kWindow sigma_j away has an exponent below -710, where exp is 0 by the
// definition used throughout (dm::exp's cut-off); the table form has no cut-off
// of its own.
constexpr double kWindow = 37.7;

// Narrower per-row window with a bound on what it leaves out.  Every column
// with |u_k - u_j| > W sigma_j has a term at most q_k e^{-W^2/2}, so all of them
// together are at most Q e^{-W^2/2} (Q = sum_k q_k).  The row sum holds the parent's own term
// L_par = q_par e^{-|u_j - u_par|^2 / (2 sigma_j^2)}, so with
//   W^2 = 2 (ln Q - ln L_par + 53 ln 2)
// the omitted mass is at most 2^-53 of the row sum: one unit roundoff of the
// sum itself.  The parent always lies inside (W^2 >= |u_j - u_par|^2 /
// sigma_j^2 because Q >= q_par).  The result is capped at kWindow; a missing
// or zero parent weight leaves kWindow.  Returns the radius W sigma_j.
__device__ __forceinline__ double window_radius(const double* uj, double sj, const double* up, double qpar,
                                                   double Q)
{
    double W = kWindow;
    if (qpar > 0.0 && Q >= qpar && sj > 0.0) {
        double d2 = 0.0;
#pragma unroll
        for (int d = 0; d < kNP; ++d) {
            const double e = uj[d] - up[d];
            d2 = d2 + e * e;
        }
        const double x = d2 / (2.0 * sj * sj);
        const double w2 = 2.0 * ((dm::log(Q) - dm::log(qpar)) + x + 53.0 * 0.6931471805599453);
        const double w = __builtin_sqrt(w2);
        if (w < W) W = w;
    }
    return W * sj;
}

// 7-bit half-octave of a step size: rows of similar sigma share windows well
// (half-octaves give 2.5% fewer evaluated terms than octaves at N = 131072
// and 6% at N = 2^20).
__device__ __forceinline__ unsigned long long sigma_half_octave(double s)
{
    int e;
    const double m = __builtin_frexp(s, &e);
    int h = 2 * (e + 40) + (m >= 0.7071067811865476 ? 1 : 0);
    h = h < 0 ? 0 : (h > 127 ? 127 : h);
    return (unsigned long long)h;
}

__device__ __forceinline__ unsigned long long wave_sum_u64(unsigned long long v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

__device__ __forceinline__ float wave_minf(float v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fminf(v, __shfl_xor(v, off, kWave));
    return v;
}
__device__ __forceinline__ float wave_maxf(float v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = fmaxf(v, __shfl_xor(v, off, kWave));
    return v;
}

// ---- sort order ------------------------------------------------------------
// Rows and columns are put in the order of a bit-interleaved (Morton) code of
// their coordinates, scaled to the columns' box, so that 64 neighbours of
// either lie close together in all eight coordinates.  The interleaving spends
// its bits where they shrink the cells most: each next bit halves the
// coordinate whose cell is widest, measured in the columns' standard deviation.
__device__ __forceinline__ uint32_t cell20(double u, double lo, double inv)
{
    const double c = (u - lo) * inv;
    return (uint32_t)((c < 0.0 ? 0.0 : (c > 1.0 ? 1.0 : c)) * 1048575.0);
}

// First 32 bits of the code; cells: this thread's column of an LDS array
// (stride threads apart), so that the coordinate may be picked at run time.
__device__ __forceinline__ uint32_t morton32(const WeightGeom& g, const uint32_t* cells, int stride)
{
    uint32_t key = 0;
    for (int i = 0; i < 32; ++i) {
        const int s = g.seq[i];
        key = (key << 1) | ((cells[(s & 7) * stride] >> (19 - (s >> 3))) & 1u);
    }
    return key;
}

// From per-coordinate sums s1, sums of squares s2, minima and maxima over M
// columns (in LDS); at least 160 threads take part.  Bit b of coordinate d has
// the cell width var_d / 4^b (squared); the bits are taken widest first, equal
// ones by coordinate, so a bit's place is the number of bits before it.
__device__ __forceinline__ void make_geom(const double* s1, const double* s2, const double* mn, const double* mx,
                                          double M, WeightGeom* g)
{
    constexpr int bits = 20;
    __shared__ double width[kNP * bits];
    const int t = threadIdx.x;
    if (t < kNP * bits) {
        const double mean = s1[t / bits] / M;
        const double var = s2[t / bits] / M - mean * mean;
        width[t] = var > 0.0 ? __builtin_ldexp(var, -2 * (t % bits)) : 0.0;
    }
    if (t < kNP) {
        const bool any = mx[t] >= mn[t];  // false without columns
        g->lo[t] = any ? mn[t] : 0.0;
        g->inv[t] = mx[t] > mn[t] ? 1.0 / (mx[t] - mn[t]) : 0.0;
        g->mid[t] = any ? 0.5 * (mn[t] + mx[t]) : 0.5;
    }
    __syncthreads();
    if (t < kNP * bits) {
        const double w = width[t];
        int place = 0;
#pragma unroll 8
        for (int o = 0; o < kNP * bits; ++o) place += (width[o] > w || (width[o] == w && o < t)) ? 1 : 0;
        if (place < 32) g->seq[place] = t / bits | ((t % bits) << 3);
    }
}

// ---- pair test -------------------------------------------------------------
// Which columns any of 64 rows needs, by one matrix product in float16: with
// f = 4096 (u - mid) = h + l (two float16 parts),
//   |f_j - f_k|^2 - R_j^2 = n_j - R_j^2 + n_k - 2 (h_j h_k + h_j l_k + l_j h_k) + ...
// in 24 products of the parts and 2 x 3 for the squared norms (three float16
// parts each, times 32768): K = 30 of 32, accumulated in float32.  The row's
// constant is lowered by a bound on everything the test may be wrong by, so
// that no pair inside a row's window is lost: at most 33 sums of partial sums
// below 2 (n_j + n_k) + R_j^2, each off by 2^-23 of it, plus the dropped l_j l_k
// and the parts' own roundings (2^-20 of n_j + n_k; 16 covers parts that are
// subnormal), where n_k <= (sqrt(n_j) + R)^2 for a column inside the window:
// together below (n_j + n_k) 2^-16 + 16.
typedef _Float16 half8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
constexpr double kOpScale = 4096.0, kNormScale = 32768.0;

__device__ __forceinline__ void split3(double v, _Float16* o)
{
    for (int i = 0; i < 3; ++i) {
        o[i] = (_Float16)(float)v;
        v -= (double)(float)o[i];
    }
}

// h, l and the squared norm (in units of f^2) of one point
__device__ __forceinline__ double split_point(const double* u, const WeightGeom& g, half8& h, half8& l)
{
    double n = 0.0;
#pragma unroll
    for (int d = 0; d < kNP; ++d) {
        const double f = (u[d] - g.mid[d]) * kOpScale;
        h[d] = (_Float16)(float)f;
        l[d] = (_Float16)(float)(f - (double)(float)h[d]);
        n += f * f;
    }
    return n;
}

__device__ __forceinline__ void column_operand(const double* u, const WeightGeom& g, half8* op)
{
    const double n = split_point(u, g, op[0], op[1]);
    _Float16 p[3];
    split3(n / kNormScale, p);
    const _Float16 s = (_Float16)(float)kNormScale;
    op[2] = half8{p[0], p[1], p[2], s, s, s, (_Float16)0, (_Float16)0};
}

__device__ __forceinline__ void row_operand(const double* u, const WeightGeom& g, double radius, half8* op)
{
    const double n = split_point(u, g, op[0], op[1]);
#pragma unroll
    for (int d = 0; d < kNP; ++d) {
        op[0][d] = op[0][d] * (_Float16)-2;
        op[1][d] = op[1][d] * (_Float16)-2;
    }
    const double R = (radius < 3.0 ? radius : 3.0) * kOpScale;  // 3 > the cube's diagonal
    const double far = __builtin_sqrt(n) + R;
    const double m = n - R * R - ((n + far * far) * 0x1p-16 + 16.0);
    _Float16 p[3];
    split3(m / kNormScale, p);
    const _Float16 s = (_Float16)(float)kNormScale;
    op[2] = half8{s, s, s, p[0], p[1], p[2], (_Float16)0, (_Float16)0};
}

// a row that needs nothing (the padding of the last group)
__device__ __forceinline__ void null_operand(half8* op)
{
    const _Float16 z = (_Float16)0, s = (_Float16)(float)kNormScale;
    op[0] = op[1] = half8{z, z, z, z, z, z, z, z};
    op[2] = half8{s, s, s, (_Float16)60000.0f, z, z, z, z};
}

// Sorted slot i of the columns or rows from point u (real: not padding).  The
// threads of a wave hold 64 consecutive slots and reduce their box.
__device__ __forceinline__ void store_box(float* box, const double* u, bool real)
{
    const int lane = threadIdx.x & (kWave - 1);
#pragma unroll
    for (int d = 0; d < kNP; ++d) {
        const float v = (float)u[d];
        const float lo = wave_minf(real ? v : __builtin_inff()), hi = wave_maxf(real ? v : -__builtin_inff());
        if (lane == 0) {
            box[d] = lo;
            box[kNP + d] = hi;
        }
    }
}

__device__ __forceinline__ float box_threshold(float radius);

__device__ __forceinline__ void gather_column(const WeightCols& c, const WeightGeom& g, size_t i, bool real,
                                              const double* src)
{
    double u[kNP];
#pragma unroll
    for (int d = 0; d < kNP; ++d) u[d] = real ? src[d] : g.mid[d];
    half8 op[3];
    column_operand(u, g, op);
#pragma unroll
    for (int d = 0; d < kNP; ++d) c.u[i * kNP + d] = u[d];
    c.q[i] = real ? src[kNP] : 0.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) ((half8*)c.op)[k * c.pad + i] = op[k];
    store_box(c.box + i / kColTile * 16, u, real);
}

__device__ __forceinline__ void gather_row(const WeightRows& w, const WeightGeom& g, size_t i, bool real,
                                           const double* src, double sigma, double radius, const double* ex)
{
    double u[kNP];
#pragma unroll
    for (int d = 0; d < kNP; ++d) u[d] = real ? src[d] : g.mid[d];
    half8 op[3];
    if (real) row_operand(u, g, radius, op);
    else null_operand(op);
#pragma unroll
    for (int d = 0; d < kNP; ++d) w.u[i * kNP + d] = u[d];
    w.scale[i] = real ? row_scale(sigma, ex) : 0.0;
    w.r2[i] = real ? radius * radius : -1.0;
#pragma unroll
    for (int k = 0; k < 3; ++k) ((half8*)w.op)[k * w.pad + i] = op[k];
    float* box = w.box + i / kWave * 17;
    store_box(box, u, real);
    const float R = wave_maxf(real ? (float)radius * 1.000001f : 0.0f);
    if ((threadIdx.x & (kWave - 1)) == 0) box[16] = box_threshold(R);
}

// Threshold of the box test on |gap|^2 (float32 coordinates are off by 6e-8, a
// gap's length by at most 3.4e-7) for the largest radius of a row group.
__device__ __forceinline__ float box_threshold(float radius)
{
    return radius * radius * 1.00001f + 1e-6f * radius + 1e-12f;
}

// Of the tiles [s0, s0 + 64) below t1, those whose box comes near enough to the
// row group's box (a lane per tile).
__device__ __forceinline__ unsigned long long near_tiles(const WeightRows& rows, const WeightCols& cols, int group,
                                                         int lane, int s0, int t1)
{
    const float* box = rows.box + (size_t)group * 17;
    bool need = false;
    if (s0 + lane < t1) {
        const float* tb = cols.box + (size_t)(s0 + lane) * 16;
        float g2 = 0.0f;
#pragma unroll
        for (int d = 0; d < kNP; ++d) {
            const float g = fmaxf(fmaxf(tb[d] - box[8 + d], box[d] - tb[8 + d]), 0.0f);
            g2 += g * g;
        }
        need = g2 <= box[16];
    }
    return __ballot(need);
}

// One wave's 64 rows (a lane each) against the column tiles [t0, t1): the sum
// of this lane's row.  Bound by FP64 issue, so the work is in choosing what to
// evaluate: a lane per tile tests the tile's box against the rows' box; a tile
// that passes is tested pair by pair on the matrix cores (pair test above, four
// 32x32 products a half tile; with the lists 11% of the instructions in stage 1
// of N = 131072);
// the columns that some row needs are the set bits of a scalar word, taken two
// at a time by scalar instructions (which issue beside the other waves' vector
// ones, though not for nothing: 21 a term instead of 14 cost 3%; three or four
// at a time run out of scalar registers, 262 against 269 ms in stage 1 of
// N = 2^20, and a list in LDS took 278).  At N = 131072 they are 53, 36, 24,
// 9, 3 and 1% of all pairs in stages 1, 2, 3, 5, 7 and 9 (a window on one
// sorted coordinate evaluated 80, 66, 53, 29, 13 and 8%; the rows' own windows
// hold 36, 21, 13, 3, 1 and 0.3%).  Two interleaved sums
// (first and second of a pair), flushed once a tile.
// part, parts: of the near tiles in turn, this wave's share.
// window: pairs of this wave inside the rows' own windows, over all lanes.
// first: near_tiles() of the first kWave tiles.
__device__ __forceinline__ double row_sum(const WeightRows& rows, const WeightCols& cols, int group, int lane, int t0,
                                          int t1, int M, unsigned long long first, const double* T, const double* ex,
                                          uint32_t& listed, uint32_t& window, int part = 0, int parts = 1)
{
    const int r = group * kWave + lane;
    double uj[kNP];
#pragma unroll
    for (int d = 0; d < kNP; ++d) uj[d] = rows.u[(size_t)r * kNP + d];
    const double cj = rows.scale[r], R2 = rows.r2[r];
    const bool upper = lane >= 32;
    half8 a0[2], a1[2];
#pragma unroll
    for (int b = 0; b < 2; ++b) {
        const size_t i = (size_t)group * kWave + 32 * b + (lane & 31);
        a0[b] = ((const half8*)rows.op)[i];
        a1[b] = ((const half8*)rows.op)[(upper ? 2 : 1) * rows.pad + i];
    }
    const half8* ch = (const half8*)cols.op;
    const half8* cb0 = ch + (upper ? cols.pad : 0);       // h below, l above
    const half8* cb1 = ch + (upper ? 2 * cols.pad : 0);   // h below, norms above
    const uint32_t kbase = (uint32_t)t0 * kColTile;
    const const_col_ptr cu = (const_col_ptr)(cols.u + (size_t)kbase * kNP), cq = (const_col_ptr)(cols.q + kbase);
    double total = 0.0;
    uint32_t cnt = 0;
    double ex1 = ex[1];  // in vector registers: an fma takes one scalar operand
    asm volatile("" : "+v"(ex1));
    auto term = [&](const Col& c, double& p) {
        const double D = dist2(uj, c);
        const unsigned long long in = __ballot(D <= R2);
        window += (uint32_t)__popcll(in);
        add_where(in, c.q, term_exp(D, cj, T, ex, ex1), p);
    };
    uint32_t odd = 0;  // a listed column without a partner yet
    bool have_odd = false;
    for (int s0 = t0; s0 < t1; s0 += kWave) {
        unsigned long long tiles = s0 == t0 ? first : near_tiles(rows, cols, group, lane, s0, t1);
        for (int i = 0; i < part; ++i) tiles &= tiles - 1;
        while (tiles) {
            const int t = s0 + __builtin_ctzll(tiles);
            for (int i = 0; i < parts; ++i) tiles &= tiles - 1;
            const int k0 = t * kColTile;
            unsigned long long bits = 0;
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const size_t k = (size_t)k0 + 32 * h + (lane & 31);
                const half8 b0 = cb0[k], b1 = cb1[k];
                f32x16 c[2];
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    c[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a0[b], b0, f32x16{}, 0, 0, 0);
                    c[b] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a1[b], b1, c[b], 0, 0, 0);
                }
                float m = fminf(c[0][0], c[1][0]);
#pragma unroll
                for (int i = 1; i < 16; ++i) m = fminf(fminf(c[0][i], c[1][i]), m);
                const unsigned long long bal = __ballot(m <= 0.0f);
                bits |= (unsigned long long)((uint32_t)bal | (uint32_t)(bal >> 32)) << (32 * h);
            }
            const int left = M - k0;
            if (left < kColTile) bits &= (1ull << left) - 1ull;
            int n = __popcll(bits);
            cnt += (uint32_t)n;
            // the next near tile on its way into the cache while this one is evaluated
            const size_t kn = (size_t)(s0 + (tiles ? __builtin_ctzll(tiles) : t - s0)) * kColTile + lane;
            const float touch0 = ((const float*)(cols.u + kn * kNP))[0], touch1 = ((const float*)(cols.q + kn))[0],
                        touch2 = ((const float*)(ch + kn))[0], touch3 = ((const float*)(ch + cols.pad + kn))[0],
                        touch4 = ((const float*)(ch + 2 * cols.pad + kn))[0];
            double p0 = 0.0, p1 = 0.0;
            const uint32_t k1 = (uint32_t)k0 - kbase;
            auto next = [&]() {
                const uint32_t k = (uint32_t)__builtin_ctzll(bits);
                asm("s_bitset0_b64 %0, %1" : "+s"(bits) : "s"(k));
                return k1 + k;
            };
            for (n += have_odd; n >= 2; n -= 2) {
                const uint32_t e0 = have_odd ? odd : next(), e1 = next();
                have_odd = false;
                const Col c0 = load_col(cu, cq, e0), c1 = load_col(cu, cq, e1);
                term(c0, p0);
                term(c1, p1);
            }
            if (bits) {
                odd = next();
                have_odd = true;
            }
            total += p0 + p1;
            asm volatile("" ::"v"(touch0), "v"(touch1), "v"(touch2), "v"(touch3), "v"(touch4));
        }
    }
    double p = 0.0;
    if (have_odd) term(load_col(cu, cq, odd), p);
    listed = cnt;
    return (total + p) * kSumScale;
}

}  // namespace wterm
}  // namespace abcsmc
