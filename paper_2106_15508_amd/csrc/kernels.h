// kernels.h -- kernel argument blocks and launch wrappers of the HIP path.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace abcsmc {

constexpr int kNP = 8;        // parameters per particle (eq. 1)
constexpr int kBlock = 256;   // threads per workgroup of the per-lane kernels
constexpr int kWave = 64;
constexpr int kWeightRows = 128;  // sorted rows per workgroup (and per window) of the weight kernel

// Model constants shared by every simulation (§II-B).
struct Model {
    double lo[kNP];     // prior box lower corner
    double width[kNP];  // hi - lo
    double P;           // population (exact integer)
    double invP;        // 1 / P
    double A0, R0, D0;  // day-0 observed state
    int32_t T;          // days
    int32_t sampler;    // 0 binomial, 1 floor-normal
    int32_t any_rates;  // parameters may be undefined or huge (ordinary_rates())
    uint64_t seed;
};

// Whether n parameters are such that no rate, probability or count of a day
// can become NaN: every one defined and below 2^1022, so that alpha0 + alpha_c
// stays finite (products that overflow end as probabilities of 0 or 1).
inline bool ordinary_rates(const double* v, int64_t n)
{
    bool all = true;
    for (int64_t i = 0; i < n; ++i) all &= __builtin_fabs(v[i]) < 0x1p1022;
    return all;
}

// Points of a stage whose device time is noted (StageCounters::ts).
enum StageMark { kTsBegin, kTsPropose, kTsProposed, kTsWeights, kTsSum, kTsSummed, kTsSelect, kTsEnd, kTsCount };

// Device counters and results of one stage (8-byte words), read back together.
struct StageCounters {
    unsigned long long accepted;   // acceptances over the batches run so far
    unsigned long long proposals;  // index of the N-th acceptance + 1 (0 until reached)
    unsigned long long invalid;    // void proposals over the batches run so far
    unsigned long long attempts;   // perturbation attempts over the batches run so far
    unsigned long long survivors;  // previous particles with q > 0
    unsigned long long fallback;   // 1 if the prior set used d <= eps (no d < eps)
    unsigned long long days;       // proposal-days simulated over the batches run so far
    unsigned long long terms;      // importance-weight terms evaluated (inside the windows)
    unsigned long long window_terms;  // sum over rows of the row's own window (terms the rows need)
    double eps_next;               // eq. 8 of the accepted distances
    double ess;                    // effective sample size
    unsigned long long crowded;    // 1: eps_next is left to launch_select_crowded
    // the constant-rate clock when the first workgroup of a phase's first kernel
    // starts: the phases' times without an event record (a few us of idle GPU
    // each) between the kernels
    unsigned long long ts[kTsCount];
};

// Population of one stage, array-of-structures for the per-particle gathers.
struct Population {
    double* u;        // N x 8
    double* d;        // N
    double* sigma;    // N
    int32_t* parent;  // N
    uint32_t* index;  // N
    int32_t* att;     // N
    double* logw;     // N
    double* W;        // N
};

struct ProposeArgs {
    Model m;
    const double* obs;  // (T+1) x 3, exact integers
    uint32_t round;
    uint32_t base;      // first proposal index of the batch
    uint32_t count;     // proposals in the batch
    int32_t max_attempts;
    double eps;         // accept iff d <= eps
    double exit_thr;    // early exit once the partial sum of squares exceeds this (+inf: off)
    // perturbation (stage >= 1)
    const double* u_prev;    // n_prev x 8
    const uint64_t* cdf;     // n_prev inclusive prefix sums of q
    int32_t n_prev;
    double beta_a;
    int32_t beta_b;
    int32_t step_is_variance;
    double s_fixed;          // >= 0: every proposal uses step size s_fixed (MCMC variant), no Beta draw
    double beta_b_real;      // > 0: real Beta shape b, general sampler (alternative parameterisations)
    // staging, indexed by p = j - base
    double* st_u;            // count x 8
    double* st_d;
    double* st_sigma;
    int32_t* st_parent;
    int32_t* st_att;
    unsigned long long* wave_mask;  // ceil(count/64) acceptance ballots
    StageCounters* ctr;
};

struct CompactArgs {
    uint32_t base;
    uint32_t count;
    unsigned long long before;  // acceptances of the stage's earlier batches
    int32_t N;
    const unsigned long long* wave_mask;
    uint32_t* wave_off;   // exclusive prefix of popcounts
    const double* st_u;
    const double* st_d;
    const double* st_sigma;
    const int32_t* st_parent;
    const int32_t* st_att;
    Population pop;
    StageCounters* ctr;
};

// Per-block partial results of the multi-block reductions and scans.
constexpr int kRedMax = 4096;  // max blocks of a reduction (N <= 2^22 at 1024 per block)
// Values of one bin that the percentile's last workgroup finishes (as many
// crowded ones 90 us); more are left to the whole chip.
constexpr int kSelectList = 1 << 14;
struct Scratch {
    unsigned long long* u0;  // kRedMax
    unsigned long long* u1;  // kRedMax
    unsigned long long* u2;  // kRedMax
    double* d0;              // kRedMax
    double* d1;              // kRedMax
    unsigned int* hist;      // 2048 bins of the multi-block select
    unsigned long long* sel; // its state: values collected, values below the bin, values in the bin;
                             // prefix of the bin, its undecided low bits, rank in it; whether crowded
    double* list;            // collected values
    uint32_t list_cap;       // as many as it holds, kSelectList at most
};

struct ResampleArgs {
    const double* d_prev;   // N
    const double* u_prev;   // N x 8
    int32_t N;
    double eps;
    uint64_t* q;            // N
    uint64_t* cdf;          // N
    double* cols;           // M x 9: u_k[8], q_k  (q_k > 0 only, index order)
    Scratch sc;
    StageCounters* ctr;
};

// N up to which one workgroup of kOneThreads threads takes a pass over the
// particles instead of a chain of launches (each about 4.5 us and 1.5 us of gap):
//   resampling     22 us at 4096 (44 at 8192) against three launches of 24 and two gaps
//   sort keys      18 us at 1024 (26 at 2048) against three launches of 19 and two gaps
//   stage end      15-20 us at 16384 (normalisation and percentile side by side)
//                  against four launches of 20 and the percentile's 20
// and up to which the sort counts smaller keys (34 us at 16384, growing with
// N^2, against 71 us and ten gaps for the bitonic launches at 20011).
constexpr int kOneThreads = 1024;
constexpr int kOneResample = 1 << 12;
constexpr int kOnePrep = 1 << 10;
constexpr int kOneEnd = 1 << 14;
constexpr int kRankSort = 24576;

// Entries of the weight kernels' exponential table (2^(i/1024)).
constexpr int kWeightTab = 1024;

// Scale and bit order of the weight pass' sort code (device).
struct WeightGeom {
    double lo[kNP], inv[kNP];  // the columns' box: (u - lo) inv in [0, 1]
    double mid[kNP];           // its centre
    int32_t seq[32];           // code bit i: coordinate | (bit of it << 3)
};

constexpr int kColTile = 64;    // columns per tile of the weight kernels

// Sorted columns (survivors of the previous stage).
struct WeightCols {
    double* u;     // M x 8
    double* q;     // M
    void* op;      // 3 x pad float16 octets: high parts, low parts, norms
    float* box;    // per tile: minima[8], maxima[8]
    size_t pad;    // columns padded to whole tiles
};

// Sorted rows (accepted particles), in groups of a wave.
struct WeightRows {
    double* u;      // pad x 8
    double* scale;  // c_j = -1024 / (2 sigma_j^2 ln 2)
    double* r2;     // squared window radius (-1 in the padding)
    void* op;       // 3 x pad float16 octets
    float* box;     // per group: minima[8], maxima[8], box test threshold
    size_t pad;     // rows padded to whole kWeightRows blocks
};

__host__ __device__ inline size_t weight_col_pad(size_t n) { return (n + kColTile - 1) / kColTile * kColTile; }
__host__ __device__ inline size_t weight_row_pad(size_t n) { return (n + kWeightRows - 1) / kWeightRows * kWeightRows; }

struct WeightArgs {
    const double* u;        // N x 8 rows
    const double* sigma;    // N
    const double* cols;     // M x 9
    int32_t N;
    int32_t chunks;         // column chunks (second grid dimension)
    const unsigned long long* M;  // device scalar: survivors
    double* partial;        // slots x N row sums per column chunk
    double* logw;           // N
    unsigned long long* rowkeys;  // Npad sort keys (row index in the low 32 bits)
    unsigned long long* colkeys;  // Npad sort keys (column index in the low 32 bits)
    unsigned long long* unsorted[2];  // up to kRankSort: the columns' and rows' keys before the sort
    StageCounters* ctr;
    WeightCols sc;
    WeightRows sr;
    double* dimpart;        // kDimBlocks x 32 per-block statistics of the columns
    WeightGeom* geom;       // device: the sort code
    size_t npad;            // padded sort length (power of two >= N)
    int32_t chunk_tiles;    // column tiles per chunk
    int32_t slots;          // chunks that `partial` holds at once
    int32_t first_chunk;    // of one pass over the chunks: its first one
    int32_t first_slot;     // and that one's slot (1 after the first pass: slot 0 holds the sums so far)
    uint2* counts;          // chunks x groups: columns listed, pairs inside the rows' own windows
    unsigned long long* terms;  // device counter of evaluated terms
    unsigned long long* window_terms;  // device counter: pairs inside the rows' own windows
    // per-row window radii from each row's parent term
    const int32_t* parent;  // N parent indices into the previous population
    const double* u_prev;   // previous population, n_prev x 8
    const uint64_t* q_prev; // its resampling weights q_k (0 for non-survivors)
    const uint64_t* cdf;    // its integer CDF (cdf[n_prev - 1] = Q)
    int32_t n_prev;
    double* rwin;           // N radii W_j sigma_j
    // table exponential: ln2/1024, its square / 2, its cube / 6, 1024/ln2
    // (kernel arguments so they sit in scalar registers)
    double ex[7];
    const double* tab;      // kWeightTab entries 2^(i/1024), written once per context
};

// Fill WeightArgs::ex.
void weight_exp_constants(double ex[7]);
// Write the kWeightTab table entries 2^(i/1024) to tab (device memory).
void launch_weight_table(double* tab, hipStream_t s);
// Test hook: n importance-weight terms, records {u_j[8], sigma_j, u_k[8], q_k}.
void launch_wterm_debug(int64_t n, const double* in, double* out, hipStream_t s);

// Regions of 64-bit keys that are sorted each by itself, side by side from
// slot 0 on: each a power of two long, in descending order of length (so every
// region lies at a multiple of its length).  n[b]: keys in regions of at least
// 2^b (n[0] all; 0 past the longest).
constexpr int kSortLevels = 32;
struct SortSpans {
    size_t n[kSortLevels];
};
// slots to allocate for n keys of regions (whole LDS tiles)
size_t sort_span_slots(size_t n);
void launch_sort_spans(unsigned long long* keys0, unsigned long long* keys1, const SortSpans& sp, hipStream_t s);

// Bitonic sort of 64-bit keys (length a power of two >= 2048).
size_t sort_padded_size(size_t n);
// both arrays (each n_pow2 keys; keys1 may be null) by the same launches
void launch_sort_u64_pair(unsigned long long* keys0, unsigned long long* keys1, size_t n_pow2, hipStream_t s);

struct NormArgs {
    double* logw;
    double* W;
    int32_t N;
    int32_t uniform;        // 1: W = 1/N, log-weights 0 (stage 0, weight-free runs)
    Scratch sc;
    double* ess;            // device scalar
};

struct SelectArgs {
    const double* x;        // N non-negative (or +inf) values
    int32_t N;
    double alpha;
    Scratch sc;
    double* out;            // device scalar: type-7 quantile
    StageCounters* ctr;     // where its start and whether the values are crowded is noted, or null
};

// Column tiles per chunk (grid y) and chunks of the weight kernel for N rows.
int weight_chunk_tiles(int64_t N);
int weight_chunks(int64_t N);
// Bytes the first versions' weight pass (and copied out parameters) took for N
// rows beside the proposals' staging.
size_t weight_first_bytes(int64_t N);
constexpr int kDimBlocks = 64;  // blocks of the column statistics

struct TrajArgs {
    Model m;
    const double* theta;    // n x 8 (prior units)
    int64_t n;
    uint32_t round;
    uint32_t index0;
    int64_t* traj;          // n x (T+1) x 6
};

void launch_propose(const ProposeArgs& a, bool round0, hipStream_t s);
// Largest first batch of a stage without a measured acceptance rate: one
// round of the proposal kernel's resident waves on the current device (its
// occupancy in workgroups per compute unit x the compute units), so a first
// batch never leaves lanes of a second round to run on a mostly idle chip.
int64_t propose_first_batch_lanes();
// Whether n trajectories of one launch are made by four lanes each.
bool propose_by_quads(int64_t n, int sampler, bool any_rates);
void launch_compact(const CompactArgs& a, hipStream_t s);
void launch_resample(const ResampleArgs& a, hipStream_t s);
// The weight pass in three parts, so that the caller can time the sum kernel
// alone: the preparation (sort code from the columns' statistics, column and
// row sorts, sorted operands), the windowed sums, and the per-row merge of the
// chunk partial sums.
void launch_weights_window(const WeightArgs& a, hipStream_t s);
// (sum notes its last pass in a for finalize.)
void launch_weights_sum(WeightArgs& a, hipStream_t s);
void launch_weights_finalize(const WeightArgs& a, hipStream_t s);
void launch_select(const SelectArgs& a, hipStream_t s);
// The quantile where launch_select noted crowded values (without a.ctr it has
// done so itself).
void launch_select_crowded(const SelectArgs& a, hipStream_t s);
// Normalised (or uniform) weights and the next tolerance.
void launch_stage_end(const NormArgs& n, const SelectArgs& q, hipStream_t s);
// The stage's counters to pinned host memory.
void launch_publish(StageCounters* ctr, StageCounters* host, hipStream_t s);
void launch_simulate_traj(const TrajArgs& a, hipStream_t s);
void launch_to_theta(const double* u, const Model& m, double* theta, int64_t n, hipStream_t s);
void launch_debug_eval(int32_t fn, int64_t n, const void* in, void* out, double pa, int32_t pb,
                       hipStream_t s);

}  // namespace abcsmc
