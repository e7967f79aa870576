// predict.hip -- posterior predictive simulation (§IV-B, Fig. 7): the
// particles of a completed stage simulated over a longer horizon, and per
// day the type-7 quantiles of A, R and D over the particles.
#include "blockselect.h"
#include "kernels.h"
#include "predict.h"
#include "propose.h"

namespace abcsmc {

namespace {

// Lane per particle j: theta = lo + u width, trajectory of the stream
// (seed, j, round) written as series[(3 t + c) N + j].
// (kQuad: a quad per particle).
template <int kSampler, bool kQuad>
__global__ __launch_bounds__(kBlock) void predict_series_kernel(PredictArgs a)
{
    const int64_t t = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    const int64_t j = kQuad ? t / 4 : t;
    if (j >= a.n) return;
    double th[kNP];
#pragma unroll
    for (int q = 0; q < kNP; ++q) th[q] = a.m.lo[q] + a.u[j * kNP + q] * a.m.width[q];
    int32_t days = 0;
    if (kQuad)
        lane::simulate_distance_quad<kSampler, true>(a.m, th, nullptr, a.round, (uint32_t)j, __builtin_inf(), nullptr,
                                                     days, nullptr, a.series + j, a.n);
    else
        lane::simulate_distance<kSampler, true>(a.m, th, nullptr, a.round, (uint32_t)j, __builtin_inf(), nullptr, days,
                                                nullptr, a.series + j, a.n);
}

// One block per (day, series) row: its n_quant quantiles, the row held in
// registers where it fits (K doubles a thread): 453 rows of 32768 values, three
// quantiles, 427 us from memory and 332 from registers.
template <int K>
__global__ __launch_bounds__(bsel::kThreads) void predict_band_kernel(PredictArgs a)
{
    __shared__ bsel::Shared sh;
    const int64_t row = blockIdx.x;  // 3 t + c
    const double* x = a.series + (size_t)row * a.n;
    const int n = (int)a.n;
    auto quantiles = [&](const auto& values) {
        for (int k = 0; k < a.n_quant; ++k) {
            const double v = bsel::quantile7(values, n, a.quant[k], sh);
            if (threadIdx.x == 0) a.bands[row * a.n_quant + k] = v;
        }
    };
    if constexpr (K > 0) quantiles(bsel::FromRegisters<K>(x, n));
    else quantiles(bsel::FromMemory{x, n});
}

}  // namespace

void launch_predict(const PredictArgs& a, hipStream_t s)
{
    const bool quad = propose_by_quads(a.n, a.m.sampler, a.m.any_rates);
    const dim3 grid((unsigned)(((quad ? 4 * a.n : a.n) + kBlock - 1) / kBlock));
    if (a.m.sampler == 0) {
        if (quad) hipLaunchKernelGGL((predict_series_kernel<0, true>), grid, dim3(kBlock), 0, s, a);
        else hipLaunchKernelGGL((predict_series_kernel<0, false>), grid, dim3(kBlock), 0, s, a);
    } else {
        if (quad) hipLaunchKernelGGL((predict_series_kernel<1, true>), grid, dim3(kBlock), 0, s, a);
        else hipLaunchKernelGGL((predict_series_kernel<1, false>), grid, dim3(kBlock), 0, s, a);
    }
    const dim3 rows((unsigned)(3 * (a.m.T + 1))), b(bsel::kThreads);
    if (a.n <= 8 * bsel::kThreads) hipLaunchKernelGGL(predict_band_kernel<8>, rows, b, 0, s, a);
    else if (a.n <= 32 * bsel::kThreads) hipLaunchKernelGGL(predict_band_kernel<32>, rows, b, 0, s, a);
    else hipLaunchKernelGGL(predict_band_kernel<0>, rows, b, 0, s, a);
}

}  // namespace abcsmc
