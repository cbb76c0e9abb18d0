// Keyframe sums from their work-groups' partials, shared by the geometric and
// the photometric term.
#pragma once
#include "gsdf_common.hpp"
#include "gsdf_se3.hpp"

namespace gsdf {

// One work-group per keyframe: fixed-order sum of its n partials (eight
// float64 values each: loss, six pose sums, count), then loss_out[kf],
// count_out[kf] and dxi_out = Jl(xi)^T (pose sums), each when asked for.
//
// Bound by latency: the loads of a partial, the sum across threads, the sines
// of Jl.  A thread takes every THREADS-th partial; the sums cross lanes by
// register moves and waves through LDS once; the last wave, which has the
// fewest partials, forms Jl meanwhile.  (256 threads, a tree in LDS with a
// barrier a level, then Jl: 9.3 us for 30 keyframes of 2686 partials, now
// 6.7; 5.6 for 300 partials, now 4.6.)
template <int THREADS>
__global__ __launch_bounds__(THREADS) void k_keyframe_finish(int64_t n, const double* __restrict__ xi,
                                                             const double* __restrict__ partials,
                                                             double* __restrict__ loss_out,
                                                             double* __restrict__ dxi_out,
                                                             double* __restrict__ count_out) {
    constexpr int kWaves = THREADS / 64, kPart = 8;
    __shared__ double s_part[kPart][kWaves];
    __shared__ double s_sum[kPart];
    __shared__ double s_jl[36];
    const int kf = blockIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    double x[kPart];
#pragma unroll
    for (int k = 0; k < kPart; ++k) x[k] = 0.0;
    for (int64_t b = threadIdx.x; b < n; b += THREADS) {
        const double* p = partials + ((size_t)kf * n + b) * kPart;
#pragma unroll
        for (int k = 0; k < kPart; ++k) x[k] += p[k];
    }
    const double y = wave_sum8(x, lane);
    if ((lane & 7) == 0) s_part[wave_sum8_value(lane)][wave] = y;
    if (dxi_out && threadIdx.x == THREADS - 64) se3_left_jacobian(xi + 6 * kf, s_jl);
    __syncthreads();
    if (threadIdx.x < kPart) {
        double v = 0.0;
        for (int w = 0; w < kWaves; ++w) v += s_part[threadIdx.x][w];
        s_sum[threadIdx.x] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        if (loss_out) loss_out[kf] = s_sum[0];
        if (count_out) count_out[kf] = s_sum[7];
    }
    if (dxi_out && threadIdx.x < 6) {
        double v = 0.0;
        for (int r = 0; r < 6; ++r) v += s_jl[6 * r + threadIdx.x] * s_sum[1 + r];
        dxi_out[6 * kf + threadIdx.x] = v;
    }
}

}  // namespace gsdf
