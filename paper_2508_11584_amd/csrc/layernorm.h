// LayerNorm of one row by one wavefront: the stand-alone kernel (rowops.h) and the workgroups that ride in an attention launch
// (attention.h) normalise the tapped rows with it.
#pragma once
#include "common.h"

namespace vpe {

// LayerNorm over the last axis of the fp32 residual stream: y = g (x - mean) / sqrt(var + eps) + b
// with the biased variance; statistics in fp32 (mean first, then centred second moment, both
// from registers).  D multiple of 64, D <= 64 * 32.
template <typename T>
__device__ __forceinline__ void layernorm_row(const float* __restrict__ x, int row, int D, const float* __restrict__ gam,
                                              const float* __restrict__ bet, float eps, T* __restrict__ y, int lane) {
    constexpr int MAXV = 16;                     // float2 per lane -> D <= 2048
    const int nv = D >> 7;                       // full float2 passes (128 elements each)
    const bool tail = (D & 64) != 0;             // one extra pass of single floats
    const float* xr = x + (int64_t)row * D;
    f32x2 v[MAXV];
    float t = 0.0f, sum = 0.0f;
#pragma unroll
    for (int i = 0; i < MAXV; ++i)
        if (i < nv) {
            v[i] = *reinterpret_cast<const f32x2*>(xr + i * 128 + 2 * lane);
            sum += v[i][0] + v[i][1];
        }
    if (tail) { t = xr[nv * 128 + lane]; sum += t; }
    const float mean = wave_sum(sum) / D;
    float sq = 0.0f;
#pragma unroll
    for (int i = 0; i < MAXV; ++i)
        if (i < nv) {
            const float a = v[i][0] - mean, b = v[i][1] - mean;
            sq += a * a + b * b;
        }
    if (tail) sq += (t - mean) * (t - mean);
    const float rstd = 1.0f / sqrtf(wave_sum(sq) / D + eps);
    T* yr = y + (int64_t)row * D;
#pragma unroll
    for (int i = 0; i < MAXV; ++i)
        if (i < nv) {
            const int c = i * 128 + 2 * lane;
            const f32x2 gg = *reinterpret_cast<const f32x2*>(gam + c);
            const f32x2 bb = *reinterpret_cast<const f32x2*>(bet + c);
            yr[c] = from_f32<T>(gg[0] * (v[i][0] - mean) * rstd + bb[0]);
            yr[c + 1] = from_f32<T>(gg[1] * (v[i][1] - mean) * rstd + bb[1]);
        }
    if (tail) {
        const int c = nv * 128 + lane;
        yr[c] = from_f32<T>(gam[c] * (t - mean) * rstd + bet[c]);
    }
}

}  // namespace vpe
