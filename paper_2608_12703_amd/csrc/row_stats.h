// LayerNorm statistics by 16 lanes per row, shared by the float32 LayerNorm kernel and the
// float32 products that normalise their own rows: the same bits wherever a row is normalised.
#pragma once
#include "common.h"
#include "top2.h"

namespace ad {

constexpr int kRowStatsMax = 512;   // widest row that 16 lanes hold in registers
constexpr int kRowParts = kRowStatsMax / 64;
constexpr float kLnEps = 1e-5f;

// Part t of a row of d <= 512 values, d a multiple of 64: lane c16 of 16 takes values
// 64 t + 4 c16 .. + 3 (parts past the row repeat its last; row_stats leaves them out).
__device__ __forceinline__ f32x4 row_part(const float* xr, int d, int c16, int t) {
  return *(const f32x4*)(xr + min(64 * t, d - 64) + 4 * c16);
}

// Sum over 16 lanes by rotations (no LDS round trip); every lane gets the same bits.
__device__ __forceinline__ float sum16(float v) {
  v += __int_as_float(ror16<8>(__float_as_int(v)));
  v += __int_as_float(ror16<4>(__float_as_int(v)));
  v += __int_as_float(ror16<2>(__float_as_int(v)));
  v += __int_as_float(ror16<1>(__float_as_int(v)));
  return v;
}

// (mean, 1 / sqrt(biased variance + eps)), two passes over the registers.
__device__ __forceinline__ float2 row_stats(const f32x4 (&x)[kRowParts], int d) {
  float s = 0.f, v = 0.f;
#pragma unroll
  for (int t = 0; t < kRowParts; ++t) s += 64 * t < d ? (x[t][0] + x[t][1]) + (x[t][2] + x[t][3]) : 0.f;
  const float mean = sum16(s) / (float)d;
#pragma unroll
  for (int t = 0; t < kRowParts; ++t) {
    const f32x4 y = x[t] - mean;
    const float q = fmaf(y[0], y[0], y[1] * y[1]) + fmaf(y[2], y[2], y[3] * y[3]);
    v += 64 * t < d ? q : 0.f;
  }
  return float2{mean, 1.0f / sqrtf(sum16(v) / (float)d + kLnEps)};
}

__device__ __forceinline__ float normalised(float x, float2 st, float g, float b) {
  return fmaf((x - st.x) * st.y, g, b);
}

}  // namespace ad
