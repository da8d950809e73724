// Cube roots and the singleton solution of the magnitude operator with p = 4/3, for kernels that need one per element.
#pragma once

#include "common.hpp"
#include "pooling.hpp"

namespace topk {

__device__ __forceinline__ float cbrt_approx(float v) {      // v > 0; a starting point only
  return __builtin_amdgcn_exp2f(__builtin_amdgcn_logf(v) * (1.0f / 3.0f));
}

// cube root of a positive double to rounding: float32 start (1e-6), two Newton steps whose quotients are
// small corrections
__device__ __forceinline__ double cbrt_f64(double v) {
  const float f = float(v);
  if (!(f > 1e-36f)) return cbrt(fmax(v, 0.0));
  float c32 = cbrt_approx(f);
  const float third = __builtin_amdgcn_rcpf(3.0f * c32 * c32);
  double c = double(c32);
  c -= double(float(c * c * c - v) * third);
  c -= double(float(c * c * c - v) * third);
  return c;
}

// y and dy/dtau of a top-k element s > 0 above the block for the magnitude operator with p = 4/3: the
// root g of (g - s)^3 + lambda^3 g = 0.  With g = s - lambda w it is w^3 + lambda w = s and g = w^3.
// float32 Halley steps from the upper bound min(s / lambda, s^(1/3)) bring w to float32 precision (the
// function is convex there: two steps bring any start, off by 47 % at most, to 5e-7), STEPS float64 Newton
// steps to 3e-13 and to rounding (g within 5e-13, resp. 7e-16 of itself for s = 1e-6 .. 3.4e38 and lambda = 1e-37 ..
// 1e38; with one step the nearest float32 is missed once in 10^6); their quotients are small corrections, for which
// float32 precision is enough.  No intermediate value exceeds s, so that the largest floats are in range.  Two steps
// in long rows, which are as exact as the safeguarded float64 solve of pooling.hpp (some 150 instructions per
// element) then, at no cost (1 x 16.7 M: bound by memory); one in rows held in registers (4096 x 4096, k = 410: 75.7 us,
// 76.0 with two).
template <int STEPS>
__device__ __forceinline__ void above_mag43(double s, const Reg& R, bool want_slope, double* g, double* slope) {
  const float s32 = float(s), l32 = float(R.lambda);
  float w = fminf(s32 * float(R.inv_lambda), cbrt_approx(s32));
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const float rD = __builtin_amdgcn_rcpf(fmaf(3.0f * w, w, l32));
    const float step = fmaf(w, fmaf(w, w, l32), -s32) * rD;
    w -= step * __builtin_amdgcn_rcpf(1.0f - 3.0f * w * rD * step);
  }
  double wd = double(w);
  if (!(R.lambda < 1e38)) {                            // (no float32: w^3 is nothing beside lambda w)
    w = 0.0f;
    wd = s * R.inv_lambda;
  }
  const float rD = __builtin_amdgcn_rcpf(fmaf(3.0f * w, w, l32));
#pragma unroll
  for (int it = 0; it < STEPS; ++it) wd -= double(float(fma(wd, fma(wd, wd, R.lambda), -s)) * rD);
  const double u = R.lambda * wd;
  *g = u > 0.75 * s ? wd * wd * wd : s - u;            // (without cancellation either way)
  if (want_slope) {
    const double a = 3.0 * wd * wd, b = a + R.lambda;
    double r = double(__builtin_amdgcn_rcpf(float(b)));
    r = fma(fma(-b, r, 1.0), r, r);
    *slope = a * fma(fma(-b, r, 1.0), r, r);
  }
}

// A wavefront's elements above the block, packed: `list` (LDS, kPackMax entries) holds `total` pairs (value, tangent) and
// gets (output for the value's magnitude, its tangent).  A cubic takes some 80 vector instructions, and done where
// the elements are, a wavefront does one for every element as soon as one lane holds one.  Forward + VJP, where they are /
// packed: 4096 x 4096, k = 410 88.3 / 75.3 us, k = 1365 91.6 / 83.7; 1 x 16.7 M, k = n / 10 (whose dense pass took the
// safeguarded float64 solve of pooling.hpp) 277 / 130.
constexpr uint32_t kPackMax = 256;
template <int STEPS>
__device__ __forceinline__ void packed_above_mag43(float2* list, uint32_t total, const Reg& R, bool want_slope) {
  __builtin_amdgcn_wave_barrier();
#pragma unroll 1
  for (uint32_t j = threadIdx.x & (kWave - 1); j < total; j += kWave) {
    const float2 q = list[j];
    double g, slope = 0.0;
    above_mag43<STEPS>(double(q.x), R, want_slope, &g, &slope);
    list[j] = make_float2(float(g), want_slope ? float(slope * double(q.y)) : 0.0f);
  }
  __builtin_amdgcn_wave_barrier();
}

}  // namespace topk
