// Pieces shared by the kernels that solve for the pooled value in passes over a row or a list (row_search.hpp,
// wide_rows.hip): the order of the floats, and sums over the threads of a group.
#pragma once

#include "common.hpp"
#include "wave.hpp"

namespace topk {

// largest float strictly below T / smallest float strictly above T
__device__ __forceinline__ float float_next_down(float f) {
  const uint32_t b = __float_as_uint(f);
  if ((b << 1) == 0u) return __uint_as_float(0x80000001u);
  return __uint_as_float((b >> 31) ? b + 1u : b - 1u);
}
__device__ __forceinline__ float float_next_up(float f) { return -float_next_down(-f); }
__device__ __forceinline__ float float_below(double T) {
  const float f = float(T);
  return double(f) >= T ? float_next_down(f) : f;
}
__device__ __forceinline__ float float_above(double T) {
  const float f = float(T);
  return double(f) <= T ? float_next_up(f) : f;
}

// floats in numeric order as unsigned words, and back (between the images of two numbers lie numbers only)
__device__ __forceinline__ uint32_t ordered_of(float f) {
  const uint32_t b = __float_as_uint(f);
  return (b >> 31) ? ~b : b | 0x80000000u;
}
__device__ __forceinline__ float float_of_ordered(uint32_t o) {
  return __uint_as_float((o >> 31) ? o & 0x7fffffffu : ~o);
}

// inclusive prefix sum over the lanes of a wavefront, and the total
__device__ __forceinline__ uint32_t wave_inclusive_scan(uint32_t v, uint32_t* total) {
  v += dpp_or0<0x111, 0xF>(v);
  v += dpp_or0<0x112, 0xF>(v);
  v += dpp_or0<0x114, 0xF>(v);
  v += dpp_or0<0x118, 0xF>(v);
  v += dpp_or0<0x142, 0xA>(v);
  v += dpp_or0<0x143, 0xC>(v);
  *total = uint32_t(__builtin_amdgcn_readlane(int(v), kWave - 1));
  return v;
}
__device__ __forceinline__ double wave_inclusive_scan(double v) {
  v += dpp_or0_f64<0x111, 0xF>(v);
  v += dpp_or0_f64<0x112, 0xF>(v);
  v += dpp_or0_f64<0x114, 0xF>(v);
  v += dpp_or0_f64<0x118, 0xF>(v);
  v += dpp_or0_f64<0x142, 0xA>(v);
  v += dpp_or0_f64<0x143, 0xC>(v);
  return v;
}
// smallest a, largest b of a wavefront (vacated lanes: their own value)
template <int CTRL, int ROWS>
__device__ __forceinline__ void wave_min_max_step(float& a, float& b) {
  const int ia = int(__float_as_uint(a)), ib = int(__float_as_uint(b));
  a = fminf(a, __uint_as_float(uint32_t(__builtin_amdgcn_update_dpp(ia, ia, CTRL, ROWS, 0xF, false))));
  b = fmaxf(b, __uint_as_float(uint32_t(__builtin_amdgcn_update_dpp(ib, ib, CTRL, ROWS, 0xF, false))));
}
__device__ __forceinline__ void wave_min_max(float& a, float& b) {
  wave_min_max_step<0x111, 0xF>(a, b);
  wave_min_max_step<0x112, 0xF>(a, b);
  wave_min_max_step<0x114, 0xF>(a, b);
  wave_min_max_step<0x118, 0xF>(a, b);
  wave_min_max_step<0x142, 0xA>(a, b);
  wave_min_max_step<0x143, 0xC>(a, b);
  a = uniform_f32(a, kWave - 1);
  b = uniform_f32(b, kWave - 1);
}

// Sums of up to six doubles per thread over a wavefront (NT = 64, no barriers) or a whole workgroup of NT threads, the
// same in every thread.  The wavefronts' partial results meet in LDS, in two buffers used in turn, so that one barrier per
// reduction suffices (a wavefront writes a buffer again only after the barrier of the reduction in between, which
// every reader of the buffer has reached).
template <int NT>
struct SumGroup {
  static constexpr int W = NT / kWave;
  double* buf;                // [2][W][6], LDS
  int turn = 0;

  template <int N>
  __device__ __forceinline__ void sum(double (&d)[N]) {
    static_assert(N <= 6 && (W == 1 || W == 16), "as laid out");
#pragma unroll
    for (int i = 0; i < N; ++i) d[i] = lanes_sum<kWave>(d[i]);
    if constexpr (W > 1) {
      const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
      double* b = buf + (turn & 1) * (W * 6);
      ++turn;
      if (lane == 0) {
#pragma unroll
        for (int i = 0; i < N; ++i) b[w * 6 + i] = d[i];
      }
      __syncthreads();
#pragma unroll
      for (int i = 0; i < N; ++i) d[i] = lanes_sum<W>(b[(lane & (W - 1)) * 6 + i]);
    }
  }
  // the same with two counts per thread, below 2^32 in all
  template <int N>
  __device__ __forceinline__ void sum_with_counts(double (&d)[N], uint32_t& c0, uint32_t& c1) {
    static_assert(N <= 4, "as laid out");
    c0 = lanes_sum<kWave>(c0);
    c1 = lanes_sum<kWave>(c1);
    if constexpr (W == 1) {
      sum(d);
    } else {
      double t[N + 2];
#pragma unroll
      for (int i = 0; i < N; ++i) t[i] = d[i];
      const bool first = (threadIdx.x & (kWave - 1)) == 0;   // (already summed over the wavefront)
      t[N] = first ? double(c0) : 0.0;
      t[N + 1] = first ? double(c1) : 0.0;
      sum(t);
#pragma unroll
      for (int i = 0; i < N; ++i) d[i] = t[i];
      c0 = uint32_t(t[N]);
      c1 = uint32_t(t[N + 1]);
    }
  }
  // smallest a, largest b of the group
  __device__ __forceinline__ void min_max(float& a, float& b) {
    wave_min_max(a, b);
    if constexpr (W > 1) {
      const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
      double* s = buf + (turn & 1) * (W * 6);
      ++turn;
      if (lane == 0) {
        s[w * 6] = double(a);
        s[w * 6 + 1] = double(b);
      }
      __syncthreads();
      a = float(s[(lane & (W - 1)) * 6]);
      b = float(s[(lane & (W - 1)) * 6 + 1]);
      wave_min_max(a, b);
    }
  }
};

}  // namespace topk
