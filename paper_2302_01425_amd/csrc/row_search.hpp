// Rows held in registers, dense outputs, WITHOUT any sort: one row per group of NT threads (a
// wavefront, or a whole workgroup), E elements per thread.
//
// The outputs depend on the row only through the pooled value gamma of the one block that
// pool-adjacent-violators grows around positions k, k+1 (App. "PAV algorithm" with w = 1_k), and the
// block is an interval of values: an element belongs to it iff its singleton minimiser as a top-k
// position lies below gamma and its value above gamma.  So gamma is the root of a function that
// never rises,
//     Psi(g) = sum_i clip((s_i - g) h(g), 0, 1)^(q-1) - k,
//         h = 1 / lambda (mask),  1 / (lambda g) (magnitude, p = 2),  1 / (lambda g^(1/3)) (p = 4/3),
// which is sum_i grad r*(s_i - v_i) = k: the elements above the block count 1, those below 0, those
// inside their output.  The row stays in registers and every evaluation is a handful of
// instructions per element and one reduction over the group:
//
//   1. a first guess from order statistics: the maxima of 1, 8 or all elements of a lane are sorted 16
//      at a time; the quantile of those maxima that corresponds to rank k estimates s_k;
//   2. bracketed secant steps on Psi in float32 (2 to 5 on normal values, sixteen at most; no
//      derivative: an evaluation is a subtraction, a clamped product and an addition per element):
//      they only have to come near the root.  Rows of few different values, on which Psi jumps, go
//      on from s_k (5) as soon as the bracket holds one value;
//   3. the elements within a third of the block's width of the block at g go to a list in LDS;
//   4. exact steps on the list: the members of the block at g are counted and their power sums taken in
//      float64, the pooled value of that set is the next g (the root of the piece of Psi that g lies
//      on); when the set no longer changes the value is final.  The membership thresholds are floats,
//      so a set is described by two counts.  (Lists that do not fit, and steps that leave the list's
//      window, take passes over the registers instead.)
//   5. where the steps above did not come to a value: s_k by bisection over the floats in their order,
//      then the set of the block from the pair (s_k, s_{k+1}) on, in passes over the registers whose
//      number is bounded whatever the values.  And where a threshold lies within rounding of an
//      element's value, that element would be a tie of the strict tests: the block is grown from the
//      elements that certainly belong to it with the strict tests of the PAV loop themselves
//      (pooling.hpp), one neighbouring value per step.  The decisions are the same as those of the
//      kernels that order the row.
//
// The kernels that order values need (log n)^2 / 2 exchanges per element; a step here costs 5 to 8
// instructions per element.
#pragma once

#include <type_traits>

#include "common.hpp"
#include "cubic.hpp"
#include "group.hpp"
#include "pooling.hpp"
#include "launch.hpp"
#include "wave.hpp"

namespace topk {
namespace {

constexpr int kSearchPlain = 0, kSearchSigned = 1, kSearchMasked = 2, kSearchLoss = 3;

// What the group reduces.  NT > 64: the wavefronts' partial results meet in LDS, in two buffers used
// in turn, so that one barrier per reduction suffices (a wavefront writes a buffer again only after
// the barrier of the reduction in between, which every reader of the buffer has reached).
struct SearchRed {
  double d[3];
  float f[2];
  uint32_t c;
};
template <int NT>
struct SearchGroup {
  static constexpr int W = NT / kWave;
  SearchRed* buf;             // [2][W], LDS
  int turn = 0;

  // sums over the threads of the group, the same in every thread: ND doubles, NF floats, NC (0 or 1)
  // word
  template <int ND, int NF, int NC>
  __device__ __forceinline__ void sum(double* d, float* f, uint32_t* c) {
#pragma unroll
    for (int i = 0; i < ND; ++i) d[i] = lanes_sum<kWave>(d[i]);
#pragma unroll
    for (int i = 0; i < NF; ++i) f[i] = lanes_sum<kWave>(f[i]);
    if (NC) *c = lanes_sum<kWave>(*c);
    if constexpr (W > 1) {
      const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
      SearchRed* b = buf + (turn & 1) * W;
      ++turn;
      if (lane == 0) {
#pragma unroll
        for (int i = 0; i < ND; ++i) b[w].d[i] = d[i];
#pragma unroll
        for (int i = 0; i < NF; ++i) b[w].f[i] = f[i];
        if (NC) b[w].c = *c;
      }
      __syncthreads();
      const SearchRed& o = b[lane & (W - 1)];
#pragma unroll
      for (int i = 0; i < ND; ++i) d[i] = lanes_sum<W>(o.d[i]);
#pragma unroll
      for (int i = 0; i < NF; ++i) f[i] = lanes_sum<W>(o.f[i]);
      if (NC) *c = lanes_sum<W>(o.c);
    }
  }
  // inclusive prefix sum over the threads of the group, and the total
  __device__ __forceinline__ uint32_t scan(uint32_t v, uint32_t* total) {
    uint32_t all;
    v = wave_inclusive_scan(v, &all);
    if constexpr (W > 1) {
      const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
      SearchRed* b = buf + (turn & 1) * W;
      ++turn;
      if (lane == 0) b[w].c = all;
      __syncthreads();
      const uint32_t o = b[lane & (W - 1)].c;
      v += lanes_sum<W>((lane & (W - 1)) < w ? o : 0u);
      all = lanes_sum<W>(o);
    }
    *total = all;
    return v;
  }
  // two counts of up to 32768 elements each, in one word
  __device__ __forceinline__ void sum_counts(uint32_t* a, uint32_t* b) {
    uint32_t c = *a | (*b << 16);
    sum<0, 0, 1>(nullptr, nullptr, &c);
    *a = c & 0xffffu;
    *b = c >> 16;
  }
  // smallest a, largest b of the group
  __device__ __forceinline__ void min_max(float& a, float& b) {
    wave_min_max(a, b);
    if constexpr (W > 1) {
      const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
      SearchRed* s = buf + (turn & 1) * W;
      ++turn;
      if (lane == 0) {
        s[w].f[0] = a;
        s[w].f[1] = b;
      }
      __syncthreads();
#pragma unroll
      for (int q = 0; q < W; ++q) {
        a = fminf(a, s[q].f[0]);
        b = fmaxf(b, s[q].f[1]);
      }
    }
    a = uniform_f32(a, 0);
    b = uniform_f32(b, 0);
  }
};

// Makes a value opaque to the compiler.  The thresholds of every pass over the registers are, so that
// the comparisons of one pass are not kept (two SGPRs each) for all E elements until the next; and
// after every fourth element the accumulators are, so that the terms of at most four elements are in
// flight (compare masks, float64 temporaries).  Without it the kernels spill.
template <class T>
__device__ __forceinline__ void opaque(T& v) {
  asm volatile("" : "+v"(v));
}
__device__ __forceinline__ void pass_fence(int) {}
template <class T, class... Rest>
__device__ __forceinline__ void pass_fence(int r, T& a, Rest&... rest) {
  if ((r & 3) == 3) {
    opaque(a);
    pass_fence(r, rest...);
  }
}

// 16 values per DPP row of lanes, in descending order of the row's lanes (bitonic network, mirror form)
template <int LM>
__device__ __forceinline__ float sort16_stage(float v, int lane) {
  const float o = __uint_as_float(lane_xor<LM>(__float_as_uint(v)));
  return (lane & top_bit(LM)) == 0 ? fmaxf(v, o) : fminf(v, o);
}
__device__ __forceinline__ float sort16_desc(float v, int lane) {
  v = sort16_stage<1>(v, lane);
  v = sort16_stage<3>(v, lane);
  v = sort16_stage<1>(v, lane);
  v = sort16_stage<7>(v, lane);
  v = sort16_stage<2>(v, lane);
  v = sort16_stage<1>(v, lane);
  v = sort16_stage<15>(v, lane);
  v = sort16_stage<4>(v, lane);
  v = sort16_stage<2>(v, lane);
  v = sort16_stage<1>(v, lane);
  return v;
}
// mean over the first `rows` (uniform, 1 .. 4) DPP rows of the value in lane i of each
__device__ __forceinline__ float rows_mean(float v, int i, int rows) {
  float t = uniform_f32(v, i);
  if (rows >= 4) return 0.25f * ((t + uniform_f32(v, 16 + i)) + (uniform_f32(v, 32 + i) + uniform_f32(v, 48 + i)));
  if (rows >= 2) t += uniform_f32(v, 16 + i);
  if (rows >= 3) t += uniform_f32(v, 32 + i);
  return rows >= 3 ? t * (1.0f / 3.0f) : (rows == 2 ? 0.5f * t : t);
}
// NT threads per row (64: four rows per workgroup of 256 threads, no barriers; more: one row per
// workgroup), at most E elements per thread.  VAR as in short_rows_value.hpp (the operators built on
// the mask, MAG = false).  Any of out / jvp may be null for the plain operators.  vec: x, tangent, out
// and jvp have the same address modulo 16 bytes.
template <int NT, int E, bool MAG, int PC, int VAR>
__global__ __launch_bounds__(NT == 64 ? 256 : NT) void row_search_kernel(
    const float* __restrict__ x_all, const float* __restrict__ tangent_all, float* __restrict__ out_all,
    float* __restrict__ jvp_all, int64_t rows, int n, int k, Reg R, bool vec,
    float* __restrict__ loss, double lam_over_p) {
  static_assert(VAR == kSearchPlain || !MAG, "the variants are built on the mask");
  static_assert(E % 4 == 0, "elements are dealt four by four");
  using P = Pool<MAG, PC>;
  constexpr bool CUBIC = (PC == kP43);
  constexpr bool ABS = MAG || VAR == kSearchSigned || VAR == kSearchMasked;
  constexpr bool LOSS = VAR == kSearchLoss;
  // the mask's JVP needs the tangent of the block's elements only: it goes through the list
  constexpr bool LIST_TAU = !MAG && VAR == kSearchPlain;
  constexpr int W = NT / kWave, RPB = NT == 64 ? 4 : 1, Q = E / 4;
  static_assert(W == 1 || RPB == 1, "a workgroup holds one row, or one row per wavefront");
  __shared__ SearchRed red[W > 1 ? 2 * W : 1];
  __shared__ struct {
    double gamma, cnt, m;
    float lo, hi;
    int flags;
  } found;
  constexpr int kListMax = NT * 4;                     // list entries of a row
  __shared__ float2 lists[RPB][kListMax];              // (value, index and sign)
  SearchGroup<NT> grp{red};
  constexpr int kSecantMax = 16;                       // steps of phase 2; then the root is found from s_k

  const int lane = threadIdx.x & (kWave - 1);
  const int tid = NT == 64 ? lane : int(threadIdx.x);              // thread of the group
  const int64_t row = int64_t(blockIdx.x) * RPB + (RPB > 1 ? int(threadIdx.x) / NT : 0);
  if (row >= rows) return;
  const int64_t base = row * n;
  const float* x = x_all + base;
  const float* tangent = tangent_all != nullptr ? tangent_all + base : nullptr;
  float* out = out_all != nullptr ? out_all + base : nullptr;
  float* jvp = jvp_all != nullptr ? jvp_all + base : nullptr;
  const bool want_jvp = jvp != nullptr;

  // The row as 16-byte groups at their natural alignment: group j = elements 4 j - shift .. + 3.
  // Groups that stick out of the row (its first and last) are accessed element by element.
  const int shift = int((reinterpret_cast<uintptr_t>(x) >> 2) & 3u);
  // (opaque, so that the bounds tests of all groups are made where they are used and not kept)
  auto first_of = [&](int c) {
    int e = (c * NT + tid) * 4 - shift;
    opaque(e);
    return e;
  };
  auto load_group = [&](const float* p, int c, float fill, float* v) {
    const int e = first_of(c);
    if (vec && e >= 0 && e + 4 <= n) {
      const float4 q = load4_stream(p + e);
      v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) v[r] = (e + r >= 0 && e + r < n) ? p[e + r] : fill;
    }
  };
  auto store_group = [&](float* p, int c, const float* v) {
    const int e = first_of(c);
    if (vec && e >= 0 && e + 4 <= n) {
      store4_stream(p + e, make_float4(v[0], v[1], v[2], v[3]));
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (e + r >= 0 && e + r < n) p[e + r] = v[r];
    }
  };

  // padding is NaN: every comparison with it is false
  const float nan = __uint_as_float(0x7fc00000u);
  float xr[E];
#pragma unroll
  for (int c = 0; c < Q; ++c) load_group(x, c, nan, xr + 4 * c);
  auto val = [&](int r) { return ABS ? fabsf(xr[r]) : xr[r]; };

  // ---- the block: members lo_f <= value <= hi_f, everything above hi_f is before it -----------------
  const float inf = __uint_as_float(0x7f800000u);
  float hi_f = k <= 0 ? inf : -inf, lo_f = inf;        // (k = 0: all below; k = n: all above)
  bool have = false;
  double gamma = 0.0, center = 0.0, cnt = 0.0, m = 0.0;

  // elements above hi, and elements from lo to hi
  auto count_pass = [&](float lo, float hi, uint32_t* above, uint32_t* members) {
    opaque(lo);
    opaque(hi);
    uint32_t c0 = 0u, c1 = 0u;
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const float v = val(r);
      c0 += v > hi ? 1u : 0u;
      c1 += v >= lo ? 1u : 0u;
      pass_fence(r, c0, c1);
    }
    grp.sum_counts(&c0, &c1);
    *above = c0;
    *members = c1 > c0 ? c1 - c0 : 0u;
  };
  // the same with the power sums of the members' values relative to c32 = center
  auto sums_pass = [&](float lo, float hi, float c32, uint32_t* above, uint32_t* members) -> Sums {
    double d[3] = {0.0, 0.0, 0.0};
    uint32_t c0 = 0u, c1 = 0u;
    opaque(lo);
    opaque(hi);
#pragma unroll
    for (int r = 0; r < E; ++r) {
      float v = val(r);
      opaque(v);                                       // (its conversion is not to be kept for all E)
      const bool ab = v > hi, ge = v >= lo;
      c0 += ab ? 1u : 0u;
      c1 += ge ? 1u : 0u;
      if (__any(ge && !ab)) {                          // (short blocks: few wavefronts hold a member)
        const double t = double((ge && !ab) ? v : c32) - double(c32);
        d[0] += t;
        if (CUBIC) {
          const double t2 = t * t;
          d[1] += t2;
          d[2] = fma(t2, t, d[2]);
        }
      }
      pass_fence(r, c0, c1);
    }
    uint32_t c = c0 | (c1 << 16);
    grp.template sum<CUBIC ? 3 : 1, 0, 1>(d, nullptr, &c);
    c0 = c & 0xffffu;
    c1 = c >> 16;
    *above = c0;
    *members = c1 > c0 ? c1 - c0 : 0u;
    return Sums{d[0], d[1], d[2]};
  };
  // the neighbouring values of [lo, hi]: smallest above, largest below
  auto neighbours = [&](float lo, float hi, float* above, float* below) {
    float a = inf, b = -inf;
    opaque(lo);
    opaque(hi);
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const float v = val(r);
      a = fminf(a, v > hi ? v : inf);
      b = fmaxf(b, v < lo ? v : -inf);
      pass_fence(r, a, b);
    }
    grp.min_max(a, b);
    *above = a;
    *below = b;
  };
  // pooled value of a set; the cubic by Newton from x0 (nearly the root), falling back to the
  // safeguarded solve
  auto pooled_of = [&](const Sums& S, double cn, double mm, double x0, double dmin, double dmax) -> double {
    if (!CUBIC) return P::pooled(cn, mm, S, R, 0.0, 0.0, 0.0);
    double g = x0;
    const double tol = 1e-13 * R.lambda;
#pragma unroll 1
    for (int it = 0; it < 8; ++it) {
      const double F = P::cubic(g, cn, mm, S, R, center);
      const double D = (3.0 * cn * g - 6.0 * S.s1) * g + 3.0 * S.s2 + (MAG ? R.lam3 * mm : 0.0);
      const double step = F * double(__builtin_amdgcn_rcpf(float(D)));   // (1e-7 off: one more step at most)
      const double next = g - step;
      if (!(next >= dmin && next <= dmax)) break;      // (also NaN)
      g = next;
      if (fabs(step) <= tol) return g;
    }
    return P::pooled(cn, mm, S, R, dmin, dmax, center);
  };

  bool use_list = false;
  uint32_t len = 0u, list_at = 0u;                     // of the list; where this thread's elements start
  float list_mid = 0.0f, list_half = -1.0f;            // its window
  const bool solve = k >= 1 && k < n;
  bool done = !solve;
  const float lam = float(R.lambda), il = float(R.inv_lambda);
  float g = 0.0f;
  float w_lo = MAG ? 0.0f : -inf, w_hi = inf;          // the root lies in between
  bool below = false, above = false;                   // the signs of Psi at w_lo and w_hi have been seen
  bool near = false;                                   // g is next to the root
  float spare = 0.3f;                                  // block widths that g may be off
  auto width_at = [&](float at) { return !MAG ? lam : (CUBIC ? lam * cbrt_approx(at) : lam * at); };
  if (!done) {
    // ---- 1. a guess of s_k, and of the number of elements per unit of value around it ------------
    // Of maxima over `mm` elements each (one per lane), a share 1 - (1 - q)^mm lies above the quantile of level
    // q = k / n; mm is chosen so that this share is neither near 0 nor near 1.
    float dens;
    {
      const float q_all = float(k) / float(NT * E), q_n = float(k) / float(n);
      float mx = val(0), share = q_n, per = float(n);  // per: elements per unit of share
      float f[2] = {0.0f, 0.0f};
      int below_r;                                     // ranks between the two values of f[1]
      if (n < 4 * NT) {
        // (one group of four per thread, and none in the last threads)
        if (q_n < 0.375f) {
#pragma unroll
          for (int r = 1; r < 4; ++r) mx = fmaxf(mx, val(r));
          const float rest = __builtin_amdgcn_exp2f(3.0f * __builtin_amdgcn_logf(1.0f - q_n));
          share = 1.0f - rest * (1.0f - q_n);
          per = float(n) * 0.25f * __builtin_amdgcn_rcpf(rest);
        }
      } else if (q_all * float(E) < 2.0f) {
#pragma unroll
        for (int r = 1; r < E; ++r) mx = fmaxf(mx, val(r));
        const float rest = __builtin_amdgcn_exp2f(float(E - 1) * __builtin_amdgcn_logf(1.0f - q_all));
        share = 1.0f - rest * (1.0f - q_all);
        per = float(NT) * __builtin_amdgcn_rcpf(rest);
      } else if (E >= 8 && q_n * 8.0f < 3.0f && n >= 8 * NT) {
#pragma unroll
        for (int r = 1; r < (E < 8 ? E : 8); ++r) mx = fmaxf(mx, val(r));
        const float rest = __builtin_amdgcn_exp2f(7.0f * __builtin_amdgcn_logf(1.0f - q_n));
        share = 1.0f - rest * (1.0f - q_n);
        per = float(n) * 0.125f * __builtin_amdgcn_rcpf(rest);
      }
      float r = share * 16.0f - 0.5f;
      r = fminf(fmaxf(r, 0.0f), 15.0f);
      const int i0 = __builtin_amdgcn_readfirstlane(int(r));
      const int j0 = i0 > 1 ? i0 - 1 : 0, j1 = i0 < 14 ? i0 + 2 : 15;
      below_r = j1 - j0;
      constexpr int kSampling = W < 4 ? W : 4;         // wavefronts that take part
      // every row of 16 lanes estimates the quantile, and the mean of the estimates is taken; in rows of fewer
      // than 4 NT elements those whose lanes all hold four elements
      const int full = n >= 4 * NT ? 4 * kSampling : (n + shift) / 64;
      int mine = 4;
      if (n < 4 * NT) mine = min(4, full - (W > 1 ? 4 * __builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave) : 0));
      if (mine > 0 && (W <= 4 || threadIdx.x < kSampling * kWave || n < 4 * NT)) {
        mx = fmaxf(mx, -3.0e38f);                      // (NaN padding)
        mx = sort16_desc(mx, lane);
        const float a = rows_mean(mx, i0, mine), b = rows_mean(mx, i0 < 15 ? i0 + 1 : 15, mine);
        const float far = rows_mean(mx, j1, mine), last = far > -1.0e37f ? far : a;
        f[0] = b > -1.0e37f ? a + (b - a) * (r - float(i0)) : a;
        f[1] = rows_mean(mx, j0, mine) - last;
      }
      if constexpr (W > 1) {
        const float part = n >= 4 * NT ? 1.0f / kSampling : float(mine) * __builtin_amdgcn_rcpf(float(full));
        f[0] = (lane == 0 && mine > 0) ? f[0] * part : 0.0f;       // (zero in wavefronts that have no part)
        f[1] = (lane == 0 && mine > 0) ? f[1] * part : 0.0f;
        grp.template sum<0, 2, 0>(nullptr, f, nullptr);
      }
      g = f[0];
      dens = per * float(below_r) * (1.0f / 16.0f) * __builtin_amdgcn_rcpf(fmaxf(f[1], fabsf(g) * 1e-6f + 1e-37f));
    }
    // from s_k to gamma: about half of the way down to the singleton minimiser of s_k (p = 4/3: the
    // cubic outputs put it at three quarters)
    constexpr float kPart = CUBIC ? 0.75f : 0.5f;
    if (!MAG) g -= kPart * lam;
    else {
      g = fmaxf(g, 1e-37f);
      if (!CUBIC) g *= 1.0f - kPart * lam / (1.0f + lam);
      else g = fmaxf(g - kPart * lam * cbrt_approx(g), 0.1f * g);
    }
    // ---- 2. secant steps on Psi, float32 ----------------------------------------------------------------
    {
      float f_lo = 0.0f, f_hi = 0.0f, g_old = g, f_old = 0.0f;
      int side = 0;
      const float kf = float(k);
      dens = fminf(dens, float(n) * __builtin_amdgcn_rcpf(width_at(g)));        // (no block holds more than the row)
#pragma unroll 1
      for (int it = 0; it < kSecantMax; ++it) {
        const float width = width_at(g);
        const float h = !MAG ? il : __builtin_amdgcn_rcpf(width);
        float f[1] = {0.0f};
#pragma unroll
        for (int r = 0; r < E; ++r) {
          const float t = __builtin_amdgcn_fmed3f((val(r) - g) * h, 0.0f, 1.0f);
          if (CUBIC) f[0] = fmaf(t * t, t, f[0]);
          else f[0] += t;
          pass_fence(r, f[0]);
        }
        grp.template sum<0, 1, 0>(nullptr, f, nullptr);
        const float F = f[0] - kf, in_width = dens * width;
        // near enough: the exact steps converge from a distance of some hundredths of a block
        if (!(fabsf(F) > fmaxf(0.3f, 0.01f * in_width))) {
          near = F == F;
          break;
        }
        const float slope = (f_old - F) * __builtin_amdgcn_rcpf(g - g_old);
        if (it > 0 && slope > 0.0f && slope < inf) dens = slope;
        // (an end that stays while the other one moves twice counts half: Illinois)
        if (F > 0.0f) {
          w_lo = g;
          f_lo = F;
          if (side == 1) f_hi *= 0.5f;
          side = 1;
          below = true;
        } else {
          w_hi = g;
          f_hi = F;
          if (side == -1) f_lo *= 0.5f;
          side = -1;
          above = true;
        }
        g_old = g;
        f_old = F;
        float next;
        if (below && above) {
          float wgt = f_lo * __builtin_amdgcn_rcpf(f_lo - f_hi);
          wgt = fminf(fmaxf(wgt, 0.05f), 0.95f);
          next = w_lo + (w_hi - w_lo) * wgt;
        } else {
          next = g + F * __builtin_amdgcn_rcpf(dens);
          if (MAG) next = fmaxf(next, 0.25f * g);
          if (it > 1) dens *= 0.5f;                    // (further each time, until the root is passed)
        }
        if (!(next > w_lo && next < w_hi) || next == g) {          // (the bracket is used up; NaN)
          near = below && above;
          break;
        }
        g = next;
        if (it == kSecantMax / 2 - 1 && below && above) {
          // (rows of few different values: Psi jumps.)  One value left: it is s_k
          float first, last;
          neighbours(float_next_up(w_hi + 1.01f * width), float_next_down(w_lo), &first, &last);
          if (!(first < last)) break;
        }
        if (MAG && !below && it == 2) {
          // (the root far below the guess: perhaps at zero.)  s_{k+1} = 0: nothing pools, and the top k
          // are the positive values and some zeros
          uint32_t pos, dummy;
          count_pass(inf, 0.0f, &pos, &dummy);
          if (int(pos) <= k) {
            hi_f = 0.0f;
            done = true;
            break;
          }
        }
      }
      if (dens * width_at(g) < 6.0f) spare = 1.2f;
      // (uniform values that live on, out of the vector registers)
      spare = uniform_f32(spare, 0);
      g = uniform_f32(g, 0);
      w_lo = uniform_f32(w_lo, 0);
      w_hi = uniform_f32(w_hi, 0);
    }
  }
  // the elements within `half` of `mid` go to the list, if they fit; the number of those above them
  uint32_t above_list = 0u;
  float2* list = lists[RPB > 1 ? int(threadIdx.x) / NT : 0];
  auto gather = [&](float mid, float half) __attribute__((always_inline)) {
    uint32_t c0 = 0u, c1 = 0u;
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const float t = val(r) - mid;
      c0 += fabsf(t) <= half ? 1u : 0u;
      c1 += t > half ? 1u : 0u;
      pass_fence(r, c0, c1);
    }
    uint32_t total, c = c0 | (c1 << 16);
    uint32_t at = (grp.scan(c, &total) & 0xffffu) - c0;
    list_at = at;
    list_mid = mid;
    list_half = half;
    len = total & 0xffffu;
    above_list = total >> 16;
    if (len <= uint32_t(kListMax)) {
#pragma unroll
      for (int r = 0; r < E; ++r) {
        const float v = val(r);
        if (fabsf(v - mid) <= half) {
          const uint32_t e = uint32_t(((r >> 2) * NT + tid) * 4 - shift + (r & 3));
          list[at] = make_float2(v, __uint_as_float(e | (__float_as_uint(xr[r]) & 0x80000000u)));
          ++at;
        }
        pass_fence(r, at);
      }
    }
    if constexpr (W > 1) __syncthreads();
    else __builtin_amdgcn_wave_barrier();
  };
  if (!done) {
    // ---- 3. the list of the elements that may belong to the block ----------------------------------------
    // (with 0.3 of a block's width to spare on either side, or more where a width holds but a few elements:
    // then a root may be that far from a value of Psi below 0.3; the last term is for blocks narrower than
    // the spacing of floats)
    const float width_g = width_at(g), mid = g + 0.5f * width_g;
    const float half = (0.5f + spare) * width_g + 5e-7f * fabsf(mid);
    if (near) gather(mid, half);
    use_list = near && len <= uint32_t(kListMax);
    auto list_pass = [&](auto& G, int first, int step, float lo, float hi, float c32, uint32_t* above,
                         uint32_t* members) -> Sums {
      double d[3] = {0.0, 0.0, 0.0};
      uint32_t c0 = 0u, c1 = 0u;
#pragma unroll 1
      for (uint32_t j = first; j < len; j += step) {
        const float v = list[j].x;
        const bool ab = v > hi, in = v >= lo && !ab;
        c0 += ab ? 1u : 0u;
        c1 += in ? 1u : 0u;
        const double t = double(in ? v : c32) - double(c32);
        d[0] += t;
        if (CUBIC) {
          const double t2 = t * t;
          d[1] += t2;
          d[2] = fma(t2, t, d[2]);
        }
      }
      uint32_t c = c0 | (c1 << 16);
      G.template sum<CUBIC ? 3 : 1, 0, 1>(d, nullptr, &c);
      *above = (c & 0xffffu) + above_list;
      *members = c >> 16;
      return Sums{d[0], d[1], d[2]};
    };
    // ---- 4. exact steps ------------------------------------------------------------------------------------
    float c32 = P::kCentered ? g : 0.0f;
    center = uniform_f64(double(c32), 0);
    gamma = double(g) - center;
    auto upper_end = [&](double ga) -> double {        // values below it are below their cap at gamma
      if (!MAG) return ga + R.lambda;
      if (!CUBIC) return ga * R.one_p_lambda;
      return ga + R.lambda * cbrt_f64(ga);
    };
    // rounding of a threshold (magnitude, p = 2: relative; else lambda takes part in its sums)
    auto slack_of = [&](double t) -> double { return (CUBIC ? 1e-11 : 1e-12) * (fabs(t) + (MAG && !CUBIC ? 0.0 : R.lambda)); };
    bool grow = true;                                  // the growth with the strict tests is needed
    // does an element lie within rounding of one of the two thresholds?  (Not only the float next to it: around
    // zero there are many.)
    auto at_a_tie = [&](auto& G, auto solo, int first, int step, double ga, double t_hi) -> bool {
      constexpr bool SOLO = decltype(solo)::value;
      const double s1 = slack_of(ga), s2 = slack_of(t_hi);
      if (!(fabs(double(float(ga)) - ga) <= s1) && !(fabs(double(float(t_hi)) - t_hi) <= s2)) return false;   // (mostly)
      const float a1 = float_above(ga - s1), b1 = float_below(ga + s1);
      const float a2 = float_above(t_hi - s2), b2 = float_below(t_hi + s2);
      uint32_t c = 0u;
      if (SOLO || use_list) {                          // (the thresholds lie inside the list's window)
#pragma unroll 1
        for (uint32_t j = first; j < len; j += step) {
          const float v = list[j].x;
          c += ((v >= a1 && v <= b1) || (v >= a2 && v <= b2)) ? 1u : 0u;
        }
      } else if constexpr (!SOLO) {
#pragma unroll
        for (int r = 0; r < E; ++r) {
          float v = val(r);
          opaque(v);
          c += ((v >= a1 && v <= b1) || (v >= a2 && v <= b2)) ? 1u : 0u;
          pass_fence(r, c);
        }
      }
      G.template sum<0, 0, 1>(nullptr, nullptr, &c);
      return c != 0u;
    };
    // While the list is used the steps stay inside its window; a root that turns out to lie outside, or
    // that some twenty passes over the registers do not reach, is found from s_k below.
    const float soft = (spare - 0.05f) * width_g + 2e-7f * fabsf(g);
    // The steps, by the group G whose threads are first, first + step, ..  SOLO: one wavefront on the
    // list alone; it returns false, with gamma as far as it came, when the registers are needed.
    auto exact_steps = [&](auto& G, auto solo, int first, int step) -> bool {
      constexpr bool SOLO = decltype(solo)::value;
      double blo = use_list ? double(g - soft) - center : -1e300, bhi = use_list ? double(g + soft) - center : 1e300;
      bool settled = false, lo_seen = false, hi_seen = false;        // (signs of Psi at blo and bhi)
      uint32_t ab = 0xffffffffu, cn = 0xffffffffu;
#pragma unroll 1
      for (int it = 0; it < (use_list ? 32 : 20); ++it) {
        const double ga = gamma + center;
        const double t_hi = upper_end(ga);
        lo_f = float_above(ga);
        hi_f = float_below(t_hi);
        uint32_t na, nc;
        Sums S{0.0, 0.0, 0.0};
        // (elements equal to the ends of the list's window may be outside it)
        use_list = use_list && lo_f > mid - 0.99f * half && hi_f < mid + 0.99f * half;
        if (SOLO || use_list) {
          if (!use_list) return false;
          S = list_pass(G, first, step, lo_f, hi_f, c32, &na, &nc);
        } else if constexpr (!SOLO) {
          if (it > 0) count_pass(lo_f, hi_f, &na, &nc);
        }
        if (it > 0 && (settled || (na == ab && nc == cn))) {       // gamma is the pooled value of its own set
          grow = at_a_tie(G, solo, first, step, ga, t_hi);
          have = true;
          return true;
        }
        if constexpr (!SOLO) {
          if (!use_list) S = sums_pass(lo_f, hi_f, c32, &na, &nc);
        }
        ab = na;
        cn = nc;
        double next = gamma;
        bool ok = false, leave = false;                // next is a pooled value inside the bracket; a pooled value
        if (cn == 0u) {
          if (int(ab) == k) {                          // Psi = 0 on an empty set: nothing pools
            grow = at_a_tie(G, solo, first, step, ga, t_hi);
            return true;
          }
          if (int(ab) > k) {
            blo = gamma;
            lo_seen = true;
          } else {
            bhi = gamma;
            hi_seen = true;
          }
        } else {
          cnt = double(cn);
          m = double(k) - double(ab);
          const double dlo = double(lo_f) - center, dhi = double(hi_f) - center;
          // the cubic's root lies above (smallest member - lambda), resp. 0, and below the largest member
          if (!(m > 0.0)) {
            blo = gamma;                               // (k or more elements above)
            lo_seen = true;
          } else if (m > cnt) {
            bhi = gamma;                               // (fewer than k elements that far)
            hi_seen = true;
          } else {
            next = pooled_of(S, cnt, m, gamma, MAG ? -center : dlo - R.lambda, dhi);
            // gamma is the pooled value of its own set up to rounding: the end of the iteration, even if an
            // element at a threshold changes sides (for ever, sometimes)
            settled = fabsf(float(next - gamma)) <= (CUBIC ? 1e-12f : 1e-13f) * (fabsf(g) + (MAG && !CUBIC ? 0.0f : lam));
            if (next > gamma) {
              blo = gamma;
              lo_seen = true;
            } else {
              bhi = gamma;
              hi_seen = true;
            }
            leave = true;
          }
          // a single member next to a gap in which Psi = 0: its own minimiser is the end of that gap.
          // The test of the pair (s_k, s_{k+1}) decides whether there is a block at all
          if (cn == 1u && (int(ab) == k || int(ab) + 1 == k)) {
            if constexpr (SOLO) return false;          // (the neighbours may lie outside the list)
            float sk = inf, sk1 = -inf;
            if constexpr (!SOLO) neighbours(lo_f, hi_f, &sk, &sk1);
            const float member = float(S.s1 + center);
            if (int(ab) == k) sk1 = member; else sk = member;
            if (!P::seed_violates(double(sk) - center, double(sk1) - center, R, center)) {
              hi_f = sk1;                              // (s_{k+1} < s_k: the top k are above it)
              grow = false;
              return true;
            }
            const double dk = double(sk) - center, dk1 = double(sk1) - center;
            next = pooled_of(Sums{dk + dk1, dk * dk + dk1 * dk1, dk * dk * dk + dk1 * dk1 * dk1}, 2.0, 1.0,
                             gamma, MAG ? -center : dk1 - R.lambda, dk);
            ab = 0xffffffffu;                          // (another set: cannot end the iteration)
            leave = true;
          }
          // outside the list's window, where it was looked for?  On without the list
          if (use_list && leave && !settled && ((!lo_seen && next < blo) || (!hi_seen && next > bhi))) {
            gamma = next;
            use_list = false;
            if (SOLO) return false;
            blo = -1e300;
            bhi = 1e300;
            ab = 0xffffffffu;
            continue;
          }
          if (settled || (next > blo && next < bhi)) ok = true;
        }
        if (!ok) {
          if (use_list && it >= 3 && !(lo_seen && hi_seen)) return true;       // (no root in the window)
          const double w = t_hi - ga;
          next = blo > -1e299 && bhi < 1e299 ? 0.5 * (blo + bhi) : gamma + ldexp(blo > -1e299 ? w : -w, 2 * it);
          if (MAG && !(next + center > 0.0)) next = 0.5 * ga - center;
          ab = 0xffffffffu;                            // (not a pooled value)
        }
        if (!(fabs(next) < 1e300)) return true;
        gamma = uniform_f64(next, 0);
      }
      return true;
    };
    bool finished = !near;                             // (then nothing is known: from s_k)
    if constexpr (W > 1) {
      // lists of up to 16 elements per lane: the first wavefront alone, without barriers, and the
      // float64 arithmetic of a step once and not once per wavefront
      if (use_list && len <= 16u * kWave) {            // (uniform)
        if (threadIdx.x < kWave) {
          SearchGroup<kWave> one{nullptr};
          const bool f = exact_steps(one, std::true_type{}, lane, kWave);
          if (lane == 0) found = {gamma, cnt, m, lo_f, hi_f, (f ? 1 : 0) | (have ? 2 : 0) | (grow ? 4 : 0) | (use_list ? 8 : 0)};
        }
        __syncthreads();
        gamma = found.gamma;
        cnt = found.cnt;
        m = found.m;
        lo_f = found.lo;
        hi_f = found.hi;
        finished = (found.flags & 1) != 0;
        have = (found.flags & 2) != 0;
        grow = (found.flags & 4) != 0;
        use_list = (found.flags & 8) != 0;
      }
    }
    if (!finished) exact_steps(grp, std::false_type{}, tid, NT);
    // ---- 5. from s_k, and growth with the strict tests (ties, and whatever did not converge) -----------------
    // A few passes per binary digit and step of the set, whatever the values: 8 x 32768 values of 1e-30 in
    // magnitude with p = 4/3 and lambda = 0.1 (gamma is about 1e-87) 275 ms when the block was grown from s_k
    // one value at a time.
    if (grow) {
      use_list = false;
      // values are taken relative to an element of the row: differences of inputs with few bits, and the
      // sums of their powers, are exact then, and an exact tie is seen as one
      float seed_lo = inf, seed_hi = -inf;             // members of the block in any case
      const bool settled = have;
      if (have) {                                      // only what is certain
        const double ga = gamma + center, t_hi = upper_end(ga);
        lo_f = float_above(ga + slack_of(ga));
        hi_f = float_below(t_hi - slack_of(t_hi));
        float a = inf, b = -inf;
#pragma unroll
        for (int r = 0; r < E; ++r) {
          const float v = val(r);
          a = fminf(a, (v >= lo_f && v <= hi_f) ? v : inf);
          pass_fence(r, a);
        }
        grp.min_max(a, b);
        seed_lo = a;
      }
      if (!(seed_lo < inf)) {
        // s_k: bisection of the interval [lo, hi] of values that holds it, over the floats in their order.
        // The ends move in to the nearest elements every fourth step, and as soon as k elements lie at or above
        // the lower end: then s_k is the smallest of them.  (4 to 24 passes.)
        have = false;
        float a = inf, b = -inf;
#pragma unroll
        for (int r = 0; r < E; ++r) {
          a = fminf(a, val(r));
          b = fmaxf(b, val(r));
          pass_fence(r, a, b);
        }
        grp.min_max(a, b);
        uint32_t lo = ordered_of(a), hi = ordered_of(b), ge = uint32_t(n);
#pragma unroll 1
        for (int step = 1; lo < hi && step <= 64; ++step) {
          uint32_t cand = hi - (hi - lo) / 2u;         // (above lo)
          if (below && above && step <= 2) {           // (the secant's bracket)
            const uint32_t h = step == 1 ? ordered_of(w_lo) : ordered_of(w_hi + 1.01f * width_at(w_hi)) + 1u;
            if (h > lo && h <= hi) cand = h;
          }
          uint32_t at, d0;
          count_pass(inf, float_next_down(float_of_ordered(cand)), &at, &d0);      // elements >= cand
          if (int(at) >= k) {
            lo = cand;
            ge = at;
          } else {
            hi = cand - 1u;
          }
          if (int(at) == k || (step & 3) == 0 || step == 2) {
            float c_lo = float_of_ordered(lo), c_hi = float_of_ordered(hi);
            opaque(c_lo);
            opaque(c_hi);
            a = inf;
            b = -inf;
#pragma unroll
            for (int r = 0; r < E; ++r) {
              const float v = val(r);
              a = fminf(a, v >= c_lo ? v : inf);
              b = fmaxf(b, v <= c_hi ? v : -inf);
              pass_fence(r, a, b);
            }
            grp.min_max(a, b);
            lo = ordered_of(a);
            hi = int(at) == k ? lo : ordered_of(b);
          }
        }
        const float sk = float_of_ordered(lo);
        float sk1 = sk, dummy;                         // (tied with s_{k+1}: the ties are the seed)
        if (int(ge) <= k) neighbours(sk, inf, &dummy, &sk1);
        if (P::kCentered) {
          c32 = sk;
          center = double(c32);
        }
        const double dk = double(sk) - center, dk1 = double(sk1) - center;
        if (sk1 > -inf && P::seed_violates(dk, dk1, R, center)) {
          seed_lo = sk1;
          seed_hi = sk;
          have = true;
        } else {
          hi_f = sk1;                                  // (s_{k+1} < s_k, or zeros: the top k are above it)
        }
        if (have && !settled) {
          // the set of the block by threshold steps from the pair on, in passes over the registers
          gamma = P::pooled(2.0, 1.0, Sums{dk + dk1, dk * dk + dk1 * dk1, dk * dk * dk + dk1 * dk1 * dk1}, R,
                            MAG ? -center : dk1 - R.lambda, dk, center);
          double blo = -1e300, bhi = 1e300;
          uint32_t ab = 0xffffffffu, cn = 0xffffffffu;
          bool piece = false, found_it = false;
#pragma unroll 1
          for (int it = 0; it < 200 && !found_it; ++it) {
            const double ga = gamma + center;
            lo_f = fminf(float_above(ga), seed_lo);
            hi_f = fmaxf(float_below(upper_end(ga)), seed_hi);
            uint32_t na, nc;
            const Sums S = sums_pass(lo_f, hi_f, c32, &na, &nc);
            const bool same = na == ab && nc == cn;
            ab = na;
            cn = nc;
            cnt = double(cn);
            m = double(k) - double(ab);
            found_it = same && piece;
            if (found_it) break;
            const double next = P::pooled(cnt, m, S, R, MAG ? -center : double(lo_f) - center - R.lambda,
                                          double(hi_f) - center, center);
            found_it = fabs(next - gamma) <= 0.1 * slack_of(ga);
            if (found_it) {
              gamma = next;
              break;
            }
            if (next > gamma) blo = gamma; else bhi = gamma;
            piece = next > blo && next < bhi;
            gamma = piece ? next : 0.5 * (blo + bhi);
          }
          const double ga = gamma + center, t_hi = upper_end(ga);
          if (found_it) {
            grow = at_a_tie(grp, std::false_type{}, tid, NT, ga, t_hi);
            if (grow) {
              seed_lo = fminf(float_above(ga + slack_of(ga)), seed_lo);
              seed_hi = fmaxf(float_below(t_hi - slack_of(t_hi)), seed_hi);
            }
          }
        }
        if (have && grow) {
          lo_f = seed_lo;
          hi_f = seed_hi;
        }
      } else if (P::kCentered) {
        c32 = seed_lo;
        center = double(c32);
      }
      // Values are added to the block at its ends as long as one of the two next ones violates: one at a time,
      // and after eight of those as many as do on either side in turn, found by bisection (a value that does not
      // violate ends the run: neither do those beyond it).
      bool right = false;
#pragma unroll 1
      for (int step = 0; have && grow && step < 2 * n + 8; ++step) {
        float wa, wb;
        neighbours(lo_f, hi_f, &wa, &wb);
        uint32_t ab, cn, ca, cb;
        const Sums S = sums_pass(lo_f, hi_f, c32, &ab, &cn);
        count_pass(wb, wa, &ca, &cb);                  // elements above wa, and from wb to wa
        cb = wb > -inf ? ca + cb - ab - cn : 0u;       // copies of wb and of wa
        ca = wa < inf ? ab - ca : 0u;
        cnt = double(cn);
        m = double(k) - double(ab);
        const bool add_l = ca > 0u && P::left_violates(double(wa) - center, cnt, m, S, R, center);
        const bool add_r = cb > 0u && P::right_violates(double(wb) - center, cnt, m, S, R, center);
        if (!add_l && !add_r) {
          const double dlo = double(lo_f) - center, dhi = double(hi_f) - center;
          gamma = P::pooled(cnt, m, S, R, MAG ? -center : dlo - R.lambda, dhi, center);
          break;
        }
        if (add_l) hi_f = wa;
        if (add_r) lo_f = wb;
        if (step < 8) continue;
        right = !right;
        // the values up to `in` are dealt with, none beyond `out` is added
        uint32_t in = ordered_of(right ? lo_f : hi_f), out = ordered_of(right ? -3.4028235e38f : 3.4028235e38f);
#pragma unroll 1
        for (int turn = 0; turn < 40 && (right ? out < in : out > in); ++turn) {
          const float at = float_of_ordered(right ? out + (in - out) / 2u : out - (out - in) / 2u);
          // the element at `at` or next to it on the block's side, and the block up to it
          float va, vb;
          neighbours(right ? lo_f : float_next_up(at), right ? float_next_down(at) : inf, &va, &vb);
          const float v = right ? va : vb;
          if (right ? v >= lo_f : v <= hi_f) {         // (none in between)
            in = ordered_of(at);
            continue;
          }
          const Sums T = sums_pass(right ? float_next_up(v) : lo_f, right ? hi_f : float_next_down(v), c32, &ab, &cn);
          const double c = double(cn), mm = double(k) - double(ab), d = double(v) - center;
          if (right ? P::right_violates(d, c, mm, T, R, center) : P::left_violates(d, c, mm, T, R, center)) {
            if (right) lo_f = v;
            else hi_f = v;
            in = ordered_of(at);
          } else {
            out = right ? ordered_of(v) + 1u : ordered_of(v) - 1u;
          }
        }
      }
      // the tangents go through the list again (600 x 20000 values on a grid of 1/16, lambda = 1e-3: 101 us, 137 with a
      // pass over the row in the caches instead)
      if (have && want_jvp) {
        const float mid_b = 0.5f * lo_f + 0.5f * hi_f;
        gather(mid_b, fmaxf(hi_f - mid_b, mid_b - lo_f));
        use_list = len <= uint32_t(kListMax);
      }
    }
  }

  // ---- outputs, element by element ----------------------------------------------------------------------
  if (!have) lo_f = inf;                               // (no element is a member)
  auto is_above = [&](float v) { return v > hi_f; };
  auto is_in = [&](float v) { return v >= lo_f && v <= hi_f; };
  float tr[LIST_TAU ? 1 : E];
  double dgamma = 0.0;
  if (!LIST_TAU && (want_jvp || LOSS)) {
    // only elements whose outputs use it need their tangent: for the magnitude operator those of the
    // block and above it (the operators built on the mask use all of them)
#pragma unroll
    for (int c = 0; c < Q; ++c) {
      bool need = VAR != kSearchPlain;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float v = val(4 * c + r);
        need |= v >= lo_f || is_above(v);
        if (!LIST_TAU) tr[4 * c + r] = 0.0f;
      }
      if (!LIST_TAU && need) load_group(tangent, c, 0.0f, tr + 4 * c);
    }
  }
  auto tau_of = [&](int r) -> float {                  // tangent in sorted-value coordinates
    float t = tr[r];
    if (ABS) {
      t = (__float_as_uint(xr[r]) >> 31) ? -t : t;
      t = (xr[r] == 0.0f) ? 0.0f : t;                  // sign(0) = 0
    }
    return t;
  };
  if (want_jvp && have) {                              // uniform over the group
    // Prop. 7: d gamma = sum_B c_j tau_j / (sum_B c_j [+ lambda m])
    double d[2] = {0.0, 0.0};
    auto add = [&](float v, float tau) {
      if (CUBIC) {
        const double wgt = P::jac_weight(double(v) - center, gamma);
        d[0] = fma(wgt, double(tau), d[0]);
        d[1] += wgt;
      } else {
        d[0] += double(tau);
      }
    };
    if (use_list) {
#pragma unroll 1
      for (uint32_t j = tid; j < len; j += NT) {
        const float2 q = list[j];
        if (q.x >= lo_f && q.x <= hi_f) {
          const uint32_t e = __float_as_uint(q.y);
          float t = tangent[e & 0x7fffffffu];
          if (ABS) {
            t = (e >> 31) ? -t : t;
            t = q.x == 0.0f ? 0.0f : t;
          }
          if (LIST_TAU) list[j].y = t;
          add(q.x, t);
        }
      }
    } else {
      // (through the caches once more: the registers would take E unrolled steps of float64 arithmetic)
#pragma unroll 1
      for (int e = tid; e < n; e += NT) {
        const float xv = x[e], v = ABS ? fabsf(xv) : xv;
        if (v >= lo_f && v <= hi_f) {
          float t = tangent[e];
          if (ABS) {
            t = (__float_as_uint(xv) >> 31) ? -t : t;
            t = v == 0.0f ? 0.0f : t;
          }
          add(v, t);
        }
      }
    }
    grp.template sum<CUBIC ? 2 : 1, 0, 0>(d, nullptr, nullptr);      // (with a barrier for W > 1)
    if constexpr (W == 1) __builtin_amdgcn_wave_barrier();
    dgamma = d[0] / P::jac_denominator(CUBIC ? d[1] : cnt, m, R);
  }
  // top-k in magnitude, p = 4/3: the cubics of the elements above the block, packed, eight elements of every lane at
  // a time (unless more than half of them are above)
  constexpr bool PACK = MAG && CUBIC;
  static_assert(!PACK || kListMax * RPB == int(kPackMax) * (W * RPB), "the list has room for every wavefront");
  uint32_t pack_at = 0u;
  bool packed = false;
  float2* pack = list + (W > 1 ? (threadIdx.x / kWave) * kPackMax : 0u);
  if constexpr (PACK && W > 1) __syncthreads();        // (the list has been read)
  double acc = 0.0, ysum = 0.0;                        // of the loss
#pragma unroll
  for (int c = 0; c < Q; ++c) {
    opaque(lo_f);
    opaque(hi_f);
    if constexpr (PACK) {
      if ((c & 1) == 0) {
        constexpr int kGroup = 8;
        const int r1 = 4 * c + kGroup < E ? 4 * c + kGroup : E;
        uint32_t cnt_above = 0u, total;
#pragma unroll
        for (int r = 4 * c; r < r1; ++r) cnt_above += is_above(val(r)) ? 1u : 0u;
        pack_at = wave_inclusive_scan(cnt_above, &total) - cnt_above;
        packed = total <= kPackMax;
        if (packed && total > 0u) {
          uint32_t to = pack_at;
#pragma unroll
          for (int r = 4 * c; r < r1; ++r) {
            const float v = val(r);
            if (is_above(v)) pack[to++] = make_float2(v, want_jvp ? tr[r] : 0.0f);
          }
          packed_above_mag43<1>(pack, total, R, want_jvp);
        }
      }
    }
    float yv[4], jv[4];
    bool some = false;
    bool listed[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float v = val(4 * c + r);
      listed[r] = LIST_TAU && use_list && fabsf(v - list_mid) <= list_half;
      some |= (LIST_TAU && use_list) ? listed[r] : is_in(v);
    }
    const bool some_in = __any(some);                  // few wavefronts hold an element of a short block
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int q = 4 * c + r;
      const float xv = xr[q], v = val(q);
      const bool ab = is_above(v);
      const bool neg = MAG && (__float_as_uint(xv) >> 31);
      float y = 0.0f, dy = 0.0f;
      double yd = 0.0;                                 // the mask before its rounding (loss)
      if (!MAG) {
        y = ab ? 1.0f : 0.0f;
        yd = ab ? 1.0 : 0.0;
      } else if (!CUBIC) {
        // (up to 2048 elements one rounding, whatever the shape, as in the kernels of those lengths; above, the
        // float32 product of the other long-row routes, whose results are the same bit for bit)
        y = ab ? (n > 2048 ? xv * float(R.inv_1pl) : float(double(xv) * R.inv_1pl)) : 0.0f;
        if (!LIST_TAU && want_jvp && ab && v != 0.0f)
          dy = n > 2048 ? tr[q] * float(R.inv_1pl) : float(double(tr[q]) * R.inv_1pl);
      } else if (packed) {
        if (ab) {
          const float2 q2 = pack[pack_at++];
          y = v == 0.0f ? 0.0f : (neg ? -q2.x : q2.x);
          dy = v == 0.0f ? 0.0f : q2.y;
        }
      } else if (__any(ab)) {
        double gd, slope = 0.0;
        above_mag43<1>(double(v), R, want_jvp, &gd, &slope);
        const float gf = float(gd);
        const bool some_y = ab && v != 0.0f;
        y = some_y ? (neg ? -gf : gf) : 0.0f;
        dy = (some_y && want_jvp) ? float(slope * double(tr[q])) : 0.0f;
      }
      const bool in = is_in(v);
      if (some_in) {
        const double d = double(v) - center;
        const double t = (d - gamma) * R.inv_lambda;
        const double yb = CUBIC ? t * t * t : t;
        float yf = float(yb);
        if (MAG) yf = yf == 0.0f ? 0.0f : (neg ? -yf : yf);
        y = in ? yf : y;
        if (LOSS) yd = in ? yb : yd;
        if (want_jvp) {
          float tau = 0.0f;
          if constexpr (LIST_TAU) {
            if (use_list) {
              if (listed[r]) tau = list[list_at++].y;
            } else if (in) {
              tau = tangent[first_of(c) + r];
            }
          } else {
            tau = tau_of(q);
          }
          const double diff = double(tau) - dgamma;
          float df = float((CUBIC ? 3.0 * t * t : 1.0) * R.inv_lambda * diff);
          if (MAG) df = (df == 0.0f || v == 0.0f) ? 0.0f : (neg ? -df : df);
          dy = in ? df : dy;
        }
      }
      if (VAR == kSearchSigned) {
        const float sg = float((xv > 0.0f) - (xv < 0.0f));
        const double u = double(v) * R.inv_lambda;
        const float cap = float(CUBIC ? u * u * u : u);
        // the truncation v >= 0 is active inside the block iff gamma < 0, above it iff s < lambda
        const bool clipped = in ? (center + gamma < 0.0) : (ab && double(v) < R.lambda);
        if (want_jvp) {
          const double hess = CUBIC ? 3.0 * u * u * R.inv_lambda : R.inv_lambda;
          const float jm = clipped ? float(hess * double(tr[q])) : sg * dy;
          dy = jm == 0.0f ? 0.0f : jm;
        }
        const float ys = sg * (clipped ? cap : y);
        y = ys == 0.0f ? 0.0f : ys;
      } else if (VAR == kSearchMasked) {
        if (want_jvp) dy = float(double(tr[q]) * double(y) + double(xv) * double(dy));
        y = xv * y;
      } else if (LOSS) {
        // <y, x> - (lambda / p) sum y^p - <x, t>; y^p = t y with t = (s - gamma) / lambda (clipped),
        // as y = t^(q-1) and p (q-1) = q
        const double xd = xv == xv ? double(xv) : 0.0;
        double yp = yd;
        if (some_in && in) yp = (double(v) - center - gamma) * R.inv_lambda * yd;
        acc += yd * xd - lam_over_p * yp - xd * double(tr[q]);
        ysum += yd;
        y -= tr[q];
      }
      yv[r] = y;
      jv[r] = dy;
    }
    if (out != nullptr) store_group(out, c, yv);
    if (want_jvp) store_group(jvp, c, jv);
    if (LOSS) {
      opaque(acc);
      opaque(ysum);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  if (LOSS) {
    double d[2] = {acc, ysum};
    grp.template sum<2, 0, 0>(d, nullptr, nullptr);
    // the multiplier term of the maximisation form (Prop. 2): zero up to the rounding of gamma
    if (have) d[0] -= (center + gamma) * (d[1] - double(k));
    if (tid == 0) loss[row] = float(d[0]);
  }
}

template <int NT, int E>
int launch_row_search_shape(int var, bool mag, int pc, bool vec, const float* x, const float* tangent,
                            float* out, float* jvp, float* loss, double lam_over_p, int64_t rows, int n,
                            int k, const Reg& R, hipStream_t st) {
  constexpr int RPB = NT == 64 ? 4 : 1;
  const int64_t blocks = (rows + RPB - 1) / RPB;
  if (blocks > 0x7fffffffLL) return -1;
#define TOPK_SEARCH(M, P, V)                                                                          \
  do {                                                                                                \
    hipLaunchKernelGGL((row_search_kernel<NT, E, M, P, V>), dim3(unsigned(blocks)),                   \
                       dim3(NT == 64 ? 256 : NT), 0, st, x, tangent, out, jvp, rows, n, k, R, vec,    \
                       loss, lam_over_p);                                                             \
    return 0;                                                                                         \
  } while (0)
  if constexpr (NT * E <= 1024) {        // (only the operator that the short-row kernels do not have)
    if (var == kSearchPlain && mag && pc == kP43) TOPK_SEARCH(true, kP43, kSearchPlain);
  } else if (var == kSearchPlain) {
    if (!mag && pc == kP2) TOPK_SEARCH(false, kP2, kSearchPlain);
    if (!mag && pc == kP43) TOPK_SEARCH(false, kP43, kSearchPlain);
    if (mag && pc == kP2) TOPK_SEARCH(true, kP2, kSearchPlain);
    if (mag && pc == kP43) TOPK_SEARCH(true, kP43, kSearchPlain);
  } else if (var == kSearchSigned) {
    if (pc == kP2) TOPK_SEARCH(false, kP2, kSearchSigned);
    if (pc == kP43) TOPK_SEARCH(false, kP43, kSearchSigned);
  } else if (var == kSearchMasked) {
    if (pc == kP2) TOPK_SEARCH(false, kP2, kSearchMasked);
    if (pc == kP43) TOPK_SEARCH(false, kP43, kSearchMasked);
  } else if (var == kSearchLoss) {
    if (pc == kP2) TOPK_SEARCH(false, kP2, kSearchLoss);
    if (pc == kP43) TOPK_SEARCH(false, kP43, kSearchLoss);
  }
#undef TOPK_SEARCH
  return -1;
}

}  // namespace
}  // namespace topk
