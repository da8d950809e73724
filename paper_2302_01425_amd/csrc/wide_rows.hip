// Wide route, the solve: rows above 32765 elements, several workgroups per row, dense outputs by value.
//
// The key window [klo, khi] of a row (radix_sort.hip: a histogram of the leading key bits) holds everything
// that can pool.  Two launches find the pooled value gamma and d gamma of the row's block:
//
//   collect : reads the row once.  Every wavefront compacts the elements of its part that lie in the window
//             into its own slot of the "b" arrays (value, index) and every workgroup counts them in kFineBins
//             bins of equal width in value.
//   solve   : the block is a set of values and gamma the root of the non-increasing function
//                 Psi(g) = #above(g) + sum over the set at g of grad r*(s - g) - k
//             (an element counts 1 if its singleton minimiser lies above g, 0 if its value lies below g and
//             its output in between).  With every element moved to the lower (upper) end of its bin Psi is
//             bounded from below (above), so the counts alone bracket gamma between bin edges, a bin or two
//             apart.  All workgroups of a row find that bracket, each for itself (one edge per thread, from prefix sums
//             over the bins), and then work through their own part of the candidates: bins that lie between
//             the two thresholds whatever gamma in the bracket are members (power sums and moments of the tangent,
//             added up in float64), bins a threshold may fall into go to the row's list.  The workgroup that
//             finishes last has the sums of the sure members and a list of some hundred elements, on which it
//             solves for gamma exactly (see boundary_solve) and adds up d gamma (Prop. 7).
//
// No step sorts, and none but the last is left to one workgroup, whose work there does not grow with the length of the
// block.  Before, the candidates went through a second histogram level, an in-place compaction, a scan and a gather (four
// launches) to one workgroup per row that solved a list of all of them: compaction to solution 103 us on
// 16 x 1 M (37000 candidates a row) and 69 us on 1 x 16.7 M, now 19 + 22 and 23 + 23.  What bounds the two: collect
// reads the row at 3.5 TB/s from the caches behind the L2; solve is a chain of some fifteen dependent steps (counts 4 us,
// prefix sums and bracket 4, candidates and their tangents 3, hand-over to the last workgroup 5, exact solve 4).
//
// Order: slots hold a wavefront's elements lane by lane, lists hold the parts in order, and sums are added in a fixed
// order, so that results do not depend on how the workgroups were scheduled.
#include <hip/hip_runtime.h>

#include "common.hpp"
#include "group.hpp"
#include "launch.hpp"
#include "pooling.hpp"
#include "radix.hpp"
#include "wave.hpp"

namespace topk {
namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / kWave;
// Bins of the window.  An end of the block is known to one or two bins, so that the list holds some four in 1024 of
// the candidates.  More bins cost more than the shorter list saves: a compute unit reads 10 to 14 bytes of counts per
// nanosecond that other dies have written.
constexpr int kFineBins = 1024;
constexpr int kItems = 16;
constexpr int kStep = kItems * kWave;            // elements a wavefront takes at a time
constexpr int kPart = kWaves * kStep;            // a workgroup's part is a multiple of this
// Counts of the parts are added up by the readers up to this many parts per row; above, the last workgroup of each of
// kGroups groups of parts to finish adds those of its group.
constexpr int kDirectParts = 32;
constexpr int kGroups = kWideGroups;
// About one workgroup per compute unit: no row has more parts.
constexpr int kMaxParts = 256;

// The value window as every kernel of the route sees it: values v_bot .. v_top in kFineBins bins.
struct Window {
  float v_top, v_bot;
  double base, scale, width;                     // of a bin: base + j width; scale = 1 / width
};
// Zeros do not pool in the magnitude operator (0 is no larger than any pooled value) and their outputs are 0: they
// are left out of the window, which for rows that are mostly zeros would hold nothing else (1 x 16.7 M, 95 % zeros:
// 28.9 ms with them, 97 us without).
template <bool MAG>
__device__ __forceinline__ Window window_of(const RowSel& s) {
  Window w;
  // key order is reversed value order, and -0 == +0 either way (bound_value clamps the keys beyond the infinities,
  // which would decode to NaN)
  w.v_top = float(bound_value(s.klo));
  w.v_bot = float(bound_value(s.khi));
  if (MAG && !(w.v_bot > 0.0f)) w.v_bot = __uint_as_float(1u);
  w.base = double(w.v_bot);
  const double span = double(w.v_top) - w.base;
  // (infinities in the window: everything in bin 0)
  const bool ok = span > 0.0 && span < 1e300;
  w.scale = ok ? double(kFineBins) / span : 0.0;
  w.width = span * (1.0 / kFineBins);
  return w;
}
// bin of a value: never falls as the value rises.  The rounding of these operations is far below a thousandth
// of a bin (a bin is at least 2^-35 of the values: the window holds at least one float)
__device__ __forceinline__ int bin_of(double v, const Window& w) {
  const double f = (v - w.base) * w.scale;
  return f > 0.0 ? (f < double(kFineBins - 1) ? int(f) : kFineBins - 1) : 0;         // (NaN: 0)
}

// Where the route keeps its arrays (all in parts of the workspace that it does not use otherwise).
struct WideScratch {
  uint32_t* slot_count;   // [rows][parts][kWaves] candidates of a wavefront's slot
  double* sums;           // [rows][parts][8] sums of a workgroup's sure members: s, s^2, s^3, t, t s, t s^2
  uint32_t* listed;       // [rows][parts] list entries of a workgroup
  uint32_t* above;        // [rows][parts] elements above the window
  uint32_t* part_bins;    // [rows][parts][kFineBins]: 16 bits each when a part has at most 65536 elements (pack_counts)
  uint32_t* group_bins;   // [rows][kGroups][kFineBins]
  uint32_t* arrived;      // [rows][kSelSlices * 2 * kSel2Bins]: [0] the row, [1 + g] group g; cleared by the window kernel
};

// Workgroups are dealt to the eight dies in turn: a run of neighbours in a row (which read the same counts) to one die.
__device__ __forceinline__ int64_t die_block(uint32_t block, uint32_t blocks) {
  constexpr uint32_t kDies = 8;
  return blocks % kDies == 0u ? int64_t(block % kDies) * (blocks / kDies) + block / kDies : int64_t(block);
}

// What one workgroup writes for another one of the same launch goes through agent-scope accesses, which are coherent
// between the dies, and the writer waits for its stores before it counts itself as arrived.  (A fence of that scope
// instead writes back and invalidates the whole L2 of the die: with one per workgroup collect took 207 us and solve
// 94 on 1 x 16.7 M, without 45 and 35.)
__device__ __forceinline__ void publish(uint32_t* p, uint32_t v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void publish(double* p, double v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <class T>
__device__ __forceinline__ T published(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// by all threads, after their last publish: is this the last of `members` workgroups to arrive?
__device__ __forceinline__ bool arrive_last(uint32_t* counter, int members, uint32_t* shared) {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (threadIdx.x == 0)
    *shared = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == uint32_t(members - 1);
  __syncthreads();
  return *shared != 0u;
}

// Two counts of a part of at most 65536 elements in one word.  (All of them in one bin: a word that two counts cannot
// make, as their sum is at most 65536.)
__device__ __forceinline__ uint32_t pack_counts(uint32_t a, uint32_t b) {
  if (a > 0xffffu) return 0xffffffffu;
  if (b > 0xffffu) return 0xfffffffeu;
  return a | (b << 16);
}
__device__ __forceinline__ uint2 unpack_counts(uint32_t t) {
  if (t >= 0xfffffffeu) return t == 0xffffffffu ? make_uint2(65536u, 0u) : make_uint2(0u, 65536u);
  return make_uint2(t & 0xffffu, t >> 16);
}
constexpr int kPairs = kFineBins / 2;            // two bins per thread: kPairs threads to a part
constexpr int kPartsAtOnce = kThreads / kPairs;

// ---- collect ---------------------------------------------------------------------------------------------------------
// Bound by memory; the next step's loads are in flight while a step is worked on, so that one workgroup per compute unit
// is enough (and few parts keep the counts short that solve reads).  VEC: rows that start 16-byte aligned.
constexpr int kStage = 384;                      // candidates staged in LDS at a time

template <bool MAG, bool VEC>
__global__ __launch_bounds__(kThreads) void wide_collect_kernel(
    const float* __restrict__ x_all, const RowSel* __restrict__ sel, uint32_t* __restrict__ slot_val,
    uint32_t* __restrict__ slot_idx, WideScratch sc, int64_t n, int64_t part_len, int parts, int group_len) {
  __shared__ uint32_t bins[kFineBins];
  __shared__ uint2 stage_all[kWaves][kStage];
  __shared__ uint32_t wave_above[kWaves];
  __shared__ uint32_t last_of_group;
  const int64_t id = die_block(blockIdx.x, gridDim.x);
  const int64_t row = id / parts;
  const int part = int(id % parts);
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  const float* x = x_all + row * n;
  const int64_t wave_len = part_len / kWaves;
  const int64_t first = part * part_len + w * wave_len;
  const int64_t last = first + wave_len < n ? first + wave_len : n;
  auto at = [&](int i) { return VEC ? ((i >> 2) * kWave + lane) * 4 + (i & 3) : i * kWave + lane; };
  auto load = [&](int64_t e0, float (&v)[kItems]) {
    const float nan = __uint_as_float(0x7fc00000u);
    const int left = last - e0 < kStep ? int(last - e0) : kStep;       // (negative beyond the part)
    if (VEC) {
#pragma unroll
      for (int q = 0; q < kItems / 4; ++q) {
        float4 f = make_float4(nan, nan, nan, nan);
        if (at(4 * q) < left) f = *reinterpret_cast<const float4*>(x + e0 + at(4 * q));
        v[4 * q] = f.x; v[4 * q + 1] = f.y; v[4 * q + 2] = f.z; v[4 * q + 3] = f.w;
      }
    } else {
#pragma unroll
      for (int i = 0; i < kItems; ++i) v[i] = at(i) < left ? x[e0 + at(i)] : nan;
    }
  };
  float next[kItems];
  load(first, next);
  for (int i = threadIdx.x; i < kFineBins; i += kThreads) bins[i] = 0u;
  const Window win = window_of<MAG>(sel[row]);
  uint32_t* val_out = slot_val + row * n + first;
  uint32_t* idx_out = slot_idx + row * n + first;
  uint2* stage = stage_all[w];
  uint32_t run = 0u, above = 0u;
  __syncthreads();
#pragma unroll 1
  for (int64_t e0 = first; e0 < last; e0 += kStep) {
    float xv[kItems];
#pragma unroll
    for (int i = 0; i < kItems; ++i) xv[i] = next[i];
    load(e0 + kStep, next);
    uint32_t over = 0u, upto = 0u;               // elements above the window, and those and its own
#pragma unroll
    for (int i = 0; i < kItems; ++i) {
      const float v = MAG ? fabsf(xv[i]) : xv[i];
      over += v > win.v_top ? 1u : 0u;
      upto += v >= win.v_bot ? 1u : 0u;
    }
    above += over;
    uint32_t total;
    const uint32_t mine = upto - over, to = wave_inclusive_scan(mine, &total) - mine;
    // staged in LDS, so that full wavefronts write (and the float64 arithmetic of the bins is done once per candidate)
#pragma unroll 1
    for (uint32_t done = 0; done < total; done += kStage) {
      uint32_t slot = to - done;
#pragma unroll
      for (int i = 0; i < kItems; ++i) {
        const float v = MAG ? fabsf(xv[i]) : xv[i];
        if (v <= win.v_top && v >= win.v_bot) {
          const uint32_t e = uint32_t(e0) + uint32_t(at(i));
          if (slot < uint32_t(kStage))
            stage[slot] = make_uint2(__float_as_uint(v), MAG ? ((e << 1) | (__float_as_uint(xv[i]) >> 31)) : e);
          ++slot;
        }
      }
      __builtin_amdgcn_wave_barrier();
      const uint32_t here = total - done < uint32_t(kStage) ? total - done : uint32_t(kStage);
      for (uint32_t j = lane; j < here; j += kWave) {
        const uint2 q = stage[j];
        val_out[run + done + j] = q.x;
        idx_out[run + done + j] = q.y;
        atomicAdd(&bins[bin_of(double(__uint_as_float(q.x)), win)], 1u);
      }
      __builtin_amdgcn_wave_barrier();
    }
    run += total;
  }
  above = lanes_sum<kWave>(above);
  if (lane == 0) {
    sc.slot_count[(row * parts + part) * kWaves + w] = run;
    wave_above[w] = above;
  }
  __syncthreads();
  if (w == 0) {
    const uint32_t all = lanes_sum<kWaves>(wave_above[lane & (kWaves - 1)]);
    if (lane == 0) sc.above[row * parts + part] = all;
  }
  const bool narrow = part_len <= 65536;
  const int pair = threadIdx.x % kPairs;
  uint32_t* mine = sc.part_bins + (row * parts + part) * int64_t(narrow ? kPairs : kFineBins);
  const bool direct = parts <= kDirectParts;
  if (threadIdx.x < kPairs) {
    const uint32_t b0 = bins[2 * pair], b1 = bins[2 * pair + 1];
    if (narrow) {
      if (direct) mine[pair] = pack_counts(b0, b1);
      else publish(mine + pair, pack_counts(b0, b1));
    } else {
      publish(mine + 2 * pair, b0);
      publish(mine + 2 * pair + 1, b1);
    }
  }
  if (direct) return;
  // ---- the last workgroup of a group adds up its counts -------------------------------------------------------------
  const int group = part / group_len, p0 = group * group_len;
  const int members = parts - p0 < group_len ? parts - p0 : group_len;
  if (!arrive_last(&sc.arrived[row * (kSelSlices * 2 * kSel2Bins) + 1 + group], members, &last_of_group)) return;
  uint32_t c0 = 0u, c1 = 0u;
  const uint32_t* src = sc.part_bins + (row * parts + p0) * int64_t(narrow ? kPairs : kFineBins);
  for (int q0 = threadIdx.x / kPairs; q0 < members; q0 += 8 * kPartsAtOnce) {      // eight loads in flight
    uint2 v[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int from = q0 + q * kPartsAtOnce;
      v[q] = make_uint2(0u, 0u);
      if (from < members) {
        if (narrow) {
          v[q].x = published(src + int64_t(from) * kPairs + pair);
        } else {
          v[q].x = published(src + int64_t(from) * kFineBins + 2 * pair);
          v[q].y = published(src + int64_t(from) * kFineBins + 2 * pair + 1);
        }
      }
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const uint2 c = narrow ? unpack_counts(v[q].x) : v[q];
      c0 += c.x;
      c1 += c.y;
    }
  }
  __syncthreads();                               // (every thread has read its own counts)
  if (threadIdx.x < kPairs) {
    bins[2 * pair] = c0;
    bins[2 * pair + 1] = c1;
  }
  __syncthreads();
  if (threadIdx.x >= kPairs) {
    atomicAdd(&bins[2 * pair], c0);
    atomicAdd(&bins[2 * pair + 1], c1);
  }
  __syncthreads();
  if (threadIdx.x < kPairs)
    reinterpret_cast<uint2*>(sc.group_bins + (row * kGroups + group) * int64_t(kFineBins))[pair] =
        make_uint2(bins[2 * pair], bins[2 * pair + 1]);
}

// ---- solve -----------------------------------------------------------------------------------------------------------

// end of the values that are below their cap at the pooled value ga (absolute)
template <bool MAG, int PC>
__device__ __forceinline__ double upper_end(double ga, const Reg& R) {
  if (!MAG) return ga + R.lambda;
  if (PC == kP2) return ga * R.one_p_lambda;
  return ga + R.lambda * cbrt(fmax(ga, 0.0));
}

// the number with the fewest significant bits between two finite floats a <= b
__device__ __forceinline__ float simplest_between(float a, float b) {
  if (!(a < b)) return a;
  if (a <= 0.0f && b >= 0.0f) return 0.0f;
  uint32_t lo = __float_as_uint(a) & 0x7fffffffu, hi = __float_as_uint(b) & 0x7fffffffu;
  const uint32_t sign = __float_as_uint(a) & 0x80000000u;
  if (sign) {
    const uint32_t t = lo;
    lo = hi;
    hi = t;
  }
  const int top = 31 - __clz(int(lo ^ hi));      // (lo < hi: the highest differing bit is set in hi)
  return __uint_as_float(sign | (hi & ~((1u << top) - 1u)));
}

// What is known before the list is looked at, and the result.
struct Sure {
  double cnt, m;          // sure members; top-k positions that are not above everything listed
  Sums S;                 // of the sure members' centred values
  double center;
  double lo, hi;          // gamma lies in between (absolute)
  bool coarse;            // lambda is lost beside the distances from this centre: s_k is to be the centre
};
struct Block {
  double gamma, center;   // the pooled value: gamma + center
  double cnt, m;
  float lo, hi;           // members: lo <= value <= hi; everything above hi is before the block
  bool have;
};

// The exact solve, by the threads of the group G: gamma from the sure members and the list.  each(f): f(value) for
// this thread's entries (and for NaN); len: entries in all.
//   1. threshold steps: the listed members at g are counted and summed, the pooled value of that set and the sure members
//      is the next g (the root of the piece of Psi that g lies on), until the set stays the same;
//   2. a threshold within rounding of an element's value: that element ties with the block, and the strict tests of the
//      PAV loop (pooling.hpp) decide, on the block without what is that near to its ends;
//   3. no set came out (no element strictly between the thresholds, or none but ties): s_k and s_{k+1} are found in the
//      list, which holds them then, and the pair decides whether there is a block at all.
template <bool MAG, int PC, class G, class EACH>
__device__ __forceinline__ Block boundary_solve(G& grp, EACH each, uint32_t len, const Sure& sure, const Reg& R) {
  using P = Pool<MAG, PC>;
  constexpr bool CUBIC = (PC == kP43);
  const float inf = __uint_as_float(0x7f800000u);
  double center = sure.center;
  Block out{0.0, center, 0.0, 0.0, inf, inf, false};
  float seed_lo = inf, seed_hi = -inf;           // members in any case
  double gamma = 0.0, cnt = 0.0, m = 0.0;
  float lo = inf, hi = -inf;
  // listed elements above hi and in [lo, hi], and with the sure members the sums of the set
  auto set_pass = [&](float plo, float phi, double* na, double* nc) -> Sums {
    uint32_t c0 = 0u, c1 = 0u;
    double d[3] = {0.0, 0.0, 0.0};
    each([&](float v) {
      const bool ab = v > phi, in = v >= plo && !ab;
      c0 += ab ? 1u : 0u;
      c1 += in ? 1u : 0u;
      const double t = in ? double(v) - center : 0.0;
      d[0] += t;
      if (CUBIC) {
        d[1] += t * t;
        d[2] = fma(t * t, t, d[2]);
      }
    });
    if constexpr (CUBIC) grp.sum_with_counts(d, c0, c1);
    else grp.sum_with_counts(reinterpret_cast<double(&)[1]>(d[0]), c0, c1);
    *na = double(c0);
    *nc = double(c1);
    return Sums{sure.S.s1 + d[0], sure.S.s2 + d[1], sure.S.s3 + d[2]};
  };
  // smallest listed value above hi, largest below lo
  auto neighbours = [&](float plo, float phi, float* above, float* below) {
    float a = inf, b = -inf;
    each([&](float v) {
      a = fminf(a, v > phi ? v : inf);
      b = fmaxf(b, v < plo ? v : -inf);
    });
    grp.min_max(a, b);
    *above = a;
    *below = b;
  };
  auto pooled_of = [&](double c, double mm, const Sums& S) {
    // (the cubic's root lies above (smallest member - lambda), resp. 0, and below the largest member)
    return P::pooled(c, mm, S, R, MAG ? -center : double(lo) - center - R.lambda, double(hi) - center, center);
  };
  auto slack_of = [&](double t) -> double {
    return (CUBIC ? 1e-11 : 1e-12) * (fabs(t) + (MAG && !CUBIC ? 0.0 : R.lambda));
  };
  const double noise = 1e-13 * (MAG && !CUBIC ? 0.0 : R.lambda);
  // (blind: steps to the middle of the bracket, at which no pooled value inside it was found; a few of them, and the
  // list's order statistics are the shorter way)
  auto threshold_steps = [&](double blo, double bhi, int most, int blind) -> bool {
    double ab = -1.0, mem = -1.0;
    bool piece = false;                          // gamma is the pooled value of the set seen last
#pragma unroll 1
    for (int it = 0; it < most; ++it) {
      const double ga = gamma + center;
      lo = fminf(float_above(ga), seed_lo);
      hi = fmaxf(float_below(upper_end<MAG, PC>(ga, R)), seed_hi);
      double na, nc;
      const Sums S = set_pass(lo, hi, &na, &nc);
      if (piece && na == ab && nc == mem) return true;
      ab = na;
      mem = nc;
      cnt = sure.cnt + nc;
      m = sure.m - na;
      double next = gamma;
      piece = false;
      if (cnt == 0.0 && m == 0.0) return false;  // Psi = 0 on an empty set
      if (m <= 0.0) {
        blo = gamma;                             // (as many above as there are top-k positions, or more)
      } else if (m > cnt) {
        bhi = gamma;                             // (fewer than k elements that far)
      } else {
        next = pooled_of(cnt, m, S);
        if (fabs(next - gamma) <= noise + 1e-13 * fabs(ga)) {
          gamma = next;
          return true;
        }
        if (next > gamma) blo = gamma;
        else bhi = gamma;
        piece = next > blo && next < bhi;
      }
      if (!piece) {
        next = 0.5 * (blo + bhi);
        if (--blind < 0) return false;
      }
      if (!(fabs(next) < 1e299) || next == gamma) return false;
      gamma = next;
    }
    return false;
  };
  // ---- 1. ------------------------------------------------------------------------------------------------------------
  gamma = 0.5 * (sure.lo + sure.hi) - center;
  const bool bracketed = fabs(gamma) < 1e299;
  bool settled = bracketed && !sure.coarse && threshold_steps(sure.lo - center, sure.hi - center, 64, sure.cnt > 0.0 ? 64 : 6);
  bool grow = true;
  float first = inf, last = -inf;                // the set that is certain
  if (settled) {
    const double ga = gamma + center, t_hi = upper_end<MAG, PC>(ga, R);
    const double s1 = slack_of(ga), s2 = slack_of(t_hi);
    grow = false;
    // (mostly no float lies that near to either)
    if (fabs(double(float(ga)) - ga) <= s1 || fabs(double(float(t_hi)) - t_hi) <= s2) {
      const float a1 = float_above(ga - s1), b1 = float_below(ga + s1);
      const float a2 = float_above(t_hi - s2), b2 = float_below(t_hi + s2);
      double d[2] = {0.0, 0.0};
      each([&](float v) {
        d[0] += ((v >= a1 && v <= b1) || (v >= a2 && v <= b2)) ? 1.0 : 0.0;
        d[1] += (v > b1 && v < a2) ? 1.0 : 0.0;
      });
      grp.sum(d);
      grow = d[0] > 0.0;
      if (grow && sure.cnt + d[1] > 0.0) {
        first = float_above(ga + s1);
        last = float_below(t_hi - s2);
      }
    }
  } else if (sure.cnt > 0.0) {                   // (the sure members alone: nothing listed lies between its ends)
    first = float_above(sure.hi);
    last = float_below(upper_end<MAG, PC>(sure.lo, R));
  }
  // ---- 3. s_k and s_{k+1}: bisection over the floats in their order; every fourth step the ends move in to the nearest
  // elements -----------------------------------------------------------------------------------------------------------
  if (grow && !(first < inf)) {
    float a = inf, b = -inf;
    each([&](float v) {
      a = fminf(a, v);
      b = fmaxf(b, v);
    });
    grp.min_max(a, b);
    uint32_t olo = ordered_of(a), ohi = ordered_of(b);
    double ge = double(len);                     // elements at or above olo
    const double k = sure.m;
    if (!(k >= 1.0 && k < double(len))) {        // (cannot be: the list holds both)
      out.hi = k >= 1.0 ? -inf : inf;
      out.lo = inf;
      return out;
    }
#pragma unroll 1
    for (int step = 0; olo < ohi && step < 40; ++step) {
      const uint32_t cand = ohi - (ohi - olo) / 2u;          // (above olo)
      const float cv = float_of_ordered(cand);
      double d[1] = {0.0};
      each([&](float v) { d[0] += v >= cv ? 1.0 : 0.0; });
      grp.sum(d);
      if (d[0] >= k) {
        olo = cand;
        ge = d[0];
      } else {
        ohi = cand - 1u;
      }
      if (d[0] == k || (step & 3) == 1) {
        const float c_lo = float_of_ordered(olo), c_hi = float_of_ordered(ohi);
        a = inf;
        b = -inf;
        each([&](float v) {
          a = fminf(a, v >= c_lo ? v : inf);
          b = fmaxf(b, v <= c_hi ? v : -inf);
        });
        grp.min_max(a, b);
        olo = ordered_of(a);
        ohi = d[0] == k ? olo : ordered_of(b);
      }
    }
    const float sk = float_of_ordered(olo);
    float sk1 = sk, none;                        // (tied with s_{k+1}: the ties are the seed)
    if (ge <= k) neighbours(sk, inf, &none, &sk1);
    if (sure.coarse && fabsf(sk) < inf) center = double(sk);
    const double dk = double(sk) - center, dk1 = double(sk1) - center;
    if (!P::seed_violates(dk, dk1, R, center)) {
      out.hi = sk1;                              // (s_{k+1} < s_k, or zeros: the top k are above it)
      return out;
    }
    seed_lo = sk1;
    seed_hi = sk;
    if (!settled) {
      gamma = P::pooled(2.0, 1.0, Sums{dk + dk1, dk * dk + dk1 * dk1, dk * dk * dk + dk1 * dk1 * dk1}, R,
                        MAG ? -center : dk1 - R.lambda, dk, center);
      settled = threshold_steps(-1e300, 1e300, 200, 200);
    }
    first = seed_lo;
    last = seed_hi;
    if (settled) {
      const double ga = gamma + center, t_hi = upper_end<MAG, PC>(ga, R);
      first = fminf(float_above(ga + slack_of(ga)), first);
      last = fmaxf(float_below(t_hi - slack_of(t_hi)), last);
    }
  }
  // ---- 2. growth: values are added at the ends as long as one of the two next ones violates, one at a time, and after
  // eight of those as many as do on either side in turn, found by bisection (a value that does not violate ends the run:
  // neither do those beyond it) -------------------------------------------------------------------------------------
  if (grow) {
    lo = first;
    hi = last;
    bool right = false;
#pragma unroll 1
    for (uint32_t step = 0; step < 2u * len + 8u; ++step) {
      float wa, wb;
      neighbours(lo, hi, &wa, &wb);
      double na, nc;
      const Sums S = set_pass(lo, hi, &na, &nc);
      cnt = sure.cnt + nc;
      m = sure.m - na;
      gamma = pooled_of(cnt, m, S);
      const bool add_l = wa < inf && P::left_violates(double(wa) - center, cnt, m, S, R, center);
      const bool add_r = wb > -inf && P::right_violates(double(wb) - center, cnt, m, S, R, center);
      if (!add_l && !add_r) break;
      if (add_l) hi = wa;
      if (add_r) lo = wb;
      if (step < 8u) continue;
      right = !right;
      // the values up to `in` are dealt with, none beyond `end` is added
      uint32_t in = ordered_of(right ? lo : hi), end = ordered_of(right ? -3.4028235e38f : 3.4028235e38f);
#pragma unroll 1
      for (int turn = 0; turn < 40 && (right ? end < in : end > in); ++turn) {
        const float at = float_of_ordered(right ? end + (in - end) / 2u : end - (end - in) / 2u);
        // the element at `at` or next to it on the block's side, and the block up to it
        float va, vb;
        neighbours(right ? lo : float_next_up(at), right ? float_next_down(at) : inf, &va, &vb);
        const float v = right ? va : vb;
        if (right ? v >= lo : v <= hi) {         // (none in between)
          in = ordered_of(at);
          continue;
        }
        const Sums T = set_pass(right ? float_next_up(v) : lo, right ? hi : float_next_down(v), &na, &nc);
        const double c = sure.cnt + nc, mm = sure.m - na, d = double(v) - center;
        if (right ? P::right_violates(d, c, mm, T, R, center) : P::left_violates(d, c, mm, T, R, center)) {
          if (right) lo = v;
          else hi = v;
          in = ordered_of(at);
        } else {
          end = right ? ordered_of(v) + 1u : ordered_of(v) - 1u;
        }
      }
    }
  }
  out = Block{gamma, center, cnt, m, lo, hi, true};
  return out;
}

__device__ __forceinline__ double part_at(const double (&v)[6], int i) {
  return i == 0 ? v[0] : i == 1 ? v[1] : i == 2 ? v[2] : i == 3 ? v[3] : i == 4 ? v[4] : v[5];
}

constexpr int kListLds = 6144;                   // list entries in LDS; longer lists stay in global memory
constexpr int kListSolo = 2048;                  // lists that one wavefront solves, without barriers
constexpr int kListFlight = 8;                   // entries that a thread looks at together

struct alignas(16) WideShared {
  uint32_t bins[kFineBins];
  uint32_t sum_c[kFineBins + 1];
  double sum_b[3][kFineBins + 1];
  uint32_t scan_c[kWaves];
  double scan_b[3][kWaves];
  double red[2][kWaves][6];
  uint32_t counts[kWaves];
  uint32_t stays[kWaves];
  uint32_t last_block;
  uint32_t start[kMaxParts];
  float value[kListLds];
  uint32_t tau[kListLds];
  Block block;
};

template <bool MAG, int PC>
__global__ __launch_bounds__(kThreads) void wide_solve_kernel(
    const uint32_t* slot_val, const uint32_t* slot_idx, uint32_t* list_val, uint32_t* list_tau, uint32_t* long_val,
    uint32_t* long_tau, const float* __restrict__ tangent_all, const RowSel* __restrict__ sel, WideScratch sc,
    RowInfo* __restrict__ info, int64_t n, int64_t part_len, int parts, int group_len, int64_t k_row, Reg R) {
  using P = Pool<MAG, PC>;
  constexpr bool CUBIC = (PC == kP43);
  __shared__ WideShared sm;
  const int64_t id = die_block(blockIdx.x, gridDim.x);
  const int64_t row = id / parts;
  const int block = int(id % parts);
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  const float inf = __uint_as_float(0x7f800000u);
  SumGroup<kThreads> grp{&sm.red[0][0][0]};
  const float* tangent = tangent_all != nullptr ? tangent_all + row * n : nullptr;

  // ---- the row's counts; this wavefront's first candidates are on their way meanwhile -----------------------------
  for (int i = threadIdx.x; i < kFineBins; i += kThreads) sm.bins[i] = 0u;
  const int64_t list_at = row * n + int64_t(block) * part_len, slot = list_at + w * (part_len / kWaves);
  const uint32_t slot_len = sc.slot_count[(row * parts + block) * kWaves + w];
  uint32_t c0 = 0u, c1 = 0u, over = 0u;
  {
    const bool direct = parts <= kDirectParts, narrow = direct && part_len <= 65536;
    const int count = direct ? parts : (parts + group_len - 1) / group_len;
    const int pair = threadIdx.x % kPairs;
    const uint32_t* src = direct ? sc.part_bins + row * parts * int64_t(narrow ? kPairs : kFineBins)
                                 : sc.group_bins + row * kGroups * int64_t(kFineBins);
    for (int q0 = threadIdx.x / kPairs; q0 < count; q0 += 8 * kPartsAtOnce) {
      uint2 v[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const int from = q0 + q * kPartsAtOnce;
        v[q] = make_uint2(0u, 0u);
        if (from < count) {
          if (narrow) v[q].x = src[int64_t(from) * kPairs + pair];
          else v[q] = reinterpret_cast<const uint2*>(src + int64_t(from) * kFineBins)[pair];
        }
      }
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        const uint2 c = narrow ? unpack_counts(v[q].x) : v[q];
        c0 += c.x;
        c1 += c.y;
      }
    }
    for (int q = threadIdx.x; q < parts; q += kThreads) over += sc.above[row * parts + q];
    __syncthreads();
    atomicAdd(&sm.bins[2 * pair], c0);
    atomicAdd(&sm.bins[2 * pair + 1], c1);
  }
  constexpr int kFlight = 5;                     // candidates of a lane in registers
  uint32_t cv[kFlight], ci[kFlight];
  auto load_candidates = [&](uint32_t j0) {
#pragma unroll
    for (int i = 0; i < kFlight; ++i) {
      const uint32_t j = j0 + i * kWave + lane;
      cv[i] = j < slot_len ? slot_val[slot + j] : 0u;
      ci[i] = (tangent != nullptr && j < slot_len) ? slot_idx[slot + j] : 0u;
    }
  };
  load_candidates(0u);
  const Window win = window_of<MAG>(sel[row]);
  over = lanes_sum<kWave>(over);
  if (lane == 0) sm.counts[w] = over;
  __syncthreads();                               // the bins are there
  const uint32_t above_window = lanes_sum<kWaves>(sm.counts[lane & (kWaves - 1)]);
  // prefix sums over the bins, one bin per thread: of the counts c and, times powers of the bin's number b, of b c (p = 4/3:
  // b^2 c and b^3 c too).  sm.sum_c[j], sm.sum_b[.][j]: the bins before j.
  static_assert(kFineBins == kThreads, "one bin per thread");
  constexpr int kMoments = CUBIC ? 3 : 1;
  {
    const uint32_t c = sm.bins[threadIdx.x];
    uint32_t wave_total;
    const uint32_t inc = wave_inclusive_scan(c, &wave_total);
    const double b = double(int(threadIdx.x));
    double mo[kMoments];
    mo[0] = b * double(c);
    if (CUBIC) {
      mo[1] = b * mo[0];
      mo[2] = b * mo[1];
    }
#pragma unroll
    for (int i = 0; i < kMoments; ++i) mo[i] = wave_inclusive_scan(mo[i]);
    if (lane == kWave - 1) {
      sm.scan_c[w] = wave_total;
#pragma unroll
      for (int i = 0; i < kMoments; ++i) sm.scan_b[i][w] = mo[i];
    }
    __syncthreads();
    const uint32_t oc = lane < w ? sm.scan_c[lane & (kWaves - 1)] : 0u;
    sm.sum_c[threadIdx.x + 1] = inc + lanes_sum<kWaves>(oc);
#pragma unroll
    for (int i = 0; i < kMoments; ++i)
      sm.sum_b[i][threadIdx.x + 1] = mo[i] + lanes_sum<kWaves>(lane < w ? sm.scan_b[i][lane & (kWaves - 1)] : 0.0);
    if (threadIdx.x == 0) {
      sm.sum_c[0] = 0u;
#pragma unroll
      for (int i = 0; i < kMoments; ++i) sm.sum_b[i][0] = 0.0;
    }
    __syncthreads();
  }
  const uint32_t candidates = sm.sum_c[kFineBins];
  const double k_win = double(k_row) - double(above_window); // top-k positions in the window
  // (no more positive values than top-k positions, for the magnitude operator; NaN among the values)
  if (!(k_win >= 1.0 && k_win < double(candidates))) {
    if (block == 0 && threadIdx.x == 0) {
      RowInfo ri;
      ri.a = ri.wa = 1;
      ri.b = ri.wb = 0;
      ri.gamma = ri.center = ri.dgamma = 0.0;
      ri.hi_incl = ri.lo_incl = k_win < 1.0 ? inf : -inf;
      ri.src = ri.pad = 0;
      info[row] = ri;
    }
    return;
  }

  // ---- bracket of gamma ------------------------------------------------------------------------------------------------
  auto edge = [&](int j) { return win.base + double(j) * win.width; };
  // May gamma lie above edge j?  Psi there with every element at the lower end of its bin (upper: at the upper end), or a
  // thousandth of a bin beyond, so that an element that the rounding of its bin's number puts into the next one does no
  // harm: bin b counts clip(a (b - j + off))^(q-1), from the prefix sums.  The rounding of the moments, 3e-9 of
  // the count for p = 4/3 and nine bins, is put on the side of a wider bracket.  False from some edge on.
  auto stays = [&](int j, bool upper) -> bool {
    const double g = edge(j), off = upper ? 1.001 : -0.001;
    double h = R.inv_lambda;
    if (MAG) h = fmin(h / fmax(CUBIC ? cbrt(fmax(g, 0.0)) : g, 1e-300), 1e250);
    const double a = win.width * h;
    // bins from `first` on count, those from `full` on count 1
    const int first = upper ? j - 1 : j + 1;
    const double reach = a > 0.0 ? 1.0 / a - off : double(2 * kFineBins);
    int full = reach < double(2 * kFineBins) ? j + int(ceil(reach)) : kFineBins;
    full = full < first ? first : (full > kFineBins ? kFineBins : full);
    const int f0 = first < 0 ? 0 : (first > kFineBins ? kFineBins : first);
    full = full < f0 ? f0 : full;
    const double c = double(sm.sum_c[full] - sm.sum_c[f0]), x = off - double(j);   // sum of (a (b + x))^(q-1)
    double s = 0.0;
    if (full - f0 <= 8) {                        // (few terms, and a may be large: bin by bin)
#pragma unroll 1
      for (int b = f0; b < full; ++b) {
        const double t = a * (double(b) + x), cb = double(sm.sum_c[b + 1] - sm.sum_c[b]);
        s = fma(cb, CUBIC ? t * t * t : t, s);
      }
    } else {
      const double m1 = sm.sum_b[0][full] - sm.sum_b[0][f0];
      if constexpr (CUBIC) {
        const double m2 = sm.sum_b[1][full] - sm.sum_b[1][f0], m3 = sm.sum_b[2][full] - sm.sum_b[2][f0];
        s = ((c * x + 3.0 * m1) * x + 3.0 * m2) * x + m3;
        s = a * a * a * s;
      } else {
        s = a * (c * x + m1);
      }
    }
    // (a thousandth of a bin outside its place counts nothing, not less)
    s = fmin(fmax(s, 0.0), c) + double(candidates - sm.sum_c[full]);
    const double noise = 1e-8 * double(candidates);
    return upper ? s + noise >= k_win : s - noise > k_win;
  };
  // gamma > edge(j_lo) (-1: not known), gamma < edge(j_up)
  int j_lo, j_up;
  {
    const unsigned long long lower = __ballot(stays(int(threadIdx.x), false));
    const unsigned long long upper = __ballot(stays(int(threadIdx.x), true));
    if (lane == 0) sm.stays[w] = uint32_t(__popcll(lower)) | (uint32_t(__popcll(upper)) << 16);
    __syncthreads();
    const uint32_t all = lanes_sum<kWaves>(sm.stays[lane & (kWaves - 1)]);
    j_lo = int(all & 0xffffu) - 1;
    j_up = int(all >> 16);
    if (j_up == kFineBins) j_up = kFineBins + 1;             // (that edge itself has not been looked at)
  }
  const double g_lo = edge(j_lo), g_hi = edge(j_up);
  // Bins that may hold an element at the lower threshold, l0 .. l1, and at the upper one, h0 .. h1.  (gamma is a
  // thousandth of a bin away from the edges, and so is the upper threshold, which rises at least as fast.)
  const int l0 = j_lo, l1 = j_up - 1;
  auto bin_index = [&](double v) -> int {
    const double f = (v - win.base) * win.scale;
    return f > 0.0 ? (f < double(2 * kFineBins) ? int(f) : 2 * kFineBins) : -1;
  };
  const int h0 = bin_index(upper_end<MAG, PC>(g_lo, R)), h1 = bin_index(upper_end<MAG, PC>(g_hi, R));
  const bool none_sure = !(win.scale > 0.0);     // (a single value, or infinities: everything is listed)
  const int top = l1 > h1 ? l1 : h1;
  auto is_sure = [&](int b) { return !none_sure && b > l1 && b < h0; };
  auto is_listed = [&](int b) { return none_sure || (b >= l0 && b <= top && !is_sure(b)); };
  Sure sure;
  uint32_t len = 0u;                             // of the row's list
  {
    auto before = [&](int b) { return sm.sum_c[b < 0 ? 0 : (b > kFineBins ? kFineBins : b)]; };
    const uint32_t listed = before(top + 1) - before(l0), all_sure = !none_sure && h0 > l1 + 1 ? before(h0) - before(l1 + 1) : 0u;
    sure.cnt = double(all_sure);
    sure.m = k_win - (none_sure ? 0.0 : double(candidates - before(top + 1)));
    len = none_sure ? candidates : listed - all_sure;
  }
  sure.lo = g_lo;
  sure.hi = g_hi;
  // values are taken relative to a number of few bits near gamma: differences from inputs of few bits, and the sums
  // of their powers, are exact then, and an exact tie is seen as one
  sure.center = 0.0;
  sure.coarse = false;
  if constexpr (P::kCentered) {
    constexpr double kMax = 3.4028234663852886e38;
    if (fabs(g_lo) <= kMax && fabs(g_hi) <= kMax)
      sure.center = win.width > 0.0 ? double(simplest_between(fminf(float_above(g_lo), float(kMax)),
                                                              fmaxf(float_below(g_hi), -float(kMax))))
                                    : double(win.v_bot);
    // That number is up to two bins away from the members.  Where lambda (the reach of a block) is a small part of
    // a bin, as among masked scores of -1e30, the sums of the differences (p = 4/3: of their cubes) would lose it: the
    // centre has to be one of the elements then.  (Sure members lie a bin apart: the reach is not small.)
    // p = 4/3 loses 1e-9 at 64 reaches to a bin; p = 2 would bear 10^5, but the steps from the bracket's middle meet no
    // member from there on either (1 x 4.2 M products of normals, lambda = 1e-6: 57 us with them, 53 without).
    const double reach = MAG ? fmin(upper_end<MAG, PC>(g_lo, R) - g_lo, upper_end<MAG, PC>(g_hi, R) - g_hi) : R.lambda;
    sure.coarse = sure.cnt == 0.0 && !(win.width * (1.0 / 64.0) <= reach);
  }

  // ---- this workgroup's candidates ----------------------------------------------------------------------------------
  auto tau_of = [&](float v, uint32_t e) -> float {        // tangent in sorted-value coordinates
    float t = tangent[MAG ? (e >> 1) : e];
    if (MAG) t = v == 0.0f ? 0.0f : ((e & 1u) ? -t : t);   // sign(0) = 0
    return t;
  };
  auto sum_parts = [&](double (&v)[6]) {         // (p = 2: the values and the tangents only)
    if constexpr (CUBIC) {
      grp.sum(v);
    } else {
      double d[2] = {v[0], v[3]};
      grp.sum(d);
      v[0] = d[0];
      v[3] = d[1];
    }
  };
  double part[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
  uint32_t mine = 0u, listed_bits = 0u;          // list entries of this lane; those among the last kFlight candidates
  float ct[kFlight];
#pragma unroll 1
  for (uint32_t j0 = 0u;;) {
    uint32_t sure_bits = 0u;
    listed_bits = 0u;
#pragma unroll
    for (int i = 0; i < kFlight; ++i) {
      const int b = bin_of(double(__uint_as_float(cv[i])), win);
      const bool valid = j0 + i * kWave + lane < slot_len;
      if (valid && is_sure(b)) sure_bits |= 1u << i;
      if (valid && is_listed(b)) listed_bits |= 1u << i;
      ct[i] = 0.0f;
    }
    if (tangent != nullptr) {
#pragma unroll
      for (int i = 0; i < kFlight; ++i)
        if (((sure_bits | listed_bits) >> i) & 1u) ct[i] = tau_of(__uint_as_float(cv[i]), ci[i]);
    }
    mine += __popc(listed_bits);
#pragma unroll
    for (int i = 0; i < kFlight; ++i) {
      if ((sure_bits >> i) & 1u) {
        const double d = double(__uint_as_float(cv[i])) - sure.center, t = double(ct[i]);
        part[0] += d;
        part[3] += t;
        if (CUBIC) {
          part[1] += d * d;
          part[2] = fma(d * d, d, part[2]);
          part[4] = fma(d, t, part[4]);
          part[5] = fma(d * d, t, part[5]);
        }
      }
    }
    j0 += kFlight * kWave;
    if (j0 >= slot_len) break;
    load_candidates(j0);
  }
  // list entries of the workgroup, wavefront after wavefront
  const uint32_t wave_listed = lanes_sum<kWave>(mine);
  if (lane == 0) sm.counts[w] = wave_listed;     // (its last readers have passed the barriers of the search)
  sum_parts(part);                               // (with a barrier)
  uint32_t at = 0u, listed = 0u;
#pragma unroll
  for (int q = 0; q < kWaves; ++q) {
    const uint32_t c = sm.counts[q];
    at += q < w ? c : 0u;
    listed += c;
  }
  if (wave_listed > 0u) {
    auto put = [&](bool take, uint32_t v, float t) {
      const unsigned long long mask = __ballot(take);
      if (take) {
        const uint32_t to = at + __popcll(mask & lanemask_lt());
        publish(list_val + list_at + to, v);
        if (tangent != nullptr) publish(list_tau + list_at + to, __float_as_uint(t));
      }
      at += __popcll(mask);
    };
    if (slot_len <= uint32_t(kFlight * kWave)) {             // (they are all in registers)
#pragma unroll
      for (int i = 0; i < kFlight; ++i) put((listed_bits >> i) & 1u, cv[i], ct[i]);
    } else {
      for (uint32_t j0 = 0; j0 < slot_len; j0 += kWave) {
        const uint32_t j = j0 + lane;
        const uint32_t v = j < slot_len ? slot_val[slot + j] : 0u;
        const bool take = j < slot_len && is_listed(bin_of(double(__uint_as_float(v)), win));
        put(take, v, (take && tangent != nullptr) ? tau_of(__uint_as_float(v), slot_idx[slot + j]) : 0.0f);
      }
    }
  }
  if (threadIdx.x < 6) publish(sc.sums + (row * parts + block) * 8 + threadIdx.x, part_at(part, threadIdx.x));
  if (threadIdx.x == 6) publish(sc.listed + row * parts + block, listed);
  if (!arrive_last(&sc.arrived[row * (kSelSlices * 2 * kSel2Bins)], parts, &sm.last_block)) return;

  // ---- the last workgroup of the row: sums and list of all of them, one workgroup per thread -------------------------
  uint32_t* lv = long_val + row * n;             // (the slots: every workgroup of the row is done with them)
  uint32_t* lt = long_tau + row * n;
  const bool in_lds = len <= uint32_t(kListLds);
#pragma unroll
  for (int i = 0; i < 6; ++i) part[i] = 0.0;
  {
    const int q = int(threadIdx.x);
    uint32_t c = 0u;
    if (q < parts) {
      const double* src = sc.sums + (row * parts + q) * 8;
      c = published(sc.listed + row * parts + q);
#pragma unroll
      for (int i = 0; i < 6; ++i)
        if (CUBIC || i == 0 || i == 3) part[i] += published(src + i);
    }
    uint32_t wave_total;
    const uint32_t inc = wave_inclusive_scan(c, &wave_total);
    if (lane == 0) sm.counts[w] = wave_total;
    __syncthreads();
    uint32_t before = 0u, all = 0u;
#pragma unroll
    for (int i = 0; i < kWaves; ++i) {
      const uint32_t o = sm.counts[i];
      before += i < w ? o : 0u;
      all += o;
    }
    if (q < kMaxParts) sm.start[q] = before + inc - c;
    __syncthreads();
    for (uint32_t j = threadIdx.x; j < all; j += kThreads) {
      // the workgroup whose entries hold number j: the last start at or before it
      int from = 0, to = kMaxParts;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int mid = (from + to) / 2;
        if (sm.start[mid] <= j) from = mid;
        else to = mid;
      }
      const int64_t src = row * n + int64_t(from) * part_len + (j - sm.start[from]);
      const uint32_t v = published(list_val + src), t = tangent != nullptr ? published(list_tau + src) : 0u;
      if (in_lds) {
        if (j < uint32_t(kListLds)) {
          sm.value[j] = __uint_as_float(v);
          sm.tau[j] = t;
        }
      } else {
        lv[j] = v;
        lt[j] = t;
      }
    }
    len = all;
  }
  if (in_lds && threadIdx.x < kListFlight * kWave) {         // (up to the end of the last turn of one wavefront)
    const uint32_t j = len + threadIdx.x;
    if (j < uint32_t(kListLds)) sm.value[j] = __uint_as_float(0x7fc00000u);
  }
  sum_parts(part);                               // (with a barrier)
  sure.S = Sums{part[0], part[1], part[2]};
  if (!in_lds) {
    __threadfence_block();
    __syncthreads();
  }
  // ---- the exact solve ---------------------------------------------------------------------------------------------------
  if (in_lds && len <= uint32_t(kListSolo)) {
    if (w == 0) {
      SumGroup<kWave> one{nullptr};
      // (filled up with NaN, for which every comparison is false)
      auto each = [&](auto f) {
#pragma unroll 1
        for (uint32_t j0 = lane; j0 < len; j0 += kListFlight * kWave) {
          float v[kListFlight];
#pragma unroll
          for (int i = 0; i < kListFlight; ++i) v[i] = sm.value[j0 + i * kWave];
#pragma unroll
          for (int i = 0; i < kListFlight; ++i) f(v[i]);
        }
      };
      const Block blk = boundary_solve<MAG, PC>(one, each, len, sure, R);
      if (lane == 0) sm.block = blk;
    }
  } else {
    auto each = [&](auto f) {
      if (in_lds) {
#pragma unroll 1
        for (uint32_t j = threadIdx.x; j < len; j += kThreads) f(sm.value[j]);
      } else {
#pragma unroll 1
        for (uint32_t j0 = threadIdx.x; j0 < len; j0 += 8 * kThreads) {
          float v[8];                            // eight loads in flight
#pragma unroll
          for (int i = 0; i < 8; ++i)
            v[i] = j0 + i * kThreads < len ? __uint_as_float(lv[j0 + i * kThreads]) : 0.0f;
#pragma unroll
          for (int i = 0; i < 8; ++i)
            if (j0 + i * kThreads < len) f(v[i]);
        }
      }
    };
    const Block blk = boundary_solve<MAG, PC>(grp, each, len, sure, R);
    if (threadIdx.x == 0) sm.block = blk;
  }
  __syncthreads();
  const Block blk = sm.block;
  // ---- d gamma (Prop. 7) ----------------------------------------------------------------------------------------------------
  double dgamma = 0.0;
  if (blk.have && tangent != nullptr) {
    double d[2] = {0.0, 0.0};
    for (uint32_t j = threadIdx.x; j < len; j += kThreads) {
      const float v = in_lds ? sm.value[j] : __uint_as_float(lv[j]);
      if (v >= blk.lo && v <= blk.hi) {
        const double wgt = P::jac_weight(double(v) - blk.center, blk.gamma);
        d[0] += wgt * double(__uint_as_float(in_lds ? sm.tau[j] : lt[j]));
        d[1] += wgt;
      }
    }
    grp.sum(d);
    // the sure members' weights (gamma - s)^2 from their moments
    if (CUBIC) {
      const double g = blk.gamma, f = MAG ? 3.0 : 1.0;
      d[0] += f * ((g * part[3] - 2.0 * part[4]) * g + part[5]);
      d[1] += f * ((g * sure.cnt - 2.0 * part[0]) * g + part[1]);
    } else {
      d[0] += part[3];
      d[1] += sure.cnt;
    }
    dgamma = d[0] / P::jac_denominator(d[1], blk.m, R);
  }
  if (threadIdx.x == 0) {
    RowInfo ri;
    ri.a = ri.wa = 1;                            // (the dense pass asks only whether there is a block)
    ri.b = ri.wb = blk.have ? 1 : 0;
    ri.gamma = blk.gamma;
    ri.center = blk.center;
    ri.dgamma = dgamma;
    ri.hi_incl = blk.hi;
    ri.lo_incl = blk.lo;
    ri.src = ri.pad = 0;
    info[row] = ri;
  }
}

}  // namespace

int launch_wide_solve(bool mag, int pc, const SortBuffers& B, const float* x, const float* tangent, int64_t rows,
                      int64_t n, int64_t k, const Reg& R, hipStream_t st) {
  int64_t part_len = (n * rows + kMaxParts - 1) / kMaxParts;
  if (part_len > n) part_len = n;
  part_len = (part_len + kPart - 1) / kPart * kPart;
  const int64_t parts = (n + part_len - 1) / part_len;
  if (parts > kMaxParts || rows * parts > 0x7fffffffLL) return -1;
  const int group_len = int((parts + kGroups - 1) / kGroups);
  WideScratch sc;
  // (parts <= tiles, the 4096-element tiles that the workspace is laid out for: 32 words per part of the 256 per tile
  // of `hist`; counts: as many parts as the first histogram has, with fewer bins)
  sc.slot_count = B.hist;
  sc.sums = reinterpret_cast<double*>(B.hist + rows * parts * kWaves);
  sc.listed = B.tcnt;
  sc.above = B.tabove;
  sc.part_bins = B.hpart;
  sc.group_bins = B.bins;
  sc.arrived = B.bins2;
  const bool vec = n % 4 == 0 && (reinterpret_cast<uintptr_t>(x) & 15u) == 0;
#define TOPK_COLLECT(M, V)                                                                                       \
  hipLaunchKernelGGL((wide_collect_kernel<M, V>), dim3(unsigned(rows * parts)), dim3(kThreads), 0, st, x, B.sel, \
                     B.keys_b, B.idx_b, sc, n, part_len, int(parts), group_len)
  if (mag) {
    if (vec) TOPK_COLLECT(true, true);
    else TOPK_COLLECT(true, false);
  } else {
    if (vec) TOPK_COLLECT(false, true);
    else TOPK_COLLECT(false, false);
  }
#undef TOPK_COLLECT
#define TOPK_SOLVE(M, P)                                                                                           \
  hipLaunchKernelGGL((wide_solve_kernel<M, P>), dim3(unsigned(rows * parts)), dim3(kThreads), 0, st, B.keys_b,     \
                     B.idx_b, B.keys_a, B.idx_a, B.keys_b, B.idx_b, tangent, B.sel, sc, B.info, n, part_len,       \
                     int(parts), group_len, k, R)
  if (!mag && pc == kP2) TOPK_SOLVE(false, kP2);
  else if (!mag && pc == kP43) TOPK_SOLVE(false, kP43);
  else if (mag && pc == kP2) TOPK_SOLVE(true, kP2);
  else if (mag && pc == kP43) TOPK_SOLVE(true, kP43);
  else return -1;
#undef TOPK_SOLVE
  return 0;
}

}  // namespace topk
