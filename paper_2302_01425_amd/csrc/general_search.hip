// General weights (Sec. 4), identity phi, p = 2, forward only, rows of 1025 .. kGeneralLongMax
// elements, WITHOUT a sort of the row.
//
// For p = 2 the pooled values are the slopes of the least concave majorant of the cumulative sums
// C(i) = sum_{j < i} (s_j - lambda w_j) of the sorted row (App. "PAV algorithm" solves exactly this).
// Only its vertices matter, and a row whose weights differ by more than its neighbouring values
// (relaxed ranks of many scores) has few: all but the tails of the row is one block.  Which parts of
// the row can hold a vertex follows from a histogram of its values alone:
//
//   1. one pass over the row: count and EXACT sum of every bin of the 12 leading key bits (values of
//      a bin share sign, exponent and three bits of mantissa, so the low 20 bits of mantissa are added
//      as integers; count and sum travel in one 64-bit LDS atomic)
//   2. C at the bins' ends from the exact sums and the prefix sums of w (a launch before this one);
//      majorant of these points by the merging rounds of general_w.hip, on at most 2816 points
//   3. between the ends of a bin of m values that span less than d, C exceeds its chord by at most
//      m d / 4: the sorted values sum to a concave curve with slopes in a range of d, and -lambda w
//      sums to a convex one (w is non-increasing).  A bin whose two ends lie further than that
//      below the majorant holds no vertex: it stays one item.  The other bins' values are
//      collected (second pass), sorted inside their bin, and become one item each
//   4. majorant of the items by the same rounds: the partition of the whole row
//   5. third pass: every element finds its bin, if need be its place in the bin, and its pooled value.
//      Equal values have equal outputs in whatever blocks they are, so no index is needed.
//
// One workgroup of 1024 threads per row; the second and third pass read the row from the L2.  Rows
// with more than 2816 items (tiny lambda: most elements are blocks of their own), more than 256
// rounds, values that are not finite, or weights that are not non-increasing (the first pass over the row is not
// made then, unless it is shared and runs beside the check) are left to the kernel that sorts the row
// (todo[row] = 1).
//
// 64 x 65536, lambda = 0.1: 909 us with a complete sort and the partition over all positions, 46 us
// here (54 before the first pass was shared by several workgroups, the scans left the LDS crossbar and the rows that
// are left over had one launch instead of two); 8 x 131072 72 -> 55, 64 x 8192 37 -> 31.  Bound by the vector instructions
// of the passes on the compute units that have a row (64 rows: a quarter of them; 6 and 9 us for the second and third at
// 65536), the rounds (1 to 2.5 us for a majorant of 230 items, 95 us where 67 rounds are needed) and three launches.
#include <hip/hip_runtime.h>

#include "common.hpp"
#include "pooling.hpp"
#include "launch.hpp"
#include "general_pav.hpp"
#include "sort_network.hpp"
#include "wave.hpp"

namespace topk {
namespace {

constexpr int kNT = 1024;                       // threads of a row's workgroup
constexpr int kNW = kNT / kWave;
constexpr int kItems = 2816;                    // items of a row (44 bytes of LDS each)
constexpr int kMaxRounds = 256;
// values of a bin that are ordered by counting: 62 ns for each of them (and twice that above 1024 items),
// against 8 us for the network over all items (2000 equal values: 300 us a call by counting, see the test)
constexpr uint32_t kCountMax = 64;
constexpr int kWTile = 2048;                    // positions of a tile of weights
constexpr int kWThreads = 256;
constexpr int kWPer = kWTile / kWThreads;
constexpr int kWTiles = int(kGeneralLongMax / kWTile);
constexpr int kCopies = 3;                      // copies of the histogram, lane % 3 chooses one
static_assert(kWTiles <= kWave, "a wavefront scans the tiles' totals");
static_assert(kItems <= 3 * kNT && kItems < 0xffff, "three items per thread, 16-bit item numbers");

struct SearchShared {
  // per bin: count << 40 | sum of the low 20 mantissa bits, bit 63 = the bin's values become items;
  // then the lookup: high word = first item | m << 16 (m = 0: one item), low word = cursor
  unsigned long long bins[kSelBins];
  union {
    unsigned long long extra[kCopies - 1][kSelBins];
    struct {
      DD p1[kItems + 1];                        // prefix sums of s at the items' starts
      DD pw[kItems + 1];                        // of w
    } i;
  } u;
  uint32_t pos[kItems + 1];                     // first sorted position of an item
  uint32_t key[kItems];                         // its key (bins: bin << 20; first majorant: the bin)
  uint16_t list[2][kItems + 2];                 // first items of the blocks, ping-pong
  DD toff[kWTiles + 1];                         // prefix sums of w at the tiles' starts
  DD wave_dd[kNW];
  unsigned long long wave_u[kNW];
  int nb, bad;
  uint32_t most;                                // values in the fullest bin that holds items
  struct {
    int lo, hi;                                 // every bin in between is one item
  } gap;
};
static_assert(sizeof(SearchShared) <= 160 * 1024, "LDS of a compute unit");

// Scans over the lanes by moves inside the rows of 16 lanes and three row totals, not through the LDS crossbar (a step
// of which waits some 100 cycles: the kernel below makes seven scans of six steps).
template <int OFF>
__device__ __forceinline__ DD row_shr_dd(const DD& v) {
  return DD{row_shr_f64<OFF>(v.h), row_shr_f64<OFF>(v.l)};
}
__device__ __forceinline__ DD lane_dd(const DD& v, int lane) {
  return DD{uniform_f64(v.h, lane), uniform_f64(v.l, lane)};
}
template <int LANES>
__device__ __forceinline__ DD row_inclusive_dd(DD v) {          // inside every row of 16 lanes, LANES of them used
  v = dd_add(row_shr_dd<1>(v), v);
  v = dd_add(row_shr_dd<2>(v), v);
  if constexpr (LANES > 4) {
    v = dd_add(row_shr_dd<4>(v), v);
    v = dd_add(row_shr_dd<8>(v), v);
  }
  return v;
}
// what lies in the rows of lanes before this lane's
__device__ __forceinline__ DD rows_before_dd(const DD& row_inc, int lane) {
  const DD b1 = lane_dd(row_inc, 15), b2 = dd_add(b1, lane_dd(row_inc, 31)), b3 = dd_add(b2, lane_dd(row_inc, 47));
  const DD zero{0.0, 0.0};
  return lane < 16 ? zero : (lane < 32 ? b1 : (lane < 48 ? b2 : b3));
}
__device__ __forceinline__ DD wave_inclusive_dd(const DD& v, int lane) {
  const DD in_row = row_inclusive_dd<16>(v);
  return dd_add(rows_before_dd(in_row, lane), in_row);
}
// exclusive scans of one value per thread over NW wavefronts; two barriers each
template <int NW>
__device__ __forceinline__ DD scan_dd(const DD& v, DD* wave_tot, DD* total) {
  const int lane = threadIdx.x & (kWave - 1), w = __builtin_amdgcn_readfirstlane(int(threadIdx.x) / kWave);
  const DD in_row = row_inclusive_dd<16>(v), rows = rows_before_dd(in_row, lane);
  const DD prev = dd_add(rows, row_shr_dd<1>(in_row));
  if (lane == kWave - 1) wave_tot[w] = dd_add(rows, in_row);
  __syncthreads();
  const DD tot = row_inclusive_dd<NW>(wave_tot[lane & (NW - 1)]);      // the wavefronts' totals, in the first NW lanes
  *total = lane_dd(tot, NW - 1);
  __syncthreads();
  return w > 0 ? dd_add(lane_dd(tot, w - 1), prev) : prev;
}
template <int CTRL, int ROWS>
__device__ __forceinline__ unsigned long long dpp_or0_u64(unsigned long long v) {
  return (unsigned long long)dpp_or0<CTRL, ROWS>(uint32_t(v >> 32)) << 32 | dpp_or0<CTRL, ROWS>(uint32_t(v));
}
__device__ __forceinline__ unsigned long long scan_u64(unsigned long long v, unsigned long long* wave_tot,
                                                       unsigned long long* total) {
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  unsigned long long inc = v;
  inc += dpp_or0_u64<0x111, 0xF>(inc);
  inc += dpp_or0_u64<0x112, 0xF>(inc);
  inc += dpp_or0_u64<0x114, 0xF>(inc);
  inc += dpp_or0_u64<0x118, 0xF>(inc);
  inc += dpp_or0_u64<0x142, 0xA>(inc);
  inc += dpp_or0_u64<0x143, 0xC>(inc);
  if (lane == kWave - 1) wave_tot[w] = inc;
  __syncthreads();
  unsigned long long before = 0, all = 0;
#pragma unroll
  for (int q = 0; q < kNW; ++q) {
    const unsigned long long c = wave_tot[q];
    if (q < w) before += c;
    all += c;
  }
  __syncthreads();
  *total = all;
  return before + inc - v;
}

// Prefix sums of the weights inside tiles of kWTile positions (local[r][i], i = 0 .. n), the tiles'
// totals, and whether a tile holds weights that increase or are not finite.  grid (tiles, weight rows)
// (by threads 0 .. kWThreads - 1; kTileBarriers barriers)
constexpr int kTileBarriers = 3;
__device__ __forceinline__ void weight_prefix_tile(const float* __restrict__ w, int n, int tile,
                                                   DD* __restrict__ loc, DD* __restrict__ total,
                                                   uint32_t* __restrict__ bad, DD* wave_dd, uint32_t* any) {
  const int e0 = tile * kWTile + threadIdx.x * kWPer;
  float v[kWPer];
  bool odd = false;
  float before = e0 > 0 && e0 < n ? w[e0 - 1] : 3.4028235e38f;
  DD sum{0.0, 0.0};
#pragma unroll
  for (int i = 0; i < kWPer; ++i) {
    v[i] = e0 + i < n ? w[e0 + i] : 0.0f;
    if (e0 + i < n) {
      odd = odd || !(v[i] <= before) || !(fabsf(v[i]) <= 3.4028235e38f);
      before = v[i];
    }
    sum = dd_add(sum, double(v[i]));
  }
  if (threadIdx.x == 0) *any = 0u;
  DD all;
  DD run = scan_dd<kWThreads / kWave>(sum, wave_dd, &all);
#pragma unroll
  for (int i = 0; i < kWPer; ++i) {
    if (e0 + i <= n) loc[e0 + i] = run;
    run = dd_add(run, double(v[i]));
  }
  if (odd) *any = 1u;
  __syncthreads();
  if (threadIdx.x == 0) {
    total[tile] = all;
    bad[tile] = *any;
  }
}
__global__ __launch_bounds__(kWThreads) void weight_prefix_kernel(const float* __restrict__ w_all, int n,
                                                                  DD* __restrict__ local,
                                                                  DD* __restrict__ total,
                                                                  uint32_t* __restrict__ bad) {
  __shared__ DD wave_dd[kWThreads / kWave];
  __shared__ uint32_t any;
  const int64_t r = blockIdx.y;
  weight_prefix_tile(w_all + r * n, n, blockIdx.x, local + r * (n + 1), total + r * kWTiles, bad + r * kWTiles,
                     wave_dd, &any);
}

// every element of the row, eight 16-byte loads per thread in flight where rows are aligned
template <bool VEC, class F>
__device__ __forceinline__ void each_value(const float* __restrict__ x, int n, F f) {
  if constexpr (VEC) {
    for (int e0 = 4 * int(threadIdx.x); e0 < n; e0 += 32 * kNT) {
      float4 q[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        q[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (e0 + i * 4 * kNT < n) q[i] = *reinterpret_cast<const float4*>(x + e0 + i * 4 * kNT);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if (e0 + i * 4 * kNT < n) {
          f(q[i].x);
          f(q[i].y);
          f(q[i].z);
          f(q[i].w);
        }
      }
    }
  } else {
    for (int e0 = int(threadIdx.x); e0 < n; e0 += 8 * kNT) {
      float q[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) q[i] = e0 + i * kNT < n ? x[e0 + i * kNT] : 0.0f;
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (e0 + i * kNT < n) f(q[i]);
    }
  }
}

// count << 40 | sum of the low 20 mantissa bits of every bin of the 12 leading key bits, in COPIES histograms
template <bool VEC, int COPIES>
__device__ __forceinline__ void count_values(const float* __restrict__ x, int n, unsigned long long* bins,
                                             unsigned long long (*extra)[kSelBins]) {
  const int copy = int(threadIdx.x & (kWave - 1)) % COPIES;
  unsigned long long* hist = copy == 0 ? bins : extra[copy - 1];
  each_value<VEC>(x, n, [&](float v) {
    atomicAdd(&hist[desc_key(v) >> (32 - kSelBits)],
              (1ull << 40) | (unsigned long long)(__float_as_uint(v) & 0xfffffu));
  });
}

// Few rows (fewer than compute units): the first pass over a row is shared by `parts` workgroups, whose counts the search
// kernel adds up, in the launch that makes the prefix sums of the weights.
// part_bins[row][parts][kSelBins].
template <bool VEC>
__global__ __launch_bounds__(kNT) void general_prepare_kernel(
    const float* __restrict__ x_all, const float* __restrict__ w_all, int n, int tiles, int weight_blocks,
    DD* __restrict__ local, DD* __restrict__ total, uint32_t* __restrict__ bad,
    unsigned long long* __restrict__ part_bins, int parts, int part_len) {
  constexpr int kPartCopies = 2;                 // (two workgroups to a compute unit: the weights' come on top of the parts)
  __shared__ unsigned long long bins[kSelBins], extra[kPartCopies - 1][kSelBins];
  __shared__ DD wave_dd[kWThreads / kWave];
  __shared__ uint32_t any;
  if (int(blockIdx.x) < weight_blocks) {
    if (threadIdx.x >= kWThreads) {              // (uniform over a wavefront)
#pragma unroll
      for (int i = 0; i < kTileBarriers; ++i) __syncthreads();
      return;
    }
    const int64_t r = blockIdx.x / tiles;
    weight_prefix_tile(w_all + r * n, n, int(blockIdx.x % tiles), local + r * (n + 1), total + r * kWTiles,
                       bad + r * kWTiles, wave_dd, &any);
    return;
  }
  const int64_t b = int64_t(blockIdx.x) - weight_blocks, row = b / parts;
  const int first = int(b % parts) * part_len, len = n - first < part_len ? n - first : part_len;
  for (int i = threadIdx.x; i < kSelBins; i += kNT) {
    bins[i] = 0;
#pragma unroll
    for (int c = 0; c < kPartCopies - 1; ++c) extra[c][i] = 0;
  }
  __syncthreads();
  count_values<VEC, kPartCopies>(x_all + row * n + first, len, bins, extra);
  __syncthreads();
  unsigned long long* dst = part_bins + b * kSelBins;
  for (int i = threadIdx.x; i < kSelBins; i += kNT) {
    unsigned long long h = bins[i];
#pragma unroll
    for (int c = 0; c < kPartCopies - 1; ++c) h += extra[c][i];
    dst[i] = h;
  }
}

// pooled value of the items [lo, hi) (no fused multiply-add: exact ties stay ties)
__device__ __forceinline__ double item_gamma(const SearchShared& sm, int lo, int hi, double lambda) {
  const double S = dd_diff(sm.u.i.p1[hi], sm.u.i.p1[lo]), W = dd_diff(sm.u.i.pw[hi], sm.u.i.pw[lo]);
  return __ddiv_rn(__dsub_rn(S, __dmul_rn(lambda, W)), double(sm.pos[hi] - sm.pos[lo]));
}

// Majorant of the items 0 .. T-1: rounds that remove every boundary between two blocks that violate
// (gamma_left < gamma_right), all at once, on a dense list of the blocks' first items.  Up to 64
// blocks one wavefront goes on without barriers.  Returns the number of blocks (their first items and
// T in sm.list[*which]), or -1 when kMaxRounds do not suffice.
__device__ int majorant(SearchShared& sm, int T, double lambda, int* which) {
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  for (int i = tid; i <= T; i += kNT) sm.list[0][i] = uint16_t(i);
  __syncthreads();
  int cur = 0, nb = T, rounds = 0;
  while (nb > kWave) {
    if (++rounds > kMaxRounds) return -1;
    const uint16_t* L = sm.list[cur];
    uint16_t* M = sm.list[cur ^ 1];
    const int per = (nb + kNT - 1) / kNT, i0 = tid * per;       // per <= 3
    uint32_t first[3];
    int kept = 0;
    if (i0 < nb) {
      int lo = L[i0];
      double g = i0 > 0 ? item_gamma(sm, L[i0 - 1], lo, lambda) : 0.0;
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        if (r < per && i0 + r < nb) {
          const int hi = L[i0 + r + 1];
          const double gn = item_gamma(sm, lo, hi, lambda);
          const bool gone = i0 + r > 0 && g < gn;
          first[r] = gone ? 0xffffffffu : uint32_t(lo);
          kept += !gone;
          g = gn;
          lo = hi;
        } else {
          first[r] = 0xffffffffu;
        }
      }
    }
    unsigned long long total;
    int at;
    if (per == 1) {                              // (kept is 0 or 1)
      const unsigned long long km = __ballot(kept != 0);
      if (lane == 0) sm.wave_u[tid / kWave] = __popcll(km);
      __syncthreads();
      uint32_t before = 0, all = 0;
#pragma unroll
      for (int q = 0; q < kNW; ++q) {
        const uint32_t c = uint32_t(sm.wave_u[q]);
        if (q < tid / kWave) before += c;
        all += c;
      }
      at = int(before) + __popcll(km & ((1ull << lane) - 1ull));
      total = all;
    } else {
      at = int(scan_u64(uint64_t(kept), sm.wave_u, &total));
    }
    if (i0 < nb) {
#pragma unroll
      for (int r = 0; r < 3; ++r)
        if (first[r] != 0xffffffffu) M[at++] = uint16_t(first[r]);
    }
    if (tid == 0) M[total] = uint16_t(T);
    __syncthreads();
    cur ^= 1;
    *which = cur;
    if (int(total) == nb) return nb;
    nb = int(total);
  }
  *which = cur;
  if (tid < kWave) {
    volatile uint16_t* L = sm.list[cur];
    for (;;) {                                   // every round but the last one removes a block
      const int lo = lane < nb ? L[lane] : T, hi = lane < nb ? L[lane + 1] : T;
      const double g = lane < nb ? item_gamma(sm, lo, hi, lambda) : 0.0;
      const double g15 = uniform_f64(g, 15), g31 = uniform_f64(g, 31), g47 = uniform_f64(g, 47);
      double gp = row_shr_f64<1>(g);             // (of the lane before)
      if ((lane & 15) == 0) gp = lane < 32 ? g15 : (lane < 48 ? g31 : g47);
      const bool keep = lane < nb && !(lane > 0 && gp < g);
      const unsigned long long km = __ballot(keep);
      const int left = __popcll(km);
      if (left == nb) break;
      __builtin_amdgcn_wave_barrier();
      if (keep) L[__popcll(km & ((1ull << lane) - 1ull))] = uint16_t(lo);
      if (lane == 0) L[left] = uint16_t(T);
      nb = left;
      __builtin_amdgcn_wave_barrier();
    }
    if (lane == 0) sm.nb = nb;
  }
  __syncthreads();
  nb = sm.nb;
  return nb;
}

// block of item i: the last list entry that is <= i
__device__ __forceinline__ int block_of(const uint16_t* L, int nb, int i) {
  int a = 0, b = nb;                             // L[a] <= i < L[b]
  while (b - a > 1) {
    const int m = (a + b) >> 1;
    if (int(L[m]) <= i) a = m;
    else b = m;
  }
  return a;
}

template <bool VEC>
__global__ __launch_bounds__(kNT) void general_search_kernel(
    const float* __restrict__ x_all, const float* __restrict__ w_all, int64_t w_stride,
    const DD* __restrict__ wlocal, const DD* __restrict__ wtotal, const uint32_t* __restrict__ wbad,
    float* __restrict__ out_all, uint32_t* __restrict__ todo, const unsigned long long* __restrict__ part_bins,
    int parts, int n, double lambda, double inv_lambda) {
  __shared__ SearchShared sm;
  const int64_t row = blockIdx.x, wrow = w_stride != 0 ? row : 0;
  const float* x = x_all + row * n;
  float* out = out_all + row * n;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  const DD* wl = wlocal + wrow * (n + 1);
  const int tiles = (n + kWTile - 1) / kWTile;

  // ---- 1. histogram with sums; the tiles' offsets of the prefix sums of w ---------------------------
  DD tile_total{0.0, 0.0};
  bool tile_bad = false;
  if (tid < kWave && lane < tiles) {
    tile_total = wtotal[wrow * kWTiles + lane];
    tile_bad = wbad[wrow * kWTiles + lane] != 0;
  }
  if (parts == 1) {
    for (int i = tid; i < kSelBins; i += kNT) {
      sm.bins[i] = 0;
#pragma unroll
      for (int c = 0; c < kCopies - 1; ++c) sm.u.extra[c][i] = 0;
    }
  }
  if (tid < kWave) {
    const bool bad = __any(tile_bad);
    if (lane == 0) sm.bad = bad;
  }
  if (tid == 0) {
    sm.gap = {-1, kSelBins};
    sm.most = 0;
  }
  __syncthreads();
  if (sm.bad) {                                  // weights that are not non-increasing: nothing to look for
    if (tid == 0) todo[row] = 1;
    return;
  }
  if (parts == 1) count_values<VEC, kCopies>(x, n, sm.bins, sm.u.extra);
  if (tid < kWave) {
    const DD t = wave_inclusive_dd(tile_total, lane);
    if (lane < tiles) sm.toff[lane + 1] = t;
    if (lane == 0) sm.toff[0] = DD{0.0, 0.0};
  }
  __syncthreads();

  // ---- 2. my four bins: counts, exact sums, positions; majorant of the bins' ends -------------------
  constexpr int kPer = kSelBins / kNT;
  uint32_t cnt[kPer];
  double sum[kPer];
  uint32_t mine = 0, used = 0;
  DD mysum{0.0, 0.0};
  bool bad = false;
  unsigned long long hsum[kPer];
#pragma unroll
  for (int q = 0; q < kPer; ++q) hsum[q] = 0;
  if (parts == 1) {
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      hsum[q] = sm.bins[tid * kPer + q];
#pragma unroll
      for (int c = 0; c < kCopies - 1; ++c) hsum[q] += sm.u.extra[c][tid * kPer + q];
    }
  } else {
    const ulonglong2* src = reinterpret_cast<const ulonglong2*>(part_bins + row * parts * kSelBins + tid * kPer);
    for (int q0 = 0; q0 < parts; q0 += 4) {      // eight 16-byte loads in flight
      ulonglong2 h[4][kPer / 2];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int q = 0; q < kPer / 2; ++q)
          h[i][q] = q0 + i < parts ? src[int64_t(q0 + i) * (kSelBins / 2) + q] : make_ulonglong2(0ull, 0ull);
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int q = 0; q < kPer / 2; ++q) {
          hsum[2 * q] += h[i][q].x;
          hsum[2 * q + 1] += h[i][q].y;
        }
    }
  }
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    const uint32_t b = uint32_t(tid * kPer + q);
    const unsigned long long h = hsum[q];
    cnt[q] = uint32_t(h >> 40);
    const uint32_t top = b >= uint32_t(kSelBins) / 2 ? b : (~b & 0x7ffu);     // leading bits of the float
    const uint32_t e = (top >> 3) & 0xffu;
    const double ulp = __longlong_as_double((long long)((e ? e : 1u) + 1023u - 150u) << 52);
    const unsigned long long m = (unsigned long long)cnt[q] * (((top & 7u) << 20) | (e ? 1u << 23 : 0u)) +
                                 (h & 0xffffffffffull);
    sum[q] = double(m) * ((top & 0x800u) ? -ulp : ulp);
    if (cnt[q] != 0 && e == 255u) bad = true;
    mine += cnt[q];
    used += cnt[q] != 0;
    mysum = dd_add(mysum, sum[q]);
  }
  unsigned long long tot64;
  const unsigned long long ex = scan_u64((unsigned long long)used << 32 | mine, sm.wave_u, &tot64);
  const uint32_t my_pos = uint32_t(ex);
  const int nbins = int(tot64 >> 32);
  DD total_s;
  const DD my_s = scan_dd<kNW>(mysum, sm.wave_dd, &total_s);
  if (__syncthreads_or(bad || nbins > kItems)) {
    if (tid == 0) todo[row] = 1;
    return;
  }
  // prefix sums of w at position p < n: the tile's offset and what w_local reads
  auto w_local = [&](uint32_t p) -> DD { return wl[p < uint32_t(n) ? p : uint32_t(n) - 1u]; };
  auto w_prefix = [&](uint32_t p, const DD& local) -> DD { return dd_add(sm.toff[p / kWTile], local); };
  {
    uint32_t p = my_pos;
    int it = int(ex >> 32);
    DD s = my_s;
    DD wp[kPer];                                 // (all loads in flight before the first store)
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      wp[q] = w_local(p);
      p += cnt[q];
    }
    p = my_pos;
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      if (cnt[q] != 0) {
        sm.pos[it] = p;
        sm.key[it] = uint32_t(tid * kPer + q);
        sm.u.i.p1[it] = s;
        sm.u.i.pw[it] = w_prefix(p, wp[q]);
        ++it;
        p += cnt[q];
        s = dd_add(s, sum[q]);
      }
      sm.bins[tid * kPer + q] = 0;
    }
    if (tid == 0) {
      sm.pos[nbins] = uint32_t(n);
      sm.u.i.p1[nbins] = total_s;
      sm.u.i.pw[nbins] = sm.toff[tiles];
    }
  }
  __syncthreads();
  int which = 0;
  int nb = majorant(sm, nbins, lambda, &which);
  if (nb < 0) {
    if (tid == 0) todo[row] = 1;
    return;
  }

  // ---- 3. bins that may hold a vertex inside --------------------------------------------------------
  {
    const float* w = w_all + wrow * w_stride;
    const double wmax = fmax(fabs(double(w[0])), fabs(double(w[n - 1])));
    const double smax = fmax(fabs(double(key_to_float(sm.key[0] << 20))),
                             fabs(double(key_to_float((sm.key[nbins - 1] << 20) | 0xfffffu))));
    // rounding of the distances below, whose terms are at most this large: 2^-53 of it, some tens of
    // times; 1e-13 leaves a factor of ten
    const double eps = 1e-13 * double(n) * (smax + lambda * wmax);
    const uint16_t* L = sm.list[which];
    for (int i = tid; i < nbins; i += kNT) {
      const uint32_t m = sm.pos[i + 1] - sm.pos[i];
      if (m < 2) continue;
      const int j = block_of(L, nb, i), a = L[j];
      const double g = item_gamma(sm, a, L[j + 1], lambda);
      auto below = [&](int q) -> double {      // of C under the majorant, at the start of item q
        const double c = dd_diff(sm.u.i.p1[q], sm.u.i.p1[a]) - lambda * dd_diff(sm.u.i.pw[q], sm.u.i.pw[a]);
        return g * double(sm.pos[q] - sm.pos[a]) - c;
      };
      const double gap = fmin(below(i), below(i + 1));
      const uint32_t b = sm.key[i];
      const uint32_t e = ((b >= uint32_t(kSelBins) / 2 ? b : ~b) >> 3) & 0xffu;
      const double width = __longlong_as_double((long long)((e ? e : 1u) + 1023u - 130u) << 52);
      if (!(gap > 0.25 * double(m) * width + eps)) sm.bins[b] = 1ull << 63;
    }
  }
  __syncthreads();

  // ---- 4. items: bins without a vertex inside, and the values of the others ------------------------------
  bool open[kPer];
  uint32_t ni = 0, nc = 0, at = my_pos;
#pragma unroll
  for (int q = 0; q < kPer; ++q) {
    open[q] = sm.bins[tid * kPer + q] != 0;
    ni += open[q] ? cnt[q] : (cnt[q] != 0 ? 1u : 0u);
    nc += open[q] ? cnt[q] : 0u;
    // the nearest open bins around the middle of the row
    if (open[q]) {
      atomicMax(&sm.most, cnt[q]);
      if (at + cnt[q] <= uint32_t(n) / 2) atomicMax(&sm.gap.lo, tid * kPer + q);
      else atomicMin(&sm.gap.hi, tid * kPer + q);
    }
    at += cnt[q];
  }
  const unsigned long long ex2 = scan_u64((unsigned long long)nc << 32 | ni, sm.wave_u, &tot64);
  const uint32_t cands = uint32_t(tot64 >> 32);
  const int T = cands > uint32_t(kItems) ? kItems + 1 : int(uint32_t(tot64));
  if (T > kItems) {
    if (tid == 0) todo[row] = 1;
    return;
  }
  uint32_t* lookup = reinterpret_cast<uint32_t*>(sm.bins);      // [2 b] cursor, [2 b + 1] the rest
  {
    uint32_t it = uint32_t(ex2);
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
      const uint32_t b = uint32_t(tid * kPer + q);
      if (cnt[q] == 0) continue;
      lookup[2 * b] = it;
      lookup[2 * b + 1] = it | (open[q] ? cnt[q] << 16 : 0u);
      if (open[q]) {
        it += cnt[q];
      } else {
        sm.key[it] = b << 20;
        sm.pos[it] = cnt[q];
        sm.u.i.p1[it] = DD{sum[q], 0.0};
        ++it;
      }
    }
  }
  __syncthreads();
  // bins strictly between these hold no separate values (most of the row: neither pass below looks
  // them up one by one)
  const int open_lo = sm.gap.lo, open_hi = sm.gap.hi;
  const uint32_t gap0 = uint32_t(open_lo + 1), gap_n = uint32_t(open_hi - open_lo - 1);
  // its first and last item
  const uint32_t l_lo = open_lo >= 0 ? lookup[2 * open_lo + 1] : 0u;
  const int gap_first = int((l_lo & 0xffffu) + (l_lo >> 16));
  const int gap_last = (open_hi < kSelBins ? int(lookup[2 * open_hi + 1] & 0xffffu) : T) - 1;
  if (cands != 0) {
    each_value<VEC>(x, n, [&](float v) {
      const uint32_t key = desc_key(v), b = key >> 20;
      if (b - gap0 >= gap_n && (lookup[2 * b + 1] >> 16)) sm.key[atomicAdd(&lookup[2 * b], 1u)] = key;
    });
    __syncthreads();
    uint32_t k[3], dst[3];
    if (sm.most <= kCountMax) {
      // order inside a bin by counting (a few dozen values: the row's weights separate the rest)
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        const uint32_t t = uint32_t(tid + r * kNT);
        dst[r] = 0xffffffffu;
        if (t < uint32_t(T)) {
          k[r] = sm.key[t];
          const uint32_t l = lookup[2 * (k[r] >> 20) + 1], m = l >> 16, at = l & 0xffffu;
          if (m != 0) {
            uint32_t less = 0;
            for (uint32_t j = at; j < at + m; ++j) {
              const uint32_t o = sm.key[j];
              less += (o < k[r] || (o == k[r] && j < t)) ? 1u : 0u;
            }
            dst[r] = at + less;
          }
        }
      }
    } else {
      // full bins (many equal values): the items are in the order of their bins, one network over all of them
      // leaves the bins in place and orders the values inside
      lds_sort<kNT>(sm.key, T);
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        const uint32_t t = uint32_t(tid + r * kNT);
        dst[r] = 0xffffffffu;
        if (t < uint32_t(T)) {
          k[r] = sm.key[t];
          if (lookup[2 * (k[r] >> 20) + 1] >> 16) dst[r] = t;
        }
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      if (dst[r] != 0xffffffffu) {
        sm.key[dst[r]] = k[r];
        sm.pos[dst[r]] = 1;
        sm.u.i.p1[dst[r]] = DD{double(key_to_float(k[r])), 0.0};
      }
    }
    __syncthreads();
  }
  {
    // counts and sums of the items -> positions and prefix sums
    uint32_t c[3], cs = 0;
    DD v[3], vs{0.0, 0.0};
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      const int t = 3 * tid + r;
      c[r] = t < T ? sm.pos[t] : 0u;
      v[r] = t < T ? sm.u.i.p1[t] : DD{0.0, 0.0};
      cs += c[r];
      vs = dd_add(vs, v[r]);
    }
    uint32_t p = uint32_t(scan_u64(cs, sm.wave_u, &tot64));
    DD wp[3];
    {
      uint32_t q = p;
#pragma unroll
      for (int r = 0; r < 3; ++r) {
        wp[r] = w_local(q);
        q += c[r];
      }
    }
    DD s = scan_dd<kNW>(vs, sm.wave_dd, &total_s);
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      const int t = 3 * tid + r;
      if (t < T) {
        sm.pos[t] = p;
        sm.u.i.p1[t] = s;
        sm.u.i.pw[t] = w_prefix(p, wp[r]);
      }
      p += c[r];
      s = dd_add(s, v[r]);
    }
    if (tid == 0) {
      sm.pos[T] = uint32_t(n);
      sm.u.i.p1[T] = total_s;
      sm.u.i.pw[T] = sm.toff[tiles];
    }
  }
  __syncthreads();
  nb = majorant(sm, T, lambda, &which);
  if (nb < 0) {
    if (tid == 0) todo[row] = 1;
    return;
  }
  // pooled value of every item
  double* gi = reinterpret_cast<double*>(sm.u.i.p1);
  {
    const uint16_t* L = sm.list[which];
    double g[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
      const int t = 3 * tid + r;
      g[r] = 0.0;
      if (t < T) {
        const int j = block_of(L, nb, t);
        g[r] = item_gamma(sm, L[j], L[j + 1], lambda);
      }
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 3; ++r)
      if (3 * tid + r < T) gi[3 * tid + r] = g[r];
  }
  __syncthreads();

  // ---- 5. outputs y = (s - gamma) / lambda --------------------------------------------------------------
  // (pooled values never rise from item to item: equal at both ends, equal in between)
  const bool one_block = gap_first <= gap_last && gi[gap_first] == gi[gap_last];
  const double gap_gamma = one_block ? gi[gap_first] : 0.0;
  const uint32_t same_n = one_block ? gap_n : 0u;
  auto value = [&](float v) -> float {
    const uint32_t key = desc_key(v);
    if ((key >> 20) - gap0 < same_n) return float((double(v + 0.0f) - gap_gamma) * inv_lambda);
    const uint32_t l = lookup[2 * (key >> 20) + 1];
    uint32_t at = l & 0xffffu;
    if (l >> 16) {
      uint32_t end = at + (l >> 16);             // first item of the bin whose key is not smaller
      while (at < end) {
        const uint32_t m = (at + end) >> 1;
        if (sm.key[m] < key) at = m + 1;
        else end = m;
      }
    }
    return float((double(v + 0.0f) - gi[at]) * inv_lambda);
  };
  if constexpr (VEC) {
    for (int e0 = 4 * tid; e0 < n; e0 += 32 * kNT) {
      float4 q[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        q[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (e0 + i * 4 * kNT < n) q[i] = *reinterpret_cast<const float4*>(x + e0 + i * 4 * kNT);
      }
#pragma unroll
      for (int i = 0; i < 8; ++i)
        if (e0 + i * 4 * kNT < n)
          *reinterpret_cast<float4*>(out + e0 + i * 4 * kNT) =
              make_float4(value(q[i].x), value(q[i].y), value(q[i].z), value(q[i].w));
    }
  } else {
    for (int e = tid; e < n; e += kNT) out[e] = value(x[e]);
  }
  if (tid == 0) todo[row] = 0;
}

}  // namespace

int launch_general_search(const GeneralBuffers& gb, const SortBuffers& B, const float* x,
                          const float* w, int64_t w_stride, float* out, int64_t rows, int64_t n,
                          const Reg& R, hipStream_t st, const uint32_t** todo) {
  if (n <= 1024 || n > kGeneralLongMax || rows > 0x7fffffffLL) return -1;
  const int64_t wrows = w_stride != 0 ? rows : 1;
  if (wrows > 65535) return -1;
  // scratch: the prefix sums of w where the kernel of the rounds keeps its own, the tiles' totals and
  // marks at the front of arrays that only that kernel uses afterwards; the rows' marks outlive it
  DD* total = gb.p1;
  uint32_t* bad = gb.hi_of;
  const int tiles = int((n + kWTile - 1) / kWTile);
  const bool vec = n % 4 == 0 && ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(out)) & 15) == 0;
  // parts of a row that the first pass is shared by: as many as there are compute units for each row, of at least
  // 8192 elements (below, the 32 KB of counts of a part cost as much as its elements), at most as many as B.bins has room
  // for (64 x 65536, lambda = 0.1: 45.9 us in this kernel with one workgroup
  // per row, 38.7 with four, and 5.4 / 9.2 in the launch before it)
  static_assert(kSelSlices * kSelBins * 4 >= 8 * kSelBins * 8, "eight parts");
  int64_t parts = 256 / rows;
  if (parts > n / 8192) parts = n / 8192;
  parts = parts > 8 ? 8 : (parts < 1 ? 1 : parts);
  int64_t part_len = (n + parts - 1) / parts;
  part_len = (part_len + 3) / 4 * 4;
  unsigned long long* part_bins = reinterpret_cast<unsigned long long*>(B.bins);
  // (n a multiple of the tile: one more tile would hold position n alone, which is never looked up)
  if (parts > 1) {
    const int weight_blocks = int(wrows) * tiles;
    const dim3 grid{unsigned(weight_blocks + rows * parts)};
    if (vec)
      hipLaunchKernelGGL(general_prepare_kernel<true>, grid, dim3(kNT), 0, st, x, w, int(n), tiles, weight_blocks,
                         gb.pw, total, bad, part_bins, int(parts), int(part_len));
    else
      hipLaunchKernelGGL(general_prepare_kernel<false>, grid, dim3(kNT), 0, st, x, w, int(n), tiles, weight_blocks,
                         gb.pw, total, bad, part_bins, int(parts), int(part_len));
  } else {
    hipLaunchKernelGGL(weight_prefix_kernel, dim3(unsigned(tiles), unsigned(wrows)), dim3(kWThreads), 0, st,
                       w, int(n), gb.pw, total, bad);
  }
  if (vec)
    hipLaunchKernelGGL(general_search_kernel<true>, dim3(unsigned(rows)), dim3(kNT), 0, st, x, w, w_stride,
                       gb.pw, total, bad, out, B.dtot, part_bins, int(parts), int(n), R.lambda, R.inv_lambda);
  else
    hipLaunchKernelGGL(general_search_kernel<false>, dim3(unsigned(rows)), dim3(kNT), 0, st, x, w, w_stride,
                       gb.pw, total, bad, out, B.dtot, part_bins, int(parts), int(n), R.lambda, R.inv_lambda);
  *todo = B.dtot;
  return 0;
}

}  // namespace topk
