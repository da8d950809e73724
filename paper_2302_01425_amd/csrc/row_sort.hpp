// Stable sort of (key, index) pairs of one row by one workgroup: short lists in LDS, longer ones through global buffers;
// shared by the one-launch kernels of medium rows and the rest of the general-weight search.
#pragma once

#include "common.hpp"
#include "launch.hpp"
#include "long_solve.hpp"
#include "radix.hpp"
#include "sort_network.hpp"
#include "wave.hpp"

namespace topk {
namespace {

// Workgroups of NT = 1024 threads for long rows; of 256 threads for rows up to kSmallRowMax
// elements, where the per-row latency is what counts and four times as many rows are in flight.
constexpr int kSmallRowMax = 8192;
constexpr int kMItems = 8;                 // elements per thread and tile of a sorting pass
constexpr int kCItems = 16;                // elements per thread and tile of the compaction
constexpr int kSelShift = 32 - kSelBits;

template <int NT>
struct MedCfg {
  static constexpr int kMW = NT / kWave;                     // wavefronts
  static constexpr int kCTile = NT * kCItems;
  static constexpr int kLdsCap = NT >= 1024 ? 2048 : 1024;   // lists up to this length are sorted in LDS
  // words of the union below: the selection histogram, later the sorted keys of a list for the solve
  static constexpr int kLdsKeys = NT >= 1024 ? 16384 : kSelBins;
};

template <int NT>
struct MedShared {
  using C = MedCfg<NT>;
  union {
    uint32_t hist[C::kLdsKeys];            // steps 1-2: kSelBins counters; later sorted keys
    struct {
      uint32_t cnt[C::kMW][kRadix];        // per-wave digit counts, then per-wave offsets
      uint32_t base[kRadix];               // running start of every digit in the output
      uint32_t gofs[kRadix];               // start of the current tile's items of every digit
      uint32_t lk[2][C::kLdsCap];          // short candidate lists: keys, ping-pong
      uint32_t li[2][C::kLdsCap];          //                        index payloads
    } sort;                                // steps 3-6
  } u;
  SolveShared<NT> solve;
  uint32_t wave_a[C::kMW], wave_b[C::kMW];
  uint32_t found[2];
};

// exclusive scan of one value per thread over the workgroup; *total gets the sum
template <int NT>
__device__ __forceinline__ uint32_t med_exclusive_scan(uint32_t v, uint32_t* wave_tot,
                                                       uint32_t* total) {
  constexpr int kMW = NT / kWave;
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  uint32_t inc = v;
#pragma unroll
  for (int off = 1; off < kWave; off <<= 1) {
    const uint32_t o = __shfl_up(inc, off, kWave);
    if (lane >= off) inc += o;
  }
  __syncthreads();
  if (lane == kWave - 1) wave_tot[w] = inc;
  __syncthreads();
  uint32_t before = 0, all = 0;
#pragma unroll
  for (int q = 0; q < kMW; ++q) {
    const uint32_t t = wave_tot[q];
    if (q < w) before += t;
    all += t;
  }
  if (total) *total = all;
  return before + inc - v;
}

// One LSD pass over the cn candidates: (kin, iin) -> (kout, iout), stable, by the 8-bit digit of
// (key - klo) at `shift`.  Tiles of ni*1024 elements; wave w owns elements w*ni*64 .. of a tile.
template <int NT, int ITEMS>
__device__ __forceinline__ void med_sort_pass(const uint32_t* kin, const uint32_t* iin, uint32_t* kout,
                              uint32_t* iout, uint32_t cn, uint32_t klo, int shift, int ni,
                              MedShared<NT>& sm) {
  constexpr int kMT = NT, kMW = NT / kWave;
  const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
  const uint32_t tile_elems = uint32_t(ni) * kMT;
  const uint32_t wave_elems = uint32_t(ni) * kWave;
  // several tiles: digit totals of the whole list first -> start of every digit (a single tile
  // gets them from its own ranking below)
  const bool single = cn <= tile_elems;
  if (!single) {
    for (int i = threadIdx.x; i < kMW * kRadix; i += kMT) (&sm.u.sort.cnt[0][0])[i] = 0;
    __syncthreads();
    for (uint32_t tile_first = 0; tile_first < cn; tile_first += tile_elems) {
#pragma unroll
      for (int i = 0; i < ITEMS; ++i) {
        if (i < ni) {
          const uint32_t e = tile_first + w * wave_elems + i * kWave + lane;
          const bool valid = e < cn;
          const uint32_t key = valid ? kin[e] : 0u;
          count_digit(sm.u.sort.cnt[w], ((key - klo) >> shift) & (kRadix - 1), valid, lane);
        }
      }
    }
    __syncthreads();
    uint32_t tot = 0;
    if (threadIdx.x < kRadix) {
#pragma unroll
      for (int q = 0; q < kMW; ++q) tot += sm.u.sort.cnt[q][threadIdx.x];
    }
    const uint32_t ex = med_exclusive_scan<NT>(tot, sm.wave_a, nullptr);
    if (threadIdx.x < kRadix) sm.u.sort.base[threadIdx.x] = ex;
  }
  // tile by tile: rank inside the wavefront, offsets of the wavefronts, scatter
  for (uint32_t tile_first = 0; tile_first < cn; tile_first += tile_elems) {
    __syncthreads();                       // previous users of cnt / gofs are done
    for (int i = threadIdx.x; i < kMW * kRadix; i += kMT) (&sm.u.sort.cnt[0][0])[i] = 0;
    __syncthreads();
    uint32_t key[ITEMS], idx[ITEMS], rank[ITEMS];
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      if (i < ni) {
        const uint32_t e = tile_first + w * wave_elems + i * kWave + lane;
        const bool valid = e < cn;
        key[i] = valid ? kin[e] : 0u;
        idx[i] = valid ? iin[e] : 0u;
        const uint32_t d = ((key[i] - klo) >> shift) & (kRadix - 1);
        const unsigned long long peers = match_digit(d, __ballot(valid));
        const unsigned long long lower = peers & lanemask_lt();
        uint32_t pre = 0;
        if (valid) {
          pre = sm.u.sort.cnt[w][d];
          if (lower == 0) sm.u.sort.cnt[w][d] = pre + __popcll(peers);
        }
        rank[i] = pre + __popcll(lower);
      }
    }
    __syncthreads();
    uint32_t run = 0;
    if (threadIdx.x < kRadix) {
#pragma unroll
      for (int q = 0; q < kMW; ++q) {
        const uint32_t c = sm.u.sort.cnt[q][threadIdx.x];
        sm.u.sort.cnt[q][threadIdx.x] = run;
        run += c;
      }
    }
    if (single) {
      const uint32_t ex = med_exclusive_scan<NT>(run, sm.wave_a, nullptr);
      if (threadIdx.x < kRadix) sm.u.sort.gofs[threadIdx.x] = ex;
    } else if (threadIdx.x < kRadix) {
      const uint32_t b = sm.u.sort.base[threadIdx.x];
      sm.u.sort.gofs[threadIdx.x] = b;
      sm.u.sort.base[threadIdx.x] = b + run;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      if (i < ni) {
        const uint32_t e = tile_first + w * wave_elems + i * kWave + lane;
        if (e < cn) {
          const uint32_t d = ((key[i] - klo) >> shift) & (kRadix - 1);
          const uint32_t dst = sm.u.sort.gofs[d] + sm.u.sort.cnt[w][d] + rank[i];
          kout[dst] = key[i];
          iout[dst] = idx[i];
        }
      }
    }
  }
  __syncthreads();          // workgroup-scope release/acquire: the next pass reads what this one wrote
}

// Where sort_candidates left the sorted list.
struct SortedList {
  const uint32_t* keys;   // LDS or global
  const uint32_t* idx;    // LDS or global
  int global_src;         // global copy of (keys, idx): 0 = (ka, ia), 1 = (kb, ib), -1 = none yet
  bool keys_in_lds;
};

// Stable LSD sort of the cn candidates in (ka, ia) on key - klo, one pass per 8 significant bits
// of khi - klo.  The passes alternate between two buffers: in LDS for short lists, else (kb, ib)
// and (ka, ia).
template <int NT, int ITEMS>
__device__ __forceinline__ SortedList sort_candidates(uint32_t* ka, uint32_t* ia, uint32_t* kb, uint32_t* ib,
                                      uint32_t cn, uint32_t klo, uint32_t khi, MedShared<NT>& sm) {
  constexpr int kMT = NT, kLdsCap = MedCfg<NT>::kLdsCap;
  const uint32_t span = khi - klo;
  const int nbits = span == 0 ? 0 : 32 - __clz(int(span));
  int ni = int((cn + kMT - 1) / kMT);
  ni = ni > ITEMS ? ITEMS : ni;
  if (nbits == 0) return SortedList{ka, ia, 0, false};
  const bool in_lds = cn <= uint32_t(kLdsCap);
  uint32_t* k0 = in_lds ? sm.u.sort.lk[0] : kb;
  uint32_t* i0 = in_lds ? sm.u.sort.li[0] : ib;
  uint32_t* k1 = in_lds ? sm.u.sort.lk[1] : ka;
  uint32_t* i1 = in_lds ? sm.u.sort.li[1] : ia;
  const uint32_t* kin = ka;
  const uint32_t* iin = ia;
  bool even = true;
  for (int shift = 0; shift < nbits; shift += 8) {
    uint32_t* kout = even ? k0 : k1;
    uint32_t* iout = even ? i0 : i1;
    med_sort_pass<NT, ITEMS>(kin, iin, kout, iout, cn, klo, shift, ni, sm);
    kin = kout;
    iin = iout;
    even = !even;
  }
  if (in_lds) return SortedList{kin, iin, -1, true};
  return SortedList{kin, iin, even ? 0 : 1, false};    // even: an even number of passes was made
}

// A row sorted completely by a workgroup of 1024 threads, keys and index payload into (ka, ia): up to kRowNetMax elements
// a bitonic network on (key, index) words in LDS, bound by its exchanges (4000 x 3000: 385 us, radix passes of one
// workgroup per row 510, the multi-workgroup sort 380); longer rows radix passes through (kb, ib) (64 x 40000 380 us,
// 4 x 131072 1030, where the multi-workgroup sort takes 135 on the whole chip).
constexpr int kRowNetMax = 8192;
struct RowSortNet {
  unsigned long long word[kRowNetMax];
};
__device__ __forceinline__ void row_sort(RowSortNet& sm, const float* x, uint32_t* ka, uint32_t* ia, uint32_t*, uint32_t*,
                                         int n) {
  for (int e = threadIdx.x; e < n; e += 1024) sm.word[e] = (unsigned long long)desc_key(x[e]) << 32 | uint32_t(e);
  lds_sort<1024>(sm.word, n);
  for (int e = threadIdx.x; e < n; e += 1024) {
    ka[e] = uint32_t(sm.word[e] >> 32);
    ia[e] = uint32_t(sm.word[e]);
  }
}
__device__ __forceinline__ void row_sort(MedShared<1024>& sm, const float* x, uint32_t* ka, uint32_t* ia, uint32_t* kb,
                                         uint32_t* ib, int n) {
  for (int e = threadIdx.x; e < n; e += 1024) {
    ka[e] = desc_key(x[e]);
    ia[e] = uint32_t(e);
  }
  __syncthreads();
  const SortedList sorted = sort_candidates<1024, 16>(ka, ia, kb, ib, uint32_t(n), 0u, 0xffffffffu, sm);
  if (sorted.keys != ka) {
    for (int e = threadIdx.x; e < n; e += 1024) {
      ka[e] = sorted.keys[e];
      ia[e] = sorted.idx[e];
    }
  }
}

}  // namespace
}  // namespace topk
