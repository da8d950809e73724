// The register-resident sorting network of the short-row kernels and the packing of
// (descending-order key, index field) into one float64 (see short_rows.hip for the layout).
#pragma once

#include "common.hpp"
#include "wave.hpp"

namespace topk {

// ---- the sorting network ---------------------------------------------------------------------
// One stage: every position p is compared with p ^ M; the lower position keeps the minimum.
// p = lane*E + r, so M splits into a register mask (M mod E) and a lane mask (M / E).
template <int GL, int E, int M>
__device__ __forceinline__ void sort_stage(double (&K)[E], int lr) {
  constexpr int RM = M & (E - 1);
  constexpr int LM = M / E;
  if constexpr (LM == 0) {
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const int r2 = r ^ RM;
      if (r < r2) {
        const double lo = min_f64(K[r], K[r2]);
        const double hi = max_f64(K[r], K[r2]);
        K[r] = lo;
        K[r2] = hi;
      }
    }
  } else {
    const bool low = (lr & top_bit(LM)) == 0;
    double O[E];
#pragma unroll
    for (int r = 0; r < E; ++r) O[r] = lane_xor_f64<LM>(K[r ^ RM]);
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const bool o_lt = O[r] < K[r];
      K[r] = (o_lt == low) ? O[r] : K[r];
    }
  }
}

template <int GL, int E, int M>
__device__ __forceinline__ void sort_stage(uint32_t (&K)[E], int lr);

template <int GL, int E, int STRIDE>
struct HalfCleaners {
  template <class T>
  static __device__ __forceinline__ void run(T (&K)[E], int lr) {
    sort_stage<GL, E, STRIDE>(K, lr);
    HalfCleaners<GL, E, STRIDE / 2>::run(K, lr);
  }
};
template <int GL, int E>
struct HalfCleaners<GL, E, 0> {
  template <class T>
  static __device__ __forceinline__ void run(T (&)[E], int) {}
};

// Bitonic merge sort in its "mirror" form: merging two sorted runs of SIZE/2 starts with the
// comparison p <-> p ^ (SIZE-1), then half-cleaners of stride SIZE/4 .. 1; every compare-exchange
// is ascending.
template <int GL, int E, int SIZE>
struct SortRuns {
  template <class T>
  static __device__ __forceinline__ void run(T (&K)[E], int lr) {
    SortRuns<GL, E, SIZE / 2>::run(K, lr);
    sort_stage<GL, E, SIZE - 1>(K, lr);
    HalfCleaners<GL, E, SIZE / 4>::run(K, lr);
  }
};
template <int GL, int E>
struct SortRuns<GL, E, 1> {
  template <class T>
  static __device__ __forceinline__ void run(T (&)[E], int) {}
};

// The same network on 32-bit words: an exchange inside a lane is two instructions, one between lanes a move and a median
// (of the two words and the end of the range that the lane's side is to take).  The float64 form takes two to three
// times as long (minima and moves of two registers each, select by comparison).
// (written out and not as assembly: the moves that read the result in the next stage need two instructions in between,
// which the compiler sees to for its own instructions only)
__device__ __forceinline__ uint32_t median_u32(uint32_t a, uint32_t b, uint32_t c) {
  return max(min(a, b), min(max(a, b), c));
}
template <int GL, int E, int M>
__device__ __forceinline__ void sort_stage(uint32_t (&K)[E], int lr) {
  constexpr int RM = M & (E - 1);
  constexpr int LM = M / E;
  if constexpr (LM == 0) {
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const int r2 = r ^ RM;
      if (r < r2) {
        const uint32_t lo = min(K[r], K[r2]), hi = max(K[r], K[r2]);
        K[r] = lo;
        K[r2] = hi;
      }
    }
  } else {
    const uint32_t end = (lr & top_bit(LM)) == 0 ? 0u : 0xffffffffu;
    uint32_t O[E];
#pragma unroll
    for (int r = 0; r < E; ++r) O[r] = lane_xor<LM>(K[r ^ RM]);
#pragma unroll
    for (int r = 0; r < E; ++r) K[r] = median_u32(K[r], O[r], end);
  }
}

// ---- packing -----------------------------------------------------------------------------------
template <int IDXB>
__device__ __forceinline__ double pack(uint32_t key, uint32_t field) {
  const uint32_t lo = (key << IDXB) | field;
  const uint32_t hi = 0x43300000u | (key >> (32 - IDXB));
  return __hiloint2double(int(hi), int(lo));
}
template <int IDXB>
__device__ __forceinline__ void unpack(double c, uint32_t& key, uint32_t& field) {
  const uint32_t lo = uint32_t(__double2loint(c)), hi = uint32_t(__double2hiint(c));
  key = (hi << (32 - IDXB)) | (lo >> IDXB);
  field = lo & ((1u << IDXB) - 1u);
}

// the same for a row dealt to the lanes by elem_of<GL, E, VEC>
template <int GL, int E, bool VEC, bool MAG, int IDXB>
__device__ __forceinline__ void make_keys_row(const float (&v)[E], int lr, int n, double (&K)[E]) {
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int e = elem_of<GL, E, VEC>(lr, r);
    uint32_t key = kSentinelKey, field = (1u << IDXB) - 1u;
    if (e < n) {
      if (MAG) {
        field = (uint32_t(e) << 1) | (__float_as_uint(v[r]) >> 31);
        key = desc_key(fabsf(v[r]));
      } else {
        field = uint32_t(e);
        key = desc_key(v[r]);
      }
    }
    K[r] = pack<IDXB>(key, field);
  }
}

template <int E, bool MAG, int IDXB>
__device__ __forceinline__ void make_keys(const float (&v)[E], int e0, int n, double (&K)[E]) {
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const int e = e0 + r;
    uint32_t key = kSentinelKey, field = (1u << IDXB) - 1u;
    if (e < n) {
      if (MAG) {
        field = (uint32_t(e) << 1) | (__float_as_uint(v[r]) >> 31);
        key = desc_key(fabsf(v[r]));
      } else {
        field = uint32_t(e);
        key = desc_key(v[r]);
      }
    }
    K[r] = pack<IDXB>(key, field);
  }
}


// Ascending sort of w[0, n) in LDS by NT threads (all of them call it, n >= 2 uniform, NT a multiple of 64): the
// bitonic network in mirror form, in which the smaller word always moves down; words beyond n would count as
// largest and are not there.  A wavefront's 64 exchanges of a stage with s <= 64 stay inside 128 words, so that
// barriers are needed around the longer ones only (15 of the 78 stages of 4096 words).
template <int NT, class T>
__device__ __forceinline__ void lds_sort(T* w, int n) {
  const int pairs = 1 << (31 - __clz(n - 1));          // half the next power of two
#pragma unroll 1
  for (int size = 2; size <= 2 * pairs; size <<= 1) {
    if (size == 2 || size >= 256) __syncthreads();
#pragma unroll 1
    for (int s = size >> 1; s >= 1; s >>= 1) {
      for (int p = threadIdx.x; p < pairs; p += NT) {
        const int off = p & (s - 1), a = (p - off) * 2 + off, b = s == size >> 1 ? a + size - 1 - 2 * off : a + s;
        if (b < n) {
          const T wa = w[a], wb = w[b];
          if (wa > wb) {
            w[a] = wb;
            w[b] = wa;
          }
        }
      }
      if (s >= 128) {
        __syncthreads();
      } else {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
      }
    }
  }
  __syncthreads();
}

}  // namespace topk
