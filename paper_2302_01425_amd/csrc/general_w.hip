// The relaxed operators y_{phi,R}(x, w) for a GENERAL non-increasing weight vector w (Sec. 4;
// soft rank, soft sort and partial ranks through the LP forms of Sec. 3), rows up to 1024 elements.
//
// With w = 1_k one pooled block suffices and the other kernels exploit that.  For a general w the
// partition of pool-adjacent-violators (App. "PAV algorithm") can have any number of blocks.  After
// the same register sort, the lanes of a row build the partition together, in ROUNDS:
//
//   * float64 prefix sums of (s, w [, s^2, s^3]) over the sorted positions live in LDS, so the sums
//     of any block [lo, hi) are two reads and a subtraction;
//   * every lane owns E consecutive positions and keeps the block starts among them as a bit mask;
//     a suffix-minimum / prefix-maximum over the lanes tells each block where its neighbours start;
//   * a round computes the pooled value of every block that changed since the last round, then
//     tests every boundary with the strict test of the PAV loop (gamma_left < gamma_right) and
//     removes ALL violating boundaries at once.
//
// Removing several violating boundaries together is legal: a violating pair of neighbours stays
// violating whatever else is merged first (merging the right block with a block that violates
// against it raises its pooled value, merging the left block with one on its left lowers it), so
// every such pair ends in one block of the sequential algorithm as well, and the partition in
// which no strict violation is left is unique.  Typical rows need a handful of rounds.  A row
// built so that only one boundary violates at a time (a low value followed by a slowly falling
// ramp) needs one round per element: after 32 + n / 4 rounds (p = 2) the wavefront gives up and one
// lane per row walks the usual left-to-right block stack instead.
//
// Pooled values of p = 2 are computed without fused multiply-adds, from sums that are exact
// whenever the float32 inputs span fewer than ~2^19 in magnitude, so exact ties are seen as ties.
// d gamma of every block (Prop. 7) comes from two more prefix sums (weights c_j and c_j tau_j);
// the outputs are then written by all lanes, each position looking up its block's start.
//
// Bound by the latency of one wavefront per row: rows of 1024 elements take 39 KB of LDS, so each
// SIMD has one wavefront, whose vector instructions (4900, 3000 of them the sort) issue for 37 % of
// its time.  4096 x 1024, lambda = 0.1, JVP: 166 us with linear LDS arrays (32-way bank conflicts),
// a first round through LDS and loads of E consecutive elements per lane; 103 us without them.  (With
// one weight vector for all rows and p = 2 the kernel at the end of this file takes these rows.)
#include "common.hpp"
#include "pooling.hpp"
#include "launch.hpp"
#include "wave.hpp"
#include "sort_network.hpp"
#include "general_pav.hpp"

namespace topk {
namespace {

constexpr int kMinRounds = 32;

template <int GL, int E, bool CUBIC>
struct GenCfg {
  static constexpr int NP = GL * E;                 // padded row length
  // entries of a prefix array: 0 .. NP by Swizzled
  static constexpr int NQ = NP + ((NP >> 5) & (E - 1)) + 1;
  static constexpr int RPW = kWave / GL;            // rows per wavefront
  static constexpr int IDXB = ilog2(NP) + 1;
  // float64 arrays per row: prefix S1, prefix W, gamma per block start (+ prefix S2, S3)
  static constexpr int ND = CUBIC ? 5 : 3;
  // bytes per wavefront: the float64 arrays, the starts on the stack of the sequential walk (16
  // bits), and the float arrays ss (sorted values), lw (weights, later y), ltau
  static constexpr int WaveBytes = RPW * (ND * NQ * 8 + (NP + 2) * 2 + 3 * NP * 4);
  // wavefronts per workgroup: rows of 1024 elements take 39 KB (p = 2), one wavefront each, so that
  // four workgroups fit the 160 KB of a compute unit
  static constexpr int WPB = (4 * WaveBytes <= 60 * 1024) ? 4 : ((2 * WaveBytes <= 60 * 1024) ? 2 : 1);
};

// An LDS array indexed by position.  A lane's E consecutive positions start a multiple of E words
// apart from the next lane's, so that the lanes of an instruction would all meet in one or a few of
// the 64 banks (16 positions per lane: a 32-way conflict for float64); the low bits of an index are
// exchanged with the bits that tell those lanes apart.
template <class T, int E>
struct Swizzled {
  T* p;
  __device__ __forceinline__ T& operator[](int i) const {
    return p[i ^ ((i >> (sizeof(T) == 8 ? 5 : 6)) & (E - 1))];
  }
};

// first block start in the lanes after this one / last block start in the lanes before it
template <int GL>
__device__ __forceinline__ int lanes_after_min(int v, int lr, int none) {
#pragma unroll
  for (int off = 1; off < GL; off <<= 1) {
    const int o = __shfl_down(v, off, GL);
    if (lr + off < GL) v = min(v, o);
  }
  const int nx = __shfl_down(v, 1, GL);
  return lr + 1 < GL ? nx : none;
}
template <int GL>
__device__ __forceinline__ int lanes_before_max(int v, int lr, int none) {
#pragma unroll
  for (int off = 1; off < GL; off <<= 1) {
    const int o = __shfl_up(v, off, GL);
    if (lr >= off) v = max(v, o);
  }
  const int pv = __shfl_up(v, 1, GL);
  return lr >= 1 ? pv : none;
}

template <int GL, int E, bool MAG, int PC>
__global__ __launch_bounds__((GenCfg<GL, E, PC == kP43>::WPB * kWave)) void general_rows_kernel(
    const float* __restrict__ x, const float* __restrict__ w_all, int64_t w_stride,
    const float* __restrict__ tangent, float* __restrict__ out, float* __restrict__ jvp,
    int64_t rows, int n, Reg R, int max_rounds) {
  constexpr bool CUBIC = (PC == kP43);
  using C = GenCfg<GL, E, CUBIC>;
  constexpr int NP = C::NP, NQ = C::NQ, RPW = C::RPW, IDXB = C::IDXB;
  static_assert(E <= 16, "the block starts of a lane are kept in a 32-bit mask");
  static_assert(NP < 0xffff, "block ends are kept in 16 bits");
  __shared__ __attribute__((aligned(16))) double ldsd[C::WPB][C::ND][RPW * NQ];
  __shared__ uint16_t lds_hi[C::WPB][RPW * (NP + 2)];
  __shared__ __attribute__((aligned(16))) float ldsf[C::WPB][3][RPW * NP];

  const int lane = threadIdx.x & (kWave - 1);
  const int lr = lane_in_group<GL>();
  const int wv = threadIdx.x / kWave;
  const int rg = lane / GL;                              // row of the wavefront
  int64_t row = (int64_t(blockIdx.x) * C::WPB + wv) * RPW + rg;
  const bool valid = row < rows;
  if (!valid) row = rows - 1;            // keep the lanes alive for the exchanges; no stores
  const int64_t base = row * n;
  const int e0 = lr * E;
  // float64 arrays of the row.  P*: prefix sums over sorted positions, P[i] = sum of j < i.
  using D = Swizzled<double, E>;
  using F = Swizzled<float, E>;
  const D P1{&ldsd[wv][0][rg * NQ]};     // of s; after the rounds: of c_j tau_j (Prop. 7)
  const D PW{&ldsd[wv][1][rg * NQ]};     // of w
  const D G{&ldsd[wv][2][rg * NQ]};      // pooled value by block start; at the very end d gamma
  const D P2{CUBIC ? &ldsd[wv][CUBIC ? 3 : 0][rg * NQ] : nullptr};   // of s^2; after the rounds: of c_j
  const D P3{CUBIC ? &ldsd[wv][CUBIC ? 4 : 0][rg * NQ] : nullptr};   // of s^3
  uint16_t* st_lo = &lds_hi[wv][rg * (NP + 2)];          // stack of the sequential walk
  const F ss{&ldsf[wv][0][rg * NP]};                     // sorted values
  const F lw{&ldsf[wv][1][rg * NP]};                     // weights by sorted position; later y
  const F ltau{&ldsf[wv][2][rg * NP]};                   // tangent in sorted order (times sign)
  const F lt{reinterpret_cast<float*>(G.p)};             // tangent, original order; later dy

  // ---- load, sort ----------------------------------------------------------------------------
  // (load_row: consecutive lanes read consecutive elements, whichever lane holds what; the weights
  // and the tangent reach their positions through LDS)
  float xin[E], win[E];
  load_row<GL, E, false, false>(x, base, lr, n, xin);
  load_row<GL, E, false, false>(w_all, row * w_stride, lr, n, win);
  if (jvp != nullptr) {
    float tin[E];
    load_row<GL, E, false, false>(tangent, base, lr, n, tin);
#pragma unroll
    for (int r = 0; r < E; ++r) lt[r * GL + lr] = tin[r];
  }
#pragma unroll
  for (int r = 0; r < E; ++r) lw[r * GL + lr] = win[r];
  double K[E];
  make_keys_row<GL, E, false, MAG, IDXB>(xin, lr, n, K);
  SortRuns<GL, E, NP>::run(K, lr);
  __builtin_amdgcn_wave_barrier();
  float s32[E];
  uint32_t field[E];
#pragma unroll
  for (int r = 0; r < E; ++r) {
    uint32_t key;
    unpack<IDXB>(K[r], key, field[r]);
    s32[r] = key_to_float(key);
    ss[e0 + r] = s32[r];
    win[r] = lw[e0 + r];
  }
  __builtin_amdgcn_wave_barrier();
  if (jvp != nullptr) {
#pragma unroll
    for (int r = 0; r < E; ++r) {
      float tf = 0.0f;
      if (e0 + r < n) tf = lt[MAG ? (field[r] >> 1) : field[r]];
      if (MAG) {
        if (field[r] & 1u) tf = -tf;
        if (s32[r] == 0.0f) tf = 0.0f;         // sign(0) = 0
      }
      ltau[e0 + r] = tf;
    }
  }

  // ---- prefix sums of the sorted row --------------------------------------------------------------
  {
    double t1 = 0.0, tw = 0.0, t2 = 0.0, t3 = 0.0;
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const bool real = e0 + r < n;
      const double sd = real ? double(s32[r]) : 0.0, wd = real ? double(win[r]) : 0.0;
      t1 += sd;
      tw += wd;
      if (CUBIC) { t2 += sd * sd; t3 += sd * sd * sd; }
    }
    double r1 = group_exclusive_scan_f64<GL>(t1, lr), rw = group_exclusive_scan_f64<GL>(tw, lr);
    double r2 = 0.0, r3 = 0.0;
    if (CUBIC) { r2 = group_exclusive_scan_f64<GL>(t2, lr); r3 = group_exclusive_scan_f64<GL>(t3, lr); }
#pragma unroll
    for (int r = 0; r < E; ++r) {
      P1[e0 + r] = r1;
      PW[e0 + r] = rw;
      if (CUBIC) { P2[e0 + r] = r2; P3[e0 + r] = r3; }
      const bool real = e0 + r < n;
      const double sd = real ? double(s32[r]) : 0.0, wd = real ? double(win[r]) : 0.0;
      r1 += sd;
      rw += wd;
      if (CUBIC) { r2 += sd * sd; r3 += sd * sd * sd; }
    }
    if (lr == GL - 1) {
      P1[NP] = r1;
      PW[NP] = rw;
      if (CUBIC) { P2[NP] = r2; P3[NP] = r3; }
    }
  }
  __builtin_amdgcn_wave_barrier();               // (also: the tangent in G's place has been read)

  auto block_sums = [&](int lo, int hi) -> Blk {
    Blk b;
    b.cnt = double(hi - lo);
    b.S2 = b.S3 = 0.0;
    if (hi - lo == 1) {                      // a singleton: its own value and weight, exactly
      b.S1 = double(ss[lo]);
      b.W = double(lw[lo]);
      if (CUBIC) { b.S2 = b.S1 * b.S1; b.S3 = b.S2 * b.S1; }
    } else {
      b.S1 = P1[hi] - P1[lo];
      b.W = PW[hi] - PW[lo];
      if (CUBIC) { b.S2 = P2[hi] - P2[lo]; b.S3 = P3[hi] - P3[lo]; }
    }
    return b;
  };

  // ---- pool adjacent violators in rounds ------------------------------------------------------------
  uint32_t hm = 0;                           // block starts among my positions (bit r: e0 + r)
#pragma unroll
  for (int r = 0; r < E; ++r)
    if (e0 + r < n) hm |= 1u << r;
  bool gave_up = false;
  int round = 0;
  if (!CUBIC) {
    // the first round, between singletons, in registers
    double gs[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const double sd = double(s32[r]);
      gs[r] = block_gamma<MAG, CUBIC>(Blk{1.0, double(win[r]), sd, 0.0, 0.0}, sd, sd, R);
    }
    double gl = 0.0;
    if (GL > 1) gl = __shfl_up(gs[E - 1], 1, GL);
    uint32_t keep = hm;
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const double left = r > 0 ? gs[r > 0 ? r - 1 : 0] : gl;
      if ((r > 0 || lr > 0) && left < gs[r]) keep &= ~(1u << r);
    }
    hm = keep;                               // (bits of padding are not set in hm)
    round = 1;
    if (round >= max_rounds) gave_up = true;
  }
  // Blocks whose end has moved since the last round have a new pooled value; a boundary between two
  // blocks that are both those of the last round was tested then.
  uint32_t moved = hm;                       // my blocks that are to be computed
  int nxt_seen = -2;
  for (; !gave_up; ++round) {
    const int first = hm ? e0 + __builtin_ctz(hm) : n;
    const int top = hm ? 31 - __builtin_clz(hm) : 0;
    const int nxt = lanes_after_min<GL>(first, lr, n);
    if (hm && nxt != nxt_seen) moved |= 1u << top;
    nxt_seen = nxt;
    // last block start of the lanes before mine, and whether that block is new
    const int before = lanes_before_max<GL>(hm ? 2 * (e0 + top) + int((moved >> top) & 1u) : -1, lr, -1);
    for (uint32_t m = moved; m != 0;) {
      const int r = __builtin_ctz(m);
      m &= m - 1;
      const uint32_t above = hm & ~((2u << r) - 1u);
      const int lo = e0 + r, hi = above ? e0 + __builtin_ctz(above) : nxt;
      G[lo] = block_gamma<MAG, CUBIC>(block_sums(lo, hi), double(ss[lo]), double(ss[hi - 1]), R);
    }
    __builtin_amdgcn_wave_barrier();
    // every boundary whose two blocks violate goes
    uint32_t keep = hm;
    for (uint32_t m = hm; m != 0;) {
      const int r = __builtin_ctz(m);
      m &= m - 1;
      const uint32_t below = hm & ((1u << r) - 1u);
      const int pr = below ? 31 - __builtin_clz(below) : 0;
      const int p = below ? e0 + pr : (before >= 0 ? before >> 1 : -1);
      if (p < 0) continue;                   // the first block of the row
      const uint32_t pnew = below ? (moved >> pr) & 1u : uint32_t(before) & 1u;
      if ((pnew | ((moved >> r) & 1u)) == 0) continue;
      const int lo = e0 + r;
      bool viol;
      if (!CUBIC) viol = G[p] < G[lo];
      else {
        const int hi = m ? e0 + __builtin_ctz(m) : nxt;
        viol = blocks_violate<MAG, CUBIC>(block_sums(p, lo), G[p], block_sums(lo, hi), G[lo], R);
      }
      if (viol) keep &= ~(1u << r);
    }
    const bool changed = keep != hm;
    // blocks that stay and whose next start (in this lane) goes
    const uint32_t gone = hm & ~keep;
    moved = 0;
    for (uint32_t m = gone; m != 0;) {
      const int r = __builtin_ctz(m);
      m &= m - 1;
      const uint32_t below = keep & ((1u << r) - 1u);
      if (below) moved |= 1u << (31 - __builtin_clz(below));
    }
    hm = keep;
    if (!__any(changed)) break;
    if (round + 1 >= max_rounds) { gave_up = true; break; }
    __builtin_amdgcn_wave_barrier();
  }
  __builtin_amdgcn_wave_barrier();

  const D DG = G;                            // d gamma by block start
  float yv[E];
  double tt[E];                              // (s - gamma) / lambda
  if (!gave_up) {
    const int last = hm ? e0 + 31 - __builtin_clz(hm) : -1;
    const int prv = lanes_before_max<GL>(last, lr, -1);
    if (CUBIC) {
      // ---- the roots once more, from sums of the blocks' own spread.  A block's sums so far are
      // differences of prefix sums over the whole row: their rounding is that of the row's values
      // cubed, while the cubic of a block whose values lie within a small lambda of each other
      // needs that of the spread cubed.  With the partition final, every position is taken
      // relative to the first value c of its own block: the prefix sums of d = s - c, d^2, d^3
      // stay as small as the blocks are narrow (a block's sums involve its own positions only),
      // and the safeguarded Newton solve of the rounds, on sum (g - d_i)^3 + lambda^3 W [c + g] = 0
      // with the same bracket, gives gamma = c + g to the rounding of the spread -----------------
      double dd[E];
      double t1 = 0.0, t2 = 0.0, t3 = 0.0;
#pragma unroll
      for (int r = 0; r < E; ++r) {
        const uint32_t upto = hm & ((2u << r) - 1u);
        int b = upto ? e0 + 31 - __builtin_clz(upto) : prv;
        if (b < 0) b = 0;
        dd[r] = (e0 + r < n) ? double(s32[r]) - double(ss[b]) : 0.0;
        t1 += dd[r];
        t2 += dd[r] * dd[r];
        t3 += dd[r] * dd[r] * dd[r];
      }
      double r1 = group_exclusive_scan_f64<GL>(t1, lr), r2 = group_exclusive_scan_f64<GL>(t2, lr);
      double r3 = group_exclusive_scan_f64<GL>(t3, lr);
      __builtin_amdgcn_wave_barrier();           // the prefix sums of the rounds have been read
#pragma unroll
      for (int r = 0; r < E; ++r) {
        P1[e0 + r] = r1;
        P2[e0 + r] = r2;
        P3[e0 + r] = r3;
        r1 += dd[r];
        r2 += dd[r] * dd[r];
        r3 += dd[r] * dd[r] * dd[r];
      }
      if (lr == GL - 1) {
        P1[NP] = r1;
        P2[NP] = r2;
        P3[NP] = r3;
      }
      __builtin_amdgcn_wave_barrier();
      const int first = hm ? e0 + __builtin_ctz(hm) : n;
      const int nxt = lanes_after_min<GL>(first, lr, n);
      for (uint32_t m = hm; m != 0;) {
        const int r = __builtin_ctz(m);
        m &= m - 1;
        const int lo = e0 + r, hi = m ? e0 + __builtin_ctz(m) : nxt;
        if (hi - lo == 1) continue;              // (singletons have closed forms)
        const double cnt = double(hi - lo), c = double(ss[lo]);
        const double S1 = P1[hi] - P1[lo], S2 = P2[hi] - P2[lo], S3 = P3[hi] - P3[lo];
        const double W = PW[hi] - PW[lo];
        // the bracket of the first solve, relative to c: [smin - lambda cbrt(W), smax] (mask), [0, smax]
        const double dmin = double(ss[hi - 1]) - c;
        const double g = MAG ? block_root<true>(cnt, W, S1, S2, S3, R, -c, 0.0, c)
                             : block_root<false>(cnt, W, S1, S2, S3, R,
                                                 dmin - R.lambda * cbrt(W) - 1e-300, 0.0);
        G[lo] = c + g;
      }
      __builtin_amdgcn_wave_barrier();
    }
    // ---- y; then Prop. 7: d gamma of every block from prefix sums of c_j tau_j and c_j --------------
    double cq[E], cc[E];
    double tq = 0.0, tc = 0.0;
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const uint32_t upto = hm & ((2u << r) - 1u);
      int b = upto ? e0 + 31 - __builtin_clz(upto) : prv;
      if (b < 0) b = 0;
      const double g = G[b];
      tt[r] = (double(s32[r]) - g) * R.inv_lambda;
      double c = 1.0;
      if (CUBIC) {
        const double d = g - double(s32[r]);
        c = MAG ? 3.0 * d * d : d * d;
      }
      const bool real = e0 + r < n;
      cc[r] = real ? c : 0.0;
      cq[r] = (real && jvp != nullptr) ? c * double(ltau[e0 + r]) : 0.0;
      tq += cq[r];
      tc += cc[r];
    }
    if (jvp != nullptr) {
      double rq = group_exclusive_scan_f64<GL>(tq, lr);
      double rc = CUBIC ? group_exclusive_scan_f64<GL>(tc, lr) : 0.0;
#pragma unroll
      for (int r = 0; r < E; ++r) {
        P1[e0 + r] = rq;
        if (CUBIC) P2[e0 + r] = rc;
        rq += cq[r];
        rc += cc[r];
      }
      if (lr == GL - 1) {
        P1[NP] = rq;
        if (CUBIC) P2[NP] = rc;
      }
      __builtin_amdgcn_wave_barrier();
      const int first = hm ? e0 + __builtin_ctz(hm) : n;
      const int nxt = lanes_after_min<GL>(first, lr, n);
      for (uint32_t m = hm; m != 0;) {
        const int r = __builtin_ctz(m);
        m &= m - 1;
        const int lo = e0 + r, hi = m ? e0 + __builtin_ctz(m) : nxt;
        double dg;
        if (hi - lo == 1) {
          const double tau = double(ltau[lo]), W = double(lw[lo]);
          if (!MAG) dg = tau;
          else if (!CUBIC) dg = tau / (1.0 + R.lambda * W);
          else if (W == 0.0) dg = tau;
          else {
            const double d = G[lo] - double(ss[lo]);
            dg = 3.0 * d * d * tau / (3.0 * d * d + R.lam3 * W);
          }
        } else {
          const double num = P1[hi] - P1[lo];
          double den = CUBIC ? P2[hi] - P2[lo] : double(hi - lo);
          if (MAG) den += (CUBIC ? R.lam3 : R.lambda) * (PW[hi] - PW[lo]);
          dg = num / den;
        }
        DG[lo] = dg;                         // G[lo] is read by this lane only, above
      }
    }
  } else {
    // ---- too many rounds: the left-to-right block stack, one lane per row ---------------------------
    // (stack columns in the arrays of the rounds; the block on top of the stack is kept in registers)
    for (int i = lr; i < NP; i += GL) st_lo[i] = 0;        // no mark but those of the walk
    __builtin_amdgcn_wave_barrier();
    if (lr == 0)
      stack_walk<MAG, CUBIC, uint16_t>(n, ss, lw, ltau, jvp != nullptr, P1, PW, G, P2, P3, st_lo,
                                       uint16_t(0xffff), P1, R);
    __builtin_amdgcn_wave_barrier();
    hm = 0;
#pragma unroll
    for (int r = 0; r < E; ++r)
      if (e0 + r < n && st_lo[e0 + r] == 0xffff) hm |= 1u << r;
    const int last = hm ? e0 + 31 - __builtin_clz(hm) : -1;
    const int prv = lanes_before_max<GL>(last, lr, -1);
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const uint32_t upto = hm & ((2u << r) - 1u);
      int b = upto ? e0 + 31 - __builtin_clz(upto) : prv;
      if (b < 0) b = 0;
      tt[r] = (double(s32[r]) - G[b]) * R.inv_lambda;
    }
  }
  __builtin_amdgcn_wave_barrier();

  // ---- outputs: y = sign o grad r*(s - v), dy = sign o hess r*(s - v) (tau - d gamma) ------------
  {
    const int last = hm ? e0 + 31 - __builtin_clz(hm) : -1;
    const int prv = lanes_before_max<GL>(last, lr, -1);
    float dv[E];
    uint32_t orig[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const uint32_t upto = hm & ((2u << r) - 1u);
      int b = upto ? e0 + 31 - __builtin_clz(upto) : prv;
      if (b < 0) b = 0;                                    // padding of an empty tail
      const bool neg = MAG && (field[r] & 1u);
      orig[r] = MAG ? (field[r] >> 1) : field[r];
      float y = float(CUBIC ? tt[r] * tt[r] * tt[r] : tt[r]);
      if (MAG) y = (y == 0.0f || s32[r] == 0.0f) ? 0.0f : (neg ? -y : y);
      yv[r] = y;
      dv[r] = 0.0f;
      if (jvp != nullptr) {
        const double h = CUBIC ? 3.0 * tt[r] * tt[r] * R.inv_lambda : R.inv_lambda;
        float dy = float(h * (double(ltau[e0 + r]) - (gave_up ? P1[b] : DG[b])));
        if (MAG) dy = (dy == 0.0f || s32[r] == 0.0f) ? 0.0f : (neg ? -dy : dy);
        dv[r] = dy;
      }
    }
    __builtin_amdgcn_wave_barrier();             // lw and G's place are free: everything was read
#pragma unroll
    for (int r = 0; r < E; ++r) {
      if (e0 + r >= n) continue;
      if (out != nullptr) lw[orig[r]] = yv[r];
      if (jvp != nullptr) lt[orig[r]] = dv[r];
    }
  }
  __builtin_amdgcn_wave_barrier();
  if (!valid) return;
  if (out != nullptr) {
    float ov[E];
#pragma unroll
    for (int r = 0; r < E; ++r) ov[r] = lw[r * GL + lr];
    store_row<GL, E, false, false>(out, base, lr, n, ov);
  }
  if (jvp != nullptr) {
    float jv[E];
#pragma unroll
    for (int r = 0; r < E; ++r) jv[r] = lt[r * GL + lr];
    store_row<GL, E, false, false>(jvp, base, lr, n, jv);
  }
}

// ---- sort on 32-bit words ----------------------------------------------------------------------------
// first block start in the lanes after this one / last block start in the lanes before it, for rows that take a whole
// wavefront: moves inside the rows of 16 lanes instead of twelve trips through the LDS crossbar
__device__ __forceinline__ int wave_after_min(int v, int none) {
#define TOPK_STEP(CTRL) v = min(v, __builtin_amdgcn_update_dpp(v, v, CTRL, 0xF, 0xF, false))
  TOPK_STEP(0x101);
  TOPK_STEP(0x102);
  TOPK_STEP(0x104);
  TOPK_STEP(0x108);
#undef TOPK_STEP
  const int m3 = __builtin_amdgcn_readlane(v, 48), m2 = min(m3, __builtin_amdgcn_readlane(v, 32));
  const int m1 = min(m2, __builtin_amdgcn_readlane(v, 16));
  const int lane = threadIdx.x & (kWave - 1);
  const int later = lane < 16 ? m1 : (lane < 32 ? m2 : (lane < 48 ? m3 : none));
  return min(__builtin_amdgcn_update_dpp(none, v, 0x101, 0xF, 0xF, false), min(later, none));
}
__device__ __forceinline__ int wave_before_max(int v, int none) {
#define TOPK_STEP(CTRL) v = max(v, __builtin_amdgcn_update_dpp(v, v, CTRL, 0xF, 0xF, false))
  TOPK_STEP(0x111);
  TOPK_STEP(0x112);
  TOPK_STEP(0x114);
  TOPK_STEP(0x118);
#undef TOPK_STEP
  const int m0 = __builtin_amdgcn_readlane(v, 15), m1 = max(m0, __builtin_amdgcn_readlane(v, 31));
  const int m2 = max(m1, __builtin_amdgcn_readlane(v, 47));
  const int lane = threadIdx.x & (kWave - 1);
  const int earlier = lane < 16 ? none : (lane < 32 ? m0 : (lane < 48 ? m1 : m2));
  return max(__builtin_amdgcn_update_dpp(none, v, 0x111, 0xF, 0xF, false), max(earlier, none));
}
template <int GL>
__device__ __forceinline__ int row_after_min(int v, int lr, int none) {
  if constexpr (GL == kWave) return wave_after_min(v, none);
  else return lanes_after_min<GL>(v, lr, none);
}
template <int GL>
__device__ __forceinline__ int row_before_max(int v, int lr, int none) {
  if constexpr (GL == kWave) return wave_before_max(v, none);
  else return lanes_before_max<GL>(v, lr, none);
}
template <int GL>
__device__ __forceinline__ double row_exclusive_scan(double v, int lr) {
  if constexpr (GL == kWave) {
    v += row_shr_f64<1>(v);
    v += row_shr_f64<2>(v);
    v += row_shr_f64<4>(v);
    v += row_shr_f64<8>(v);
    const double t0 = uniform_f64(v, 15), t1 = t0 + uniform_f64(v, 31), t2 = t1 + uniform_f64(v, 47);
    const int lane = threadIdx.x & (kWave - 1);
    const double before = lane < 16 ? 0.0 : (lane < 32 ? t0 : (lane < 48 ? t1 : t2));
    return row_shr_f64<1>(v) + before;
  } else {
    return group_exclusive_scan_f64<GL>(v, lr);
  }
}
// the number nearest to zero among those of the first 16 lanes
__device__ __forceinline__ float nearest_zero16(float v) {
  const uint32_t b = __float_as_uint(v);
  uint32_t m = (b << 1) | (b >> 31);
#define TOPK_STEP(CTRL) m = min(m, uint32_t(__builtin_amdgcn_update_dpp(int(m), int(m), CTRL, 0xF, 0xF, false)))
  TOPK_STEP(0x111);
  TOPK_STEP(0x112);
  TOPK_STEP(0x114);
  TOPK_STEP(0x118);
#undef TOPK_STEP
  const uint32_t r = uint32_t(__builtin_amdgcn_readlane(int(m), 15));
  return __uint_as_float((r >> 1) | (r << 31));
}
// a lane's own value from the lane after it / before it (the last / first lane: its own)
template <int CTRL>
__device__ __forceinline__ double neighbour_f64(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = int(b), hi = int(b >> 32);
  const uint32_t l = uint32_t(__builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xF, 0xF, false));
  const uint32_t h = uint32_t(__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xF, 0xF, false));
  return __longlong_as_double((long long)(uint64_t(h) << 32 | l));
}
__device__ __forceinline__ double lane_after_f64(double v) { return neighbour_f64<0x130>(v); }
__device__ __forceinline__ double lane_before_f64(double v) { return neighbour_f64<0x138>(v); }
// Among the lanes and four others each (in their rows of 16): do two pairs of different values agree in all but the low
// bits of their words?
template <int ROR>
__device__ __forceinline__ unsigned long long pairs_alike(uint32_t word, float v, uint32_t low_bits) {
  // (moves first: every lane takes part in them)
  const uint32_t w2 = uint32_t(__builtin_amdgcn_update_dpp(0, int(word), 0x120 + ROR, 0xF, 0xF, false));
  const int v2 = __builtin_amdgcn_update_dpp(0, int(__float_as_uint(v)), 0x120 + ROR, 0xF, 0xF, false);
  const bool near = (word ^ w2) <= low_bits, differ = v != __uint_as_float(uint32_t(v2));
  return __ballot(near & differ);
}
__device__ __forceinline__ bool words_collide(uint32_t word, float v, uint32_t low_bits) {
  const unsigned long long a = pairs_alike<1>(word, v, low_bits), b = pairs_alike<2>(word, v, low_bits);
  const unsigned long long c = pairs_alike<3>(word, v, low_bits), d = pairs_alike<5>(word, v, low_bits);
  return __popcll(a) + __popcll(b) + __popcll(c) + __popcll(d) >= 2;
}
// Sorted (key, field) words of a row (as SortRuns on make_keys_row makes them) by way of 32-bit words: the leading
// 32 - log2(NP) bits of the key of a value less one of the row's, and the element's number.  The difference never falls as
// the value rises, so that only values with the same leading bits may come in the wrong order (some ten pairs in a row
// of 1024 normal values), which a few rounds of exchanges between neighbours set right.  Of the row's first 16 the value
// nearest to zero is taken off: a few large ones among many small ones (scores masked out by -1e9) leave the small ones
// apart then.  Rows with a cluster of values that agree to 13 bits, far from that one, are not settled so and are sorted by
// complete keys, without the attempt where two of 256 pairs of the row's first 64 elements agree (normal values: one
// row in 10^5).
// xs: the row in LDS by element.  JVP with rank weights, lambda = 0.1, us a call, sorted by complete keys (with scans
// through the LDS crossbar) / so, without a look at the pairs and with the median of three values taken off / so:
//                                                        4096 x 1024          6697 x 425           69 x 538
//   normal values                                     54.8 / 44.4 / 44.5   42.8 / 34.6 / 35.2   22.7 / 17.9 / 17.9
//   half at 0 +- 1e-3, half at 100 +- 1e-3            42.7 / 57.2 / 41.8   31.1 / 39.1 / 30.2   16.5 / 21.7 / 16.0
//   half normal, half at 100 +- 0.01                  55.6 / 65.3 / 51.5   43.9 / 48.0 / 44.4   23.1 / 26.2 / 20.7
//   half normal, half at -1e9                         55.9 / 66.2 / 45.1   43.5 / 48.0 / 36.1   23.1 / 26.6 / 18.4
//   a tenth at 100 +- 1e-3 (half of such rows seen)   54.6 / 65.9 / 65.6   42.8 / 49.1 / 49.3   22.5 / 25.8 / 25.8
// Rows of up to 256 elements, two to a wavefront, gain 2 % at most and lose up to 27 %: complete keys.
template <int E, bool MAG, int IDXB>
__device__ __forceinline__ void sort_row(const float (&xin)[E], const float* xs, int n, double (&K)[E]) {
  constexpr int GL = kWave, NP = GL * E;
  const int lr = threadIdx.x & (kWave - 1);
  const float sample = xin[0], of_row = MAG ? fabsf(sample) : sample;
  float mid = nearest_zero16(of_row);
  mid = fabsf(mid) < 1e37f ? mid : 0.0f;
  auto word = [&](float v) { return desc_key((MAG ? fabsf(v) : v) - mid); };
  if (!words_collide(word(of_row), of_row, uint32_t(NP - 1))) {
    uint32_t W[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const int e = r * GL + lr;
      W[r] = ((e < n ? word(xin[r]) : kSentinelKey) & ~uint32_t(NP - 1)) | uint32_t(e);
    }
    SortRuns<GL, E, NP>::run(W, lr);
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const uint32_t e = W[r] & uint32_t(NP - 1);
      uint32_t key = kSentinelKey, field = (1u << IDXB) - 1u;
      if (int(e) < n) {
        const float v = xs[e];
        key = desc_key(MAG ? fabsf(v) : v);
        field = MAG ? ((e << 1) | (__float_as_uint(v) >> 31)) : e;
      }
      K[r] = pack<IDXB>(key, field);
    }
    constexpr int kRepairs = 5;
#pragma unroll 1
    for (int round = 0;; ++round) {
      const double next = lane_after_f64(K[0]);
      bool wrong = lr != GL - 1 && K[E - 1] > next;      // (the last lane has none)
#pragma unroll
      for (int r = 1; r < E; ++r) wrong |= K[r - 1] > K[r];
      if (!__any(wrong)) return;
      if (round == kRepairs) break;
#pragma unroll
      for (int odd = 0; odd < 2; ++odd) {
#pragma unroll
        for (int r = 1 - odd; r + 1 < E; r += 2) {
          const double lo = min_f64(K[r], K[r + 1]), hi = max_f64(K[r], K[r + 1]);
          K[r] = lo;
          K[r + 1] = hi;
        }
        if (odd == 0) {                            // with the first and the last of the neighbouring lanes
          const double after = lane_after_f64(K[0]), before = lane_before_f64(K[E - 1]);
          if (lr != GL - 1) K[E - 1] = min_f64(K[E - 1], after);
          if (lr != 0) K[0] = max_f64(K[0], before);
        }
      }
    }
  }
  make_keys_row<GL, E, false, MAG, IDXB>(xin, lr, n, K);
  SortRuns<GL, E, NP>::run(K, lr);
}

// ---- p = 2 with one weight vector for all rows ------------------------------------------------------
// The same rounds in 16 bytes of LDS per element instead of 38, so that twice (rows above 512
// elements) to four times as many wavefronts hide each other's latency.  The prefix sums of w are those
// of every row: one copy per workgroup.  A block of one element gets its pooled value from the
// registers in the first round and is never computed again, so neither the sorted values nor the
// weights are looked up; the tangent stays in registers; inputs and outputs change their order through
// the arrays of the rounds before and after these.  There is no hand-over to the sequential walk: a
// round costs one walk step per moved block and two lane scans, and a row of n elements settles in n - 1
// rounds at most.
// JVP, us, against the kernel above: 4096 x 1024 (lambda = 0.1) 103 -> 55 (44 with the sort on 32-bit words),
// 6697 x 425 206 -> 94, 2061 x 186 40 -> 26, 69 x 538 (lambda = 0.0065) 113 -> 58; 1024 rows of 1024 that lose one boundary per
// round 1740 (walk after 288 rounds, at the time) -> 1060.
template <int GL, int E>
struct LeanCfg {
  static constexpr int NP = GL * E, RPW = kWave / GL;
  static constexpr int NQ = NP + ((NP >> 5) & (E - 1)) + 1;
  static constexpr int IDXB = ilog2(NP) + 1;
  static constexpr int WPB = 4;
};

template <int GL, int E, bool MAG>
__global__ __launch_bounds__((LeanCfg<GL, E>::WPB * kWave)) void general_shared_kernel(
    const float* __restrict__ x, const float* __restrict__ w, const float* __restrict__ tangent,
    float* __restrict__ out, float* __restrict__ jvp, int64_t rows, int n, Reg R) {
  using C = LeanCfg<GL, E>;
  using D = Swizzled<double, E>;
  using F = Swizzled<float, E>;
  constexpr int NP = C::NP, NQ = C::NQ, RPW = C::RPW, IDXB = C::IDXB;
  static_assert(E <= 16, "the block starts of a lane are kept in a 32-bit mask");
  __shared__ __attribute__((aligned(16))) double lds_w[NQ];
  __shared__ __attribute__((aligned(16))) double ldsd[C::WPB][2][RPW * NQ];

  const int lane = threadIdx.x & (kWave - 1);
  const int lr = lane_in_group<GL>();
  const int wv = threadIdx.x / kWave;
  const int rg = lane / GL;
  int64_t row = (int64_t(blockIdx.x) * C::WPB + wv) * RPW + rg;
  const bool valid = row < rows;
  if (!valid) row = rows - 1;            // keep the lanes alive for the exchanges; no stores
  const int64_t base = row * n;
  const int e0 = lr * E;
  const D PW{lds_w};                                     // prefix sums of w
  const D P1{&ldsd[wv][0][rg * NQ]};                     // of s; after the rounds: of the tangent
  const D G{&ldsd[wv][1][rg * NQ]};                      // pooled value, then d gamma, by block start
  const F in_w{reinterpret_cast<float*>(P1.p)};          // before the prefix sums: weights
  const F in_t{reinterpret_cast<float*>(G.p)};           // before the rounds: tangent, original order
  const F out_y{reinterpret_cast<float*>(P1.p)};         // at the end: the outputs, original order
  const F out_d{reinterpret_cast<float*>(G.p)};

  // ---- load, sort ----------------------------------------------------------------------------
  float xin[E], win[E], tau[E];
  load_row<GL, E, false, false>(x, base, lr, n, xin);
  load_row<GL, E, false, false>(w, 0, lr, n, win);
  if (jvp != nullptr) {
    load_row<GL, E, false, false>(tangent, base, lr, n, tau);
#pragma unroll
    for (int r = 0; r < E; ++r) in_t[r * GL + lr] = tau[r];
  }
#pragma unroll
  for (int r = 0; r < E; ++r) in_w[r * GL + lr] = win[r];
  double K[E];
  if constexpr (GL == kWave) {               // (see there)
    float* xs = reinterpret_cast<float*>(P1.p) + NP;       // (after the weights)
#pragma unroll
    for (int r = 0; r < E; ++r) xs[r * GL + lr] = xin[r];
    __builtin_amdgcn_wave_barrier();
    sort_row<E, MAG, IDXB>(xin, xs, n, K);
  } else {
    make_keys_row<GL, E, false, MAG, IDXB>(xin, lr, n, K);
    SortRuns<GL, E, NP>::run(K, lr);
  }
  __builtin_amdgcn_wave_barrier();
  float s32[E];
  uint32_t field[E];
#pragma unroll
  for (int r = 0; r < E; ++r) {
    uint32_t key;
    unpack<IDXB>(K[r], key, field[r]);
    s32[r] = key_to_float(key);
    win[r] = in_w[e0 + r];
    tau[r] = 0.0f;
    if (jvp != nullptr && e0 + r < n) {
      float tf = in_t[MAG ? (field[r] >> 1) : field[r]];
      if (MAG) {
        if (field[r] & 1u) tf = -tf;
        if (s32[r] == 0.0f) tf = 0.0f;         // sign(0) = 0
      }
      tau[r] = tf;
    }
  }
  __builtin_amdgcn_wave_barrier();

  // ---- prefix sums; pooled values of the singletons and the first round between them ---------------
  uint32_t hm = 0;                           // block starts among my positions (bit r: e0 + r)
  {
    double t1 = 0.0, tw = 0.0;
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const bool real = e0 + r < n;
      t1 += real ? double(s32[r]) : 0.0;
      tw += double(win[r]);                  // (0 beyond the row)
    }
    double r1 = row_exclusive_scan<GL>(t1, lr), rw = row_exclusive_scan<GL>(tw, lr);
    const bool weights = wv == 0 && rg == 0;
    double gs[E];
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const bool real = e0 + r < n;
      const double sd = real ? double(s32[r]) : 0.0;
      P1[e0 + r] = r1;
      if (weights) PW[e0 + r] = rw;
      r1 += sd;
      rw += double(win[r]);
      gs[r] = block_gamma<MAG, false>(Blk{1.0, double(win[r]), sd, 0.0, 0.0}, sd, sd, R);
      G[e0 + r] = gs[r];
      if (real) hm |= 1u << r;
    }
    if (lr == GL - 1) {
      P1[NP] = r1;
      if (weights) PW[NP] = rw;
    }
    double gl = 0.0;
    if (GL > 1) gl = __shfl_up(gs[E - 1], 1, GL);
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const double left = r > 0 ? gs[r > 0 ? r - 1 : 0] : gl;
      if ((r > 0 || lr > 0) && left < gs[r]) hm &= ~(1u << r);
    }
  }
  __syncthreads();                           // PW (written by the first wavefront)

  // ---- pool adjacent violators in rounds (see general_rows_kernel) ---------------------------------
  int nxt = 0, nxt_seen = 0;
  uint32_t moved = 0;                        // my blocks that are to be computed
  bool first_time = true;
  for (;;) {
    const int first = hm ? e0 + __builtin_ctz(hm) : n;
    const int top = hm ? 31 - __builtin_clz(hm) : 0;
    nxt = row_after_min<GL>(first, lr, n);
    if (first_time) {
      // everything longer than one element
      moved = hm & ~(hm >> 1);
      if (nxt == e0 + top + 1) moved &= ~(1u << top);
      first_time = false;
    } else if (hm && nxt != nxt_seen) {
      moved |= 1u << top;
    }
    nxt_seen = nxt;
    const int before = row_before_max<GL>(hm ? 2 * (e0 + top) + int((moved >> top) & 1u) : -1, lr, -1);
    for (uint32_t m = moved; m != 0;) {
      const int r = __builtin_ctz(m);
      m &= m - 1;
      const uint32_t above = hm & ~((2u << r) - 1u);
      const int lo = e0 + r, hi = above ? e0 + __builtin_ctz(above) : nxt;
      G[lo] = block_gamma<MAG, false>(Blk{double(hi - lo), PW[hi] - PW[lo], P1[hi] - P1[lo], 0.0, 0.0}, 0.0,
                                      0.0, R);
    }
    __builtin_amdgcn_wave_barrier();
    // boundaries next to a moved block
    uint32_t keep = hm;
    uint32_t test = moved;
    {
      const uint32_t low = hm & (0u - hm);                       // my first block: its left neighbour
      if (before >= 0 && (before & 1)) test |= low;
      for (uint32_t m = moved; m != 0;) {                        // right neighbours of moved blocks
        const int r = __builtin_ctz(m);
        m &= m - 1;
        const uint32_t above = hm & ~((2u << r) - 1u);
        test |= above & (0u - above);
      }
    }
    for (uint32_t m = test; m != 0;) {
      const int r = __builtin_ctz(m);
      m &= m - 1;
      const uint32_t below = hm & ((1u << r) - 1u);
      const int p = below ? e0 + 31 - __builtin_clz(below) : (before >= 0 ? before >> 1 : -1);
      if (p >= 0 && G[p] < G[e0 + r]) keep &= ~(1u << r);
    }
    // blocks that stay and whose next start (in this lane) goes
    moved = 0;
    for (uint32_t m = hm & ~keep; m != 0;) {
      const int r = __builtin_ctz(m);
      m &= m - 1;
      const uint32_t below = keep & ((1u << r) - 1u);
      if (below) moved |= 1u << (31 - __builtin_clz(below));
    }
    const bool changed = keep != hm;
    hm = keep;
    if (!__any(changed)) break;
    __builtin_amdgcn_wave_barrier();
  }

  // ---- y; d gamma of every block (Prop. 7) from prefix sums of the tangent ----------------------------
  const int prv = row_before_max<GL>(hm ? e0 + 31 - __builtin_clz(hm) : -1, lr, -1);
  auto start_of = [&](int r) {
    const uint32_t upto = hm & ((2u << r) - 1u);
    const int b = upto ? e0 + 31 - __builtin_clz(upto) : prv;
    return b < 0 ? 0 : b;                                  // (padding of an empty tail)
  };
  float yv[E], dv[E];
#pragma unroll
  for (int r = 0; r < E; ++r) {
    const bool neg = MAG && (field[r] & 1u);
    float y = float((double(s32[r]) - G[start_of(r)]) * R.inv_lambda);
    if (MAG) y = (y == 0.0f || s32[r] == 0.0f) ? 0.0f : (neg ? -y : y);
    yv[r] = y;
    dv[r] = 0.0f;
  }
  if (jvp != nullptr) {
    double tq = 0.0;
#pragma unroll
    for (int r = 0; r < E; ++r) tq += double(tau[r]);
    double rq = row_exclusive_scan<GL>(tq, lr);
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < E; ++r) {
      P1[e0 + r] = rq;
      rq += double(tau[r]);
    }
    if (lr == GL - 1) P1[NP] = rq;
    __builtin_amdgcn_wave_barrier();
    uint32_t longer = hm & ~(hm >> 1);
    if (hm && nxt == e0 + 31 - __builtin_clz(hm) + 1) longer &= ~(1u << (31 - __builtin_clz(hm)));
#pragma unroll
    for (int r = 0; r < E; ++r) {
      // one element: from its own tangent and weight
      if (((hm & ~longer) >> r) & 1u) {
        const double t = double(tau[r]);
        G[e0 + r] = MAG ? t / (1.0 + R.lambda * double(win[r])) : t;
      }
    }
    for (uint32_t m = longer; m != 0;) {
      const int r = __builtin_ctz(m);
      m &= m - 1;
      const uint32_t above = hm & ~((2u << r) - 1u);
      const int lo = e0 + r, hi = above ? e0 + __builtin_ctz(above) : nxt;
      double den = double(hi - lo);
      if (MAG) den += R.lambda * (PW[hi] - PW[lo]);
      G[lo] = (P1[hi] - P1[lo]) / den;
    }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < E; ++r) {
      const bool neg = MAG && (field[r] & 1u);
      float dy = float(R.inv_lambda * (double(tau[r]) - G[start_of(r)]));
      if (MAG) dy = (dy == 0.0f || s32[r] == 0.0f) ? 0.0f : (neg ? -dy : dy);
      dv[r] = dy;
    }
  }
  __builtin_amdgcn_wave_barrier();           // everything has been read

  // ---- outputs in the original order ---------------------------------------------------------------
#pragma unroll
  for (int r = 0; r < E; ++r) {
    if (e0 + r >= n) continue;
    const uint32_t orig = MAG ? (field[r] >> 1) : field[r];
    if (out != nullptr) out_y[orig] = yv[r];
    if (jvp != nullptr) out_d[orig] = dv[r];
  }
  __builtin_amdgcn_wave_barrier();
  if (!valid) return;
  if (out != nullptr) {
#pragma unroll
    for (int r = 0; r < E; ++r) yv[r] = out_y[r * GL + lr];
    store_row<GL, E, false, false>(out, base, lr, n, yv);
  }
  if (jvp != nullptr) {
#pragma unroll
    for (int r = 0; r < E; ++r) dv[r] = out_d[r * GL + lr];
    store_row<GL, E, false, false>(jvp, base, lr, n, dv);
  }
}

template <int GL, int E>
int launch_general_shared(bool mag, const float* x, const float* w, const float* t, float* out, float* jvp,
                          int64_t rows, int n, const Reg& R, hipStream_t st) {
  using C = LeanCfg<GL, E>;
  const int64_t blocks = (rows + C::RPW * C::WPB - 1) / (C::RPW * C::WPB);
  if (blocks > 0x7fffffffLL) return -1;
  if (mag)
    hipLaunchKernelGGL((general_shared_kernel<GL, E, true>), dim3((unsigned)blocks), dim3(C::WPB * kWave), 0,
                       st, x, w, t, out, jvp, rows, n, R);
  else
    hipLaunchKernelGGL((general_shared_kernel<GL, E, false>), dim3((unsigned)blocks), dim3(C::WPB * kWave), 0,
                       st, x, w, t, out, jvp, rows, n, R);
  return 0;
}

template <int GL, int E>
int launch_general_shape(bool mag, int pc, const float* x, const float* w, int64_t w_stride,
                         const float* t, float* out, float* jvp, int64_t rows, int n, const Reg& R,
                         hipStream_t st, int max_rounds) {
#define TOPK_GENERAL_CALL(MAGV, PCV)                                                            \
  do {                                                                                          \
    using C = GenCfg<GL, E, PCV == kP43>;                                                       \
    const int64_t waves = (rows + C::RPW - 1) / C::RPW;                                         \
    const int64_t blocks = (waves + C::WPB - 1) / C::WPB;                                       \
    if (blocks > 0x7fffffffLL) return -1;                                                       \
    hipLaunchKernelGGL((general_rows_kernel<GL, E, MAGV, PCV>), dim3((unsigned)blocks),          \
                       dim3(C::WPB * kWave), 0, st, x, w, w_stride, t, out, jvp, rows, n, R,   \
                       max_rounds);                                                             \
    return 0;                                                                                   \
  } while (0)
  if (!mag && pc == kP2) TOPK_GENERAL_CALL(false, kP2);
  if (!mag && pc == kP43) TOPK_GENERAL_CALL(false, kP43);
  if (mag && pc == kP2) TOPK_GENERAL_CALL(true, kP2);
  if (mag && pc == kP43) TOPK_GENERAL_CALL(true, kP43);
#undef TOPK_GENERAL_CALL
  return -1;
}

}  // namespace

int launch_general_rows(bool mag, int pc, const float* x, const float* w, int64_t w_stride,
                        const float* tangent, float* out, float* jvp, int64_t rows, int n,
                        const Reg& R, hipStream_t st) {
  int np = 2;
  while (np < n) np <<= 1;
  // Rounds before the hand-over to the sequential walk.  A round costs about as much as four
  // steps of the walk for p = 2; for p = 4/3 every step of the walk solves a cubic, and the rounds
  // (n - 1 of them at most: each removes a boundary) always win.
  const int forced = routes().general_rounds;            // test control
  const int max_rounds = forced > 0 ? forced : (pc == kP43 ? n + 1 : kMinRounds + n / 4);
  // one weight vector, p = 2 (forced rounds ask for the kernel that hands over)
  const bool shared = pc == kP2 && w_stride == 0 && forced == 0;
#define CALL(GL, E)                                                                                \
  (shared ? launch_general_shared<GL, E>(mag, x, w, tangent, out, jvp, rows, n, R, st)              \
          : launch_general_shape<GL, E>(mag, pc, x, w, w_stride, tangent, out, jvp, rows, n, R, st, \
                                        max_rounds))
  switch (np) {
    case 2: return CALL(1, 2);
    case 4: return CALL(1, 4);
    case 8: return CALL(1, 8);
    case 16: return CALL(2, 8);
    case 32: return CALL(4, 8);
    case 64: return CALL(8, 8);
    case 128: return CALL(16, 8);
    case 256: return CALL(32, 8);
    case 512: return CALL(64, 8);
    case 1024: return CALL(64, 16);
    default: return -1;
  }
#undef CALL
}

}  // namespace topk
