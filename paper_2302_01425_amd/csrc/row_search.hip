// Choice of the shape of row_search.hpp for a row length.
#include <cstdint>

#include "launch.hpp"

namespace topk {

#define TOPK_SEARCH_ARGS                                                                              \
  int threads, int e, int var, bool mag, int pc, bool vec, const float *x, const float *tangent,      \
      float *out, float *jvp, float *loss, double lam_over_p, int64_t rows, int n, int k, const Reg &R, \
      hipStream_t st
int launch_row_search_a(TOPK_SEARCH_ARGS);
int launch_row_search_b(TOPK_SEARCH_ARGS);
int launch_row_search_c(TOPK_SEARCH_ARGS);
int launch_row_search_d(TOPK_SEARCH_ARGS);
int launch_row_search_e(TOPK_SEARCH_ARGS);
int launch_row_search_f(TOPK_SEARCH_ARGS);
int launch_row_search_g(TOPK_SEARCH_ARGS);
int launch_row_search_h(TOPK_SEARCH_ARGS);

int launch_row_search(int var, bool mag, int pc, const float* x, const float* tangent, float* out,
                      float* jvp, float* loss, double lam_over_p, int64_t rows, int64_t n, int64_t k,
                      const Reg& R, hipStream_t st) {
  // the arrays that are accessed have to agree modulo 16 bytes for 16-byte accesses
  const uintptr_t at = reinterpret_cast<uintptr_t>(x) & 15u;
  auto agrees = [&](const void* p) { return p == nullptr || (reinterpret_cast<uintptr_t>(p) & 15u) == at; };
  const bool vec = agrees(tangent) && agrees(out) && agrees(jvp);
  // rows that do not all start at a 16-byte boundary need room for up to three elements before them
  const int64_t span = n + (at == 0 && n % 4 == 0 ? 0 : 3);
#define TOPK_SHAPE(F, T, E)                                                                                \
  if (span <= int64_t(T) * E)                                                                              \
  return launch_row_search_##F(T, E, var, mag, pc, vec, x, tangent, out, jvp, loss, lam_over_p, rows,      \
                               int(n), int(k), R, st)
  // The fewest threads a row fits: every pass costs its group one reduction, and float64 arithmetic is
  // done by every wavefront of a row; but at most 24 elements per thread until there are rows enough
  // to fill the chip without (32: 108 registers and half the wavefronts; 8192 elements, p = 2: 512
  // rows 16.5 us with 512 threads against 19.0 with 256, 2048 rows 50.3 / 48.5; p = 4/3 65.1 / 52.9),
  // and 8 where there are not even as many rows as compute units (4096 elements, 256 rows: 512
  // threads 9.8 us, 256 threads 11.4), or four rows per workgroup would leave compute units without one
  // (1200 elements, 300 / 1000 / 1500 rows: 14.7 / 15.2 / 16.7 us with 64 threads, 10.4 / 12.5 / 15.8 with
  // 256; 2000 elements, 128 against 256 threads: 12.0 / 13.2 / 15.6 and 10.5 / 13.2 / 15.7).
  if (rows <= 256 || (rows <= 1536 && n > 1024)) TOPK_SHAPE(b, 256, 8);
  if (rows <= 256) {
    TOPK_SHAPE(c, 512, 8);
    TOPK_SHAPE(f, 1024, 8);
    TOPK_SHAPE(g, 1024, 16);
  }
  TOPK_SHAPE(a, 64, 8);
  TOPK_SHAPE(a, 64, 16);
  TOPK_SHAPE(a, 64, 24);
  TOPK_SHAPE(b, 128, 16);
  // (3000 elements, 4 M in all: p = 2 20.4 us with 128 threads, 18.5 with 256; p = 4/3 22.8 / 25.5)
  if (pc == kP43) TOPK_SHAPE(b, 128, 24);
  TOPK_SHAPE(c, 256, 12);
  TOPK_SHAPE(c, 256, 16);
  TOPK_SHAPE(d, 256, 20);
  TOPK_SHAPE(d, 256, 24);
  if (rows <= 1024) TOPK_SHAPE(e, 512, 16);
  TOPK_SHAPE(e, 256, 32);
  TOPK_SHAPE(f, 512, 20);
  TOPK_SHAPE(f, 512, 24);
  if (rows <= 512) TOPK_SHAPE(g, 1024, 16);
  TOPK_SHAPE(g, 512, 32);
  TOPK_SHAPE(h, 1024, 20);
  TOPK_SHAPE(h, 1024, 24);
  TOPK_SHAPE(h, 1024, 32);
#undef TOPK_SHAPE
  return -2;
}

}  // namespace topk
