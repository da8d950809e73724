// Shapes of row_search.hpp (threads per row x elements per thread): 1024 x 20, 1024 x 24, 1024 x 32.
#include "row_search.hpp"

namespace topk {

int launch_row_search_h(int threads, int e, int var, bool mag, int pc, bool vec, const float* x, const float* tangent, float* out,
                          float* jvp, float* loss, double lam_over_p, int64_t rows, int n, int k,
                          const Reg& R, hipStream_t st) {
  if (threads == 1024 && e == 20)
    return launch_row_search_shape<1024, 20>(var, mag, pc, vec, x, tangent, out, jvp, loss, lam_over_p,
                                           rows, n, k, R, st);
  if (threads == 1024 && e == 24)
    return launch_row_search_shape<1024, 24>(var, mag, pc, vec, x, tangent, out, jvp, loss, lam_over_p,
                                           rows, n, k, R, st);
  if (threads == 1024 && e == 32)
    return launch_row_search_shape<1024, 32>(var, mag, pc, vec, x, tangent, out, jvp, loss, lam_over_p,
                                           rows, n, k, R, st);
  return -2;
}

}  // namespace topk
