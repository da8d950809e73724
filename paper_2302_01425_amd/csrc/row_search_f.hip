// Shapes of row_search.hpp (threads per row x elements per thread): 512 x 20, 512 x 24, 1024 x 8.
#include "row_search.hpp"

namespace topk {

int launch_row_search_f(int threads, int e, int var, bool mag, int pc, bool vec, const float* x, const float* tangent, float* out,
                          float* jvp, float* loss, double lam_over_p, int64_t rows, int n, int k,
                          const Reg& R, hipStream_t st) {
  if (threads == 512 && e == 20)
    return launch_row_search_shape<512, 20>(var, mag, pc, vec, x, tangent, out, jvp, loss, lam_over_p,
                                           rows, n, k, R, st);
  if (threads == 512 && e == 24)
    return launch_row_search_shape<512, 24>(var, mag, pc, vec, x, tangent, out, jvp, loss, lam_over_p,
                                           rows, n, k, R, st);
  if (threads == 1024 && e == 8)
    return launch_row_search_shape<1024, 8>(var, mag, pc, vec, x, tangent, out, jvp, loss, lam_over_p,
                                           rows, n, k, R, st);
  return -2;
}

}  // namespace topk
