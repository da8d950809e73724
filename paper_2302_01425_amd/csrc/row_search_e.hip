// Shapes of row_search.hpp (threads per row x elements per thread): 256 x 32, 512 x 16.
#include "row_search.hpp"

namespace topk {

int launch_row_search_e(int threads, int e, int var, bool mag, int pc, bool vec, const float* x, const float* tangent, float* out,
                          float* jvp, float* loss, double lam_over_p, int64_t rows, int n, int k,
                          const Reg& R, hipStream_t st) {
  if (threads == 256 && e == 32)
    return launch_row_search_shape<256, 32>(var, mag, pc, vec, x, tangent, out, jvp, loss, lam_over_p,
                                           rows, n, k, R, st);
  if (threads == 512 && e == 16)
    return launch_row_search_shape<512, 16>(var, mag, pc, vec, x, tangent, out, jvp, loss, lam_over_p,
                                           rows, n, k, R, st);
  return -2;
}

}  // namespace topk
