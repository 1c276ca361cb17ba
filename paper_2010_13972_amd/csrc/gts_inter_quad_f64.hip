// Instantiates the quadrature interaction kernel for fp64 models.
#include "gts_inter_quad.h"

namespace gts {

size_t quad_lds_f64(int M, int rows, int waves, bool wide) {
  return quad_lds<double>(M, rows, waves, wide);
}

gts_status launch_inter_quad_f64(const KernelArgs& a, const Plan& p) {
  return launch_quad_shape<double>(a, p);
}

}  // namespace gts
