// Instantiates the quadrature interaction kernel for fp32 models.
#include "gts_inter_quad.h"

namespace gts {

size_t quad_lds_f32(int M, int rows, int waves, bool wide) {
  return quad_lds<float>(M, rows, waves, wide);
}

gts_status launch_inter_quad_f32(const KernelArgs& a, const Plan& p) {
  return launch_quad_shape<float>(a, p);
}

}  // namespace gts
