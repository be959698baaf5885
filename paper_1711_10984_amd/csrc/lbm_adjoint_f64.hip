// FP64 instantiation of the adjoint kernels (lbm_adjoint_impl.h), built without contraction like the
// forward FP64 kernels.
#include "lbm_adjoint_impl.h"

namespace lbm {
hipError_t launch_adjoint_total(hipStream_t s, const double* part, int n, double* out) {
  hipLaunchKernelGGL(k_adj_total, dim3(1), dim3(ADJ_THREADS), 0, s, part, n, out);
  return hipGetLastError();
}
LBM_INSTANTIATE_ADJOINT(double)
}  // namespace lbm
