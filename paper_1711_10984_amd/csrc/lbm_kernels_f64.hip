// FP64 instantiation of the timestep kernels (lbm_kernels_impl.h) and the centre-of-mass reduction.
// Built without floating-point contraction: every FP64 expression is evaluated term by term in the
// order written, which is the order of the plain definitions.
#include "lbm_kernels_impl.h"
#include "lbm_tile_impl.h"

namespace lbm {

hipError_t launch_reduce(hipStream_t s, int tiling, int ndrop_total, const InstDev* inst, DropDev* drops, DropDev* out,
                         const double* part, const uint64_t* mask, int64_t* step, int increment) {
  const dim3 g(ndrop_total > 0 ? ndrop_total : 1), b(NTHREADS);
  if (out)
    hipLaunchKernelGGL((k_reduce<true>), g, b, 0, s, tiling, ndrop_total, inst, drops, out, part, mask, step, increment);
  else
    hipLaunchKernelGGL((k_reduce<false>), g, b, 0, s, tiling, ndrop_total, inst, drops, out, part, mask, step,
                       increment);
  return hipGetLastError();
}

hipError_t launch_tile_final(hipStream_t s, int ndrop_total, const InstDev* inst, DropDev* drops, const TileSeq& q,
                             int64_t* step, int64_t count) {
  hipLaunchKernelGGL(k_tile_final, dim3(ndrop_total > 0 ? ndrop_total : 1), dim3(64), 0, s, ndrop_total, inst, drops, q,
                     step, count);
  return hipGetLastError();
}

hipError_t launch_obs_final(hipStream_t s, const InstDev* insts, int inst, int ndrop, const DropDev* drops,
                            const double* part, int stride, double* res) {
  hipLaunchKernelGGL(k_obs_final, dim3(6 + ndrop), dim3(NTHREADS), 0, s, insts, inst, drops, part, stride, res);
  return hipGetLastError();
}

LBM_INSTANTIATE_FIELDS(double)
LBM_INSTANTIATE_POPS(double, double)
LBM_INSTANTIATE_TILE(double, double)

}  // namespace lbm
