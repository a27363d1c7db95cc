// Launches of the plane passes for one precision PL_T (included by
// pl_plane_f64.hip / pl_plane_f32.hip).
#include "pl_passes.hpp"
#include "pl_plane.hpp"

namespace pl {

template <int CLS>
static hipError_t launch_plane_cls(int op, const RowArgs<PL_T>& a, dim3 grid, dim3 block, size_t lds, hipStream_t st) {
  switch (op) {
    case ROW_R2C: hipLaunchKernelGGL((plane_kernel<PL_T, ROW_R2C, CLS>), grid, block, lds, st, a); break;
    case ROW_C2R: hipLaunchKernelGGL((plane_kernel<PL_T, ROW_C2R, CLS>), grid, block, lds, st, a); break;
    case ROW_HVP: hipLaunchKernelGGL((plane_kernel<PL_T, ROW_HVP, CLS>), grid, block, lds, st, a); break;
    case ROW_C2R_DIAG: hipLaunchKernelGGL((plane_kernel<PL_T, ROW_C2R_DIAG, CLS>), grid, block, lds, st, a); break;
#if PL_T_IS_DOUBLE
    case ROW_GRAD: hipLaunchKernelGGL((plane_kernel<PL_T, ROW_GRAD, CLS>), grid, block, lds, st, a); break;
    case ROW_GRAD_STEP: hipLaunchKernelGGL((plane_kernel<PL_T, ROW_GRAD_STEP, CLS>), grid, block, lds, st, a); break;
    case ROW_C2R_GRADLIK:
      hipLaunchKernelGGL((plane_kernel<PL_T, ROW_C2R_GRADLIK, CLS>), grid, block, lds, st, a);
      break;
    case ROW_LB_IN:
      if constexpr (CLS == 0) {
        hipLaunchKernelGGL((plane_kernel<PL_T, ROW_LB_IN, CLS>), grid, block, lds, st, a);
        break;
      } else {
        return hipErrorInvalidValue;
      }
    case ROW_LB_OUT: hipLaunchKernelGGL((plane_kernel<PL_T, ROW_LB_OUT, CLS>), grid, block, lds, st, a); break;
#endif
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <>
hipError_t launch_plane<PL_T>(int op, const RowArgs<PL_T>& a, hipStream_t st, int* nblocks) {
  if (!plane_fits(a.ny, a.n, (int)sizeof(cx<PL_T>)) || a.nplanes < 1 || ((op == ROW_GRAD || op == ROW_GRAD_STEP) && a.model != MODEL_LOGNORMAL))
    return hipErrorInvalidValue;
  const dim3 grid(a.nplanes), block(64 * plane_waves(a.ny, a.n));
  const size_t lds = plane_lds_bytes(a.ny, a.n, (int)sizeof(cx<PL_T>));
  *nblocks = a.nplanes;
  return plane_class(a.ny, a.n) == 0 ? launch_plane_cls<0>(op, a, grid, block, lds, st)
                                     : launch_plane_cls<1>(op, a, grid, block, lds, st);
}

template <int CLS>
static hipError_t launch_plane_batch_cls(int op, const RowArgs<PL_T>* args, const int4* work, int nblocks, int threads,
                                         int lds, hipStream_t st) {
  const dim3 grid(nblocks), block(threads);
  switch (op) {
    case ROW_R2C: hipLaunchKernelGGL((row_batch_kernel<PL_T, ROW_R2C, CLS>), grid, block, lds, st, args, work); break;
    case ROW_C2R: hipLaunchKernelGGL((row_batch_kernel<PL_T, ROW_C2R, CLS>), grid, block, lds, st, args, work); break;
    case ROW_HVP: hipLaunchKernelGGL((row_batch_kernel<PL_T, ROW_HVP, CLS>), grid, block, lds, st, args, work); break;
#if PL_T_IS_DOUBLE
    case ROW_GRAD:
      hipLaunchKernelGGL((row_batch_kernel<PL_T, ROW_GRAD, CLS>), grid, block, lds, st, args, work);
      break;
#endif
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <>
hipError_t launch_plane_batch<PL_T>(int op, int cls, const RowArgs<PL_T>* args, const int4* work, int nblocks,
                                    int threads, int lds_bytes, hipStream_t st) {
  if (nblocks < 1 || threads < 64 || threads > 64 * PLANE_BATCH_WAVES || threads % 64 || lds_bytes < 0 || (size_t)lds_bytes > PLANE_LDS_MAX) return hipErrorInvalidValue;
  return cls == 0 ? launch_plane_batch_cls<0>(op, args, work, nblocks, threads, lds_bytes, st)
                  : launch_plane_batch_cls<1>(op, args, work, nblocks, threads, lds_bytes, st);
}

}  // namespace pl
