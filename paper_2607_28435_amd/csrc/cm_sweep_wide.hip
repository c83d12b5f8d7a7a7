// The rounding sweeps on four waves per train, for small batches of long trains (see
// wide_sweep).
#define CM_WG 256
#include "cm_qtt_round.h"
#include "cm_round_kernel.h"

cm_status cm_round_wide(const TTView &v, int batch, double tol, int cap, int incap, double *err_out, int32_t *status,
                        char *ws, int slots, int n_max, int skip, hipStream_t s) {
  CM_HIP_CHECK(cm_allow_lds(k_tt_round<double2>, RLDS));
  hipLaunchKernelGGL(k_tt_round<double2>, dim3(slots), dim3(CM_WG), RLDS, s, v, batch, tol, cap, incap, err_out, status,
                     ws, n_max, CM_C128, skip);
  CM_LAUNCH_CHECK();
  return CM_OK;
}

cm_status cm_build_round_wide(const cm_problem *prob, int cnt, double tol, int cap, const TTView &x, int32_t *status,
                              char *ws, size_t slab, int n_max, hipStream_t s) {
  CM_HIP_CHECK(cm_allow_lds(k_build_round<double2>, QLDS));
  hipLaunchKernelGGL(k_build_round<double2>, dim3(cnt), dim3(CM_WG), QLDS, s, prob, tol, cap, x, status, ws, slab, n_max);
  CM_LAUNCH_CHECK();
  return CM_OK;
}
