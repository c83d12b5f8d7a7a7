// cm_tt_round: in-place TT rounding (the recompression of Section 3.1, after Oseledets
// 2011) of every train in a batch, one workgroup per train, FP64 factorisations.
// One wavefront per train: the factorisations are chains of small dependent steps, so
// barriers over a single wave and more trains per CU beat wider workgroups.
#define CM_WG 64
#include "cm_round_kernel.h"

extern "C" size_t cm_round_slab_bytes(int n_max, int d, int cap) { return round_slab_bytes(n_max, d, cap); }
cm_status cm_round_wide(const TTView &v, int batch, double tol, int cap, int incap, double *err_out, int32_t *status,
                        char *ws, int slots, int n_max, int skip, hipStream_t s);
extern "C" int cm_slots_for_ws(int op, int batch, int n_max, int cap_rank, int dtype, size_t ws_bytes);

extern "C" cm_status cm_tt_round(cm_tt_batch *t, double tol, int cap_rank, double *err_out, int32_t *status,
                                 void *ws, size_t ws_bytes, void *stream) {
  if (!t || !(tol >= 0.0) || cap_rank < 1 || cap_rank > 64) return CM_E_INVALID;
  if (t->batch < 0 || t->n_max < 1 || t->n_max > CM_MAX_N) return CM_E_INVALID;
  if (t->dtype != CM_C64 && t->dtype != CM_C128) return CM_E_INVALID;
  if (t->d_out < 1 || t->d_in < 1 || t->d_out * t->d_in > 4) return CM_E_INVALID;
  if (t->cap_rank < 1 || t->cap_rank > 64) return CM_E_UNSUPPORTED;
  if (t->batch == 0) return CM_OK;
  // one workgroup per workspace slab (cm_workspace_bytes gives the default count)
  const int slots = cm_slots_for_ws(CM_OP_TT_ROUND, t->batch, t->n_max, t->cap_rank, t->dtype, ws ? ws_bytes : 0);
  if (slots < 1) return CM_E_INVALID;
  const int d = t->d_out * t->d_in;
  const size_t lds = RLDS;
  TTView v = tt_view(t);
  hipStream_t s = (hipStream_t)stream;
  const int skip = (t->flags & CM_TT_LEFT_ORTHO) ? 1 : 0;
  if (t->dtype == CM_C128 && wide_sweep(t->batch, t->n_max, cap_rank, tol, WIDE_TOL_ROUND)) {
    const cm_status e = cm_round_wide(v, t->batch, tol, cap_rank, t->cap_rank, err_out, status, (char *)ws, slots,
                                      t->n_max, skip, s);
    if (e == CM_OK) t->flags = CM_TT_RIGHT_ORTHO;
    return e;
  }
  CM_HIP_CHECK(cm_allow_lds(k_tt_round<float2>, lds));
  CM_HIP_CHECK(cm_allow_lds(k_tt_round<double2>, lds));
  if (t->dtype == CM_C64)
    hipLaunchKernelGGL(k_tt_round<float2>, dim3(slots), dim3(CM_WG), lds, s, v, t->batch, tol, cap_rank, t->cap_rank,
                       err_out, status, (char *)ws, t->n_max, t->dtype, skip);
  else
    hipLaunchKernelGGL(k_tt_round<double2>, dim3(slots), dim3(CM_WG), lds, s, v, t->batch, tol, cap_rank, t->cap_rank,
                       err_out, status, (char *)ws, t->n_max, t->dtype, skip);
  CM_LAUNCH_CHECK();
  t->flags = CM_TT_RIGHT_ORTHO;
  return CM_OK;
}
