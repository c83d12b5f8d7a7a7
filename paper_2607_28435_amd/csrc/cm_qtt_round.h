// Workspace slab of the QTT build, and k_build_round, its rounding sweep over one workgroup of
// CM_WG threads per train (compiled for the workgroup size of each including file).
#pragma once
#include "cm_tt.h"

namespace {

constexpr int QP = 10;          // Chebyshev nodes per polynomial leaf
constexpr int QNC = 96;         // max candidate intervals per depth
constexpr int QI = QNC / 2;     // max split intervals per depth
constexpr int QNPT = 2 * QP - 1;
constexpr int PRE_CAP = QI + QP + 1;   // bond bound before rounding (<= 64)
// LDS arena per workgroup: small on purpose (see cm_round.hip), and with the static LDS
// within a sixteenth of the CU's 160 KB so that the rounding launch keeps four one-wave
// workgroups per SIMD; the tree phase's candidate values live in the slab.
constexpr int QLDS = CM_WG == 64 ? 7680 : 32 * 1024;

struct TreeDepth {
  int n_int;                 // split intervals at this depth
  int n_cand;                // candidates = 2 * split intervals of the previous depth
  int64_t int_a[QI];         // prefixes of split intervals
  int8_t kind[QNC];          // 0 zero leaf, 1 split, 2 value leaf
  int8_t idx[QNC];           // index into int_a (kind 1)
  double2 vals[QNC][QP];     // values of value leaves at their nodes (or points)
};

struct QttSlab {
  TreeDepth *tree;    // [n+1]
  double2 *pre;       // pre-rounding train, n cores of PRE_CAP*2*PRE_CAP
  int32_t *pre_ranks; // [CM_MAX_N + 1]
  int64_t *pre_off;   // [CM_MAX_N]
  RoundScratch rs;
};

__host__ __device__ inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

// Slab layout (bytes) for one workgroup; also used by the host workspace query.
__host__ __device__ inline size_t qtt_slab_bytes(int n_max, int cap, size_t *parts) {
  const int capm = cap > PRE_CAP ? cap : PRE_CAP;
  const size_t core_cap = (size_t)capm * 2 * capm;
  size_t o = 0;
  parts[0] = o; o += align256(sizeof(TreeDepth) * (size_t)(n_max + 1));
  parts[1] = o; o += align256(sizeof(double2) * (size_t)PRE_CAP * 2 * PRE_CAP * n_max);
  parts[2] = o; o += align256(sizeof(int32_t) * (CM_MAX_N + 2));   // ranks, then the instance mark
  parts[3] = o; o += align256(sizeof(int64_t) * CM_MAX_N);
  parts[4] = o; o += align256(sizeof(double2) * core_cap * n_max);  // rs.tt
  parts[5] = o; o += align256(sizeof(double2) * core_cap * 6);      // rs.Y..C
  parts[6] = o; o += align256(sizeof(double2) * 2 * 64 * 64);        // global Jacobi pair
  parts[7] = o; o += align256(sizeof(double2) * QNC * QNPT);         // candidate values
  return o;
}

// Index of the slab's instance mark: the instance whose pre-rounding train the slab holds,
// or -1 (set by k_build_qtt, read by k_build_round).
constexpr int QMARK = CM_MAX_N + 1;

__device__ inline QttSlab qtt_slab_view(char *slab, int n_max, int cap) {
  size_t parts[8];
  qtt_slab_bytes(n_max, cap, parts);
  QttSlab W;
  W.tree = (TreeDepth *)(slab + parts[0]);
  W.pre = (double2 *)(slab + parts[1]);
  W.pre_ranks = (int32_t *)(slab + parts[2]);
  W.pre_off = (int64_t *)(slab + parts[3]);
  const int capm = cap > PRE_CAP ? cap : PRE_CAP;
  W.rs.core_cap = (int64_t)capm * 2 * capm;
  W.rs.tt = (double2 *)(slab + parts[4]);
  double2 *mats = (double2 *)(slab + parts[5]);
  W.rs.Y = mats; W.rs.X = mats + W.rs.core_cap; W.rs.Z = mats + 2 * W.rs.core_cap;
  W.rs.L = mats + 3 * W.rs.core_cap; W.rs.R = mats + 4 * W.rs.core_cap; W.rs.C = mats + 5 * W.rs.core_cap;
  W.rs.S = (double2 *)(slab + parts[6]);
  W.rs.J = W.rs.S + 64 * 64;
  return W;
}

}  // namespace

// Rounds the pre-rounding train of slab g (if k_build_qtt marked one) into x, with cores
// 1..n-1 right-orthonormal, and writes the instance's status.
#if CM_WG == 64
inline namespace wg64 {
#else
inline namespace wg256 {
#endif
template <typename OutT>
__global__ __launch_bounds__(CM_WG, 4) void k_build_round(const cm_problem *__restrict__ prob, double tol, int cap,
                                                       TTView x, int32_t *__restrict__ status,
                                                       char *__restrict__ ws, size_t slab_bytes, int n_max) {
  extern __shared__ __align__(16) char lds_arena[];
  __shared__ la::Sh sh;
  __shared__ int code_sh;
  const int tid = threadIdx.x;
  QttSlab W = qtt_slab_view(ws + (size_t)blockIdx.x * slab_bytes, n_max, cap);
  const int b = W.pre_ranks[QMARK];
  if (b < 0) return;
  const int n = prob[b].n;
  if (tid == 0) code_sh = CM_OK;
  __syncthreads();
  CoreSrc src;
  src.cores = W.pre; src.off = W.pre_off; src.ranks = W.pre_ranks; src.dtype = CM_C128;
  const double err = round_train_auto<OutT>(n, 2, src, tol, cap, (OutT *)x.cores, x.off + (int64_t)b * CM_MAX_N,
                                            x.rk(b), W.rs, lds_arena, QLDS, sh, &code_sh);
  (void)err;
  __syncthreads();
  if (tid == 0 && status) status[b] = code_sh;
}
}  // namespace wg64 or wg256
