// cm_sample_outcomes: measurement outcomes of the QFT register (Section 2.2, Eq.
// qft_probabilities) drawn from an SFFT output train without forming its 2^n amplitudes.
//
// Output core l carries outcome bit 2^l, so the probability mass of the outcomes whose low
// t+1 bits are (b_0, ..., b_t) is
//   q(b_0..b_t) = w E_{t+1} w^H,   w = Y_0[0,b_0,:] Y_1[:,b_1,:] ... Y_t[:,b_t,:]  (a row),
// with the right environments E_l = sum_b Y_l[:,b,:] E_{l+1} Y_l[:,b,:]^H, E_n = [1]: E_l
// is the Gram matrix of the right partial contractions, and E_0 = ||y||^2. A shot fixes
// bit 0 first. With prefix row w of mass q, let w0 = w Y_t[:,0,:] and q0 = w0 E_{t+1} w0^H;
// bit t is 1 iff U_t q >= q0 for the shot's uniform U_t, and the prefix becomes
// w Y_t[:,bit,:] with its own mass. Every decision is taken in FP64 whatever the storage
// precision of the train.
//
// k_envs: one workgroup per instance builds E_n, ..., E_0 in LDS and stores E_1..E_n and
// the FP64 cores in the workspace, zero-padded to even bond dimensions (multiples of 4 in
// trains with bonds above 16). k_sample: one lane per shot holding its prefix row in registers
// (sized by a compile-time bound on the instance's largest bond); the products run over 4 x 4
// blocks of the padded operands, 2 wide at the remainder, whose addresses are the same for
// every lane, so the operands arrive through scalar loads and each block's loads are issued
// together.
//
// k_sample is bound by the FP64 multiply-adds it executes and, with three waves a SIMD, by the
// scalar loads between them; so what counts is how much of the work is padding and how far the
// loads run ahead. Blocks of 4 made 1.43 times the work out of a bond of 10. Up to bonds of 16
// the padding is to 2, bonds up to 4, 8, 12 and 16 have an instantiation each, and the two largest even
// sizes of each have branch-free code. Up to 4 it fits eight waves a SIMD, up to 8 and 12 it is held
// to four, up to 16 to three (at 12 and 16 that spills a few registers: 24 and 6). 512 Heston trains of
// n = 24 (bonds <= 10), 4096 shots: 2.53 -> 1.93 ms. 64 trains of n = 20, 4096 shots, the whole call,
// in us (4 x 4 blocks in front): bonds of 2 117 -> 83, 4 123 -> 118 (128 in the instantiation for 8), 6
// 231 -> 176, 8 239 -> 237, 10 559 -> 332, 12 573 -> 417. 256 trains, ms: 14 2.54 -> 1.92,
// 16: 2.57 -> 2.31. Above 16 the same blocks of 2 are 9 % slower than whole ones (24: 14.2 against
// 12.7 ms; one wave a SIMD, and the remainder is a small part): those keep blocks of 4. Orthonormal
// rows in place of the environments (a mass is then ||w||^2: a third of the work less) took
// 1.60 ms here, but the factorisations 0.64 against k_envs' 0.11, and the masses' error against
// extended precision is 2.6e-15 against 1.0e-15.
#include "cm_internal.h"

namespace {

constexpr int SMP_WG = 256;
constexpr int SMP_RS = 32;  // largest bond dimension the sampler takes

__device__ __forceinline__ int max_bond_of(const int32_t *rk, int n) {
  int r = 1;
  for (int l = 0; l <= n; ++l) r = rk[l] > r ? rk[l] : r;
  return r;
}

__host__ __device__ __forceinline__ int pad4(int r) { return (r + 3) & ~3; }
// bonds up to PAD2_MAX are padded to multiples of 2, wider trains' to multiples of 4
constexpr int PAD2_MAX = 16;
__device__ __forceinline__ int pad_bond(int r, bool wide) { return wide ? pad4(r) : (r + 1) & ~1; }

// Workspace slab of one instance (complex FP64 elements):
//   the largest bond, an int, at 0
//   E_l, l = 1..n:   at l * RS * RS, [p(r_l)][p(r_l)]
//   Y_l, l = 0..n-1: at (n_max + 1) RS^2 + l * 2 RS^2, [p(r_l)][2][p(r_{l+1})]
// with p = pad_bond and zeros in the padding.
template <typename T>
__global__ __launch_bounds__(SMP_WG) void k_envs(TTView y, int RS, int n_max, int64_t inst_stride,
                                                 double2 *__restrict__ ws, double *__restrict__ norm2,
                                                 int32_t *__restrict__ status) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  double2 *Yd = (double2 *)lds_raw;   // [r_l][2][r_{l+1}]
  double2 *Tm = Yd + 2 * RS * RS;     // [2][r_l][r_{l+1}]
  double2 *Ea = Tm + 2 * RS * RS;     // E_{l+1}
  double2 *Eb = Ea + RS * RS;         // E_l
  const int tid = threadIdx.x;
  const int b = blockIdx.x;
  const int n = y.n[b];
  if (n < 0 || n > n_max) {   // the slab holds n_max levels
    if (tid == 0) {
      norm2[b] = NAN;
      set_status(status, b, CM_E_INVALID);
    }
    return;
  }
  const int32_t *rk = y.rk(b);
  const int rmax = max_bond_of(rk, n);
  double2 *Eg = ws + (int64_t)b * inst_stride;
  if (tid == 0) *(int32_t *)Eg = rmax;
  if (rmax > RS) {
    if (tid == 0) {
      norm2[b] = NAN;
      set_status(status, b, CM_E_UNSUPPORTED);
    }
    return;
  }
  double2 *Yg = Eg + (int64_t)(n_max + 1) * RS * RS;
  const T *cores = (const T *)y.cores;
  const bool wide = rmax > PAD2_MAX;
  // E_n = [1], padded to at most 4 x 4 (a train of no cores has no level that reads it, and its
  // place is the largest bond's)
  for (int e = tid; e < 16 && n > 0; e += SMP_WG) Eg[(int64_t)n * RS * RS + e] = cmk(e == 0 ? 1.0 : 0.0, 0.0);
  if (tid == 0) Ea[0] = cmk(1.0, 0.0);
  __syncthreads();
  for (int l = n - 1; l >= 0; --l) {
    const int ra = rk[l], rb = rk[l + 1];
    const int pa = pad_bond(ra, wide), pb = pad_bond(rb, wide);
    const T *C = cores + y.coff(b, l);
    for (int e = tid; e < ra * 2 * rb; e += SMP_WG) Yd[e] = cstore<T>::ld(C, e);
    // padded FP64 copy of the core for the sampler
    double2 *Yl = Yg + (int64_t)l * 2 * RS * RS;
    for (int e = tid; e < pa * 2 * pb; e += SMP_WG) {
      const int a = e / (2 * pb), bit = (e / pb) % 2, c = e % pb;
      Yl[e] = (a < ra && c < rb) ? cstore<T>::ld(C, (a * 2 + bit) * rb + c) : cmk(0.0, 0.0);
    }
    __syncthreads();
    // Tm[bit][c][f] = sum_e Y[c][bit][e] E_{l+1}[e][f]
    for (int e = tid; e < 2 * ra * rb; e += SMP_WG) {
      const int bit = e / (ra * rb), c = (e / rb) % ra, f = e % rb;
      const double2 *row = Yd + (c * 2 + bit) * rb;
      double2 acc = cmk(0.0, 0.0);
      for (int q = 0; q < rb; ++q) cfma(acc, row[q], Ea[q * rb + f]);
      Tm[e] = acc;
    }
    __syncthreads();
    // E_l[c][d] = sum_bit sum_f Tm[bit][c][f] conj(Y[d][bit][f])
    for (int e = tid; e < ra * ra; e += SMP_WG) {
      const int c = e / ra, d = e % ra;
      double2 acc = cmk(0.0, 0.0);
      for (int bit = 0; bit < 2; ++bit) {
        const double2 *tr = Tm + (bit * ra + c) * rb;
        const double2 *yr = Yd + (d * 2 + bit) * rb;
        for (int f = 0; f < rb; ++f) ccfma(acc, yr[f], tr[f]);
      }
      Eb[e] = acc;
    }
    __syncthreads();
    if (l > 0) {
      double2 *El = Eg + (int64_t)l * RS * RS;
      for (int e = tid; e < pa * pa; e += SMP_WG) {
        const int c = e / pa, d = e % pa;
        El[e] = (c < ra && d < ra) ? Eb[c * ra + d] : cmk(0.0, 0.0);
      }
    }
    double2 *t = Ea; Ea = Eb; Eb = t;
  }
  if (tid == 0) {
    const double nv = Ea[0].x;
    norm2[b] = nv;
    if (!isfinite(nv)) set_status(status, b, CM_E_NONFINITE);
    else if (!(nv > 0.0)) set_status(status, b, CM_E_INVALID);
  }
}

// w <- v Y[:, bit, :] over blocks of the padded core Y (rows of ld, pb of them used; pa, pb <= RM).
// Entries of v past the bond are zero, and so is Y's padding. WHOLE: pa and pb are multiples of 4;
// else they are even and the last block of each is 2 wide where that is enough.
template <int RM> constexpr bool WHOLE = RM > PAD2_MAX;

template <int RA, int RB>
__device__ __forceinline__ void block_product(const double2 *v, const double2 *__restrict__ Y, int ld, double2 *w) {
  double2 yb[RA][RB];
#pragma unroll
  for (int i = 0; i < RA; ++i)
#pragma unroll
    for (int j = 0; j < RB; ++j) yb[i][j] = Y[i * ld + j];
#pragma unroll
  for (int i = 0; i < RA; ++i)
#pragma unroll
    for (int j = 0; j < RB; ++j) cfma(w[j], v[i], yb[i][j]);
}

template <int RM, int RB>
__device__ __forceinline__ void column_product(const double2 *v, const double2 *__restrict__ Y, int pa, int ld,
                                               double2 *w) {
#pragma unroll
  for (int a = 0; a < RM; a += 4) {
    if (a + 4 <= pa) block_product<4, RB>(v + a, Y + a * ld, ld, w);
    else if (!WHOLE<RM> && a < pa) block_product<2, RB>(v + a, Y + a * ld, ld, w);
  }
}

template <int RM>
__device__ __forceinline__ void row_times_core(const double2 *v, const double2 *__restrict__ Y, int pa, int pb,
                                               double2 *w) {
#pragma unroll
  for (int c = 0; c < RM; ++c) w[c] = cmk(0.0, 0.0);
#pragma unroll
  for (int c = 0; c < RM; c += 4) {
    if (c + 4 <= pb) column_product<RM, 4>(v, Y + c, pa, 2 * pb, w + c);
    else if (!WHOLE<RM> && c < pb) column_product<RM, 2>(v, Y + c, pa, 2 * pb, w + c);
  }
}

// w E w^H for Hermitian E (padded [p][p], p <= RM) from its upper triangle, by blocks.
// z_i += sum_d conj(E[i][d]) w[d] over one block of CW rows and DW columns
template <int CW, int DW>
__device__ __forceinline__ void form_block(const double2 *w, const double2 *__restrict__ E, int p, double2 *z) {
  double2 eb[CW][DW];
#pragma unroll
  for (int i = 0; i < CW; ++i)
#pragma unroll
    for (int j = 0; j < DW; ++j) eb[i][j] = E[i * p + j];
#pragma unroll
  for (int i = 0; i < CW; ++i)
#pragma unroll
    for (int j = 0; j < DW; ++j) ccfma(z[i], eb[i][j], w[j]);
}

// rows c .. c + CW - 1 of the form: w and E start at entry (c, c), `rest` entries from there on
template <bool W, int MAXD, int CW>
__device__ __forceinline__ void form_rows(const double2 *w, const double2 *__restrict__ E, int p, int rest,
                                          double &acc) {
  double2 z[CW], eb[CW][CW];   // the diagonal block, its upper triangle
#pragma unroll
  for (int i = 0; i < CW; ++i)
#pragma unroll
    for (int j = i; j < CW; ++j) eb[i][j] = E[i * p + j];
#pragma unroll
  for (int i = 0; i < CW; ++i) {
    z[i] = cmk(0.0, 0.0);
#pragma unroll
    for (int j = i + 1; j < CW; ++j) ccfma(z[i], eb[i][j], w[j]);
  }
  if (CW == 4) {
#pragma unroll
    for (int d = 4; d < MAXD; d += 4) {
      if (d + 4 <= rest) form_block<CW, 4>(w + d, E + d, p, z);
      else if (!W && d < rest) form_block<CW, 2>(w + d, E + d, p, z);
    }
  }
#pragma unroll
  for (int i = 0; i < CW; ++i) {
    acc = fma(eb[i][i].x, cabs2(w[i]), acc);
    acc = fma(2.0, w[i].x * z[i].x + w[i].y * z[i].y, acc);
  }
}

template <int RM, int C>
__device__ __forceinline__ void form_from(const double2 *w, const double2 *__restrict__ E, int p, double &acc) {
  if constexpr (C < RM) {
    if (C + 4 <= p) form_rows<WHOLE<RM>, RM - C, 4>(w + C, E + C * p + C, p, p - C, acc);
    else if (!WHOLE<RM> && C < p) form_rows<WHOLE<RM>, RM - C, 2>(w + C, E + C * p + C, p, p - C, acc);
    form_from<RM, C + 4>(w, E, p, acc);
  }
}

// one continuation: w <- v Y, returns its mass
template <int RM>
__device__ __forceinline__ double continuation(const double2 *v, const double2 *Y, const double2 *E, int pa, int pb,
                                               double2 *w) {
  double acc = 0.0;
  row_times_core<RM>(v, Y, pa, pb, w);
  form_from<RM, 0>(w, E, pb, acc);
  return acc;
}

template <int RM>
__global__ __launch_bounds__(SMP_WG, RM <= 4 ? 8 : RM <= 12 ? 4 : RM <= 16 ? 3 : 1) void k_sample(TTView y, const double2 *__restrict__ ws, int RS, int n_max,
                                                   int64_t inst_stride, const double *__restrict__ norm2,
                                                   const double *__restrict__ uni, int ustride, int R,
                                                   int64_t *__restrict__ out, int rm_lo) {
  const int tid = threadIdx.x;
  const int b = blockIdx.y;
  const int n = y.n[b];
  const int s = blockIdx.x * SMP_WG + tid;
  if (n < 0 || n > n_max) {   // k_envs has set CM_E_INVALID
    if (rm_lo == 0 && s < R) out[(int64_t)b * R + s] = -1;   // the always-launched bound marks it
    return;
  }
  const int32_t *rk = y.rk(b);
  // this instantiation serves instances whose largest bond lies in (rm_lo, RM]; the widest
  // one also writes -1 for instances above every bound
  const double2 *Eg = ws + (int64_t)b * inst_stride;
  const int rmax = *(const int32_t *)Eg;
  if (rmax <= rm_lo) return;
  if (s >= R) return;
  const double q_all = norm2[b];
  if (rmax > RM || !(q_all > 0.0) || !isfinite(q_all)) {
    if (rmax <= RM || RM == SMP_RS) out[(int64_t)b * R + s] = -1;
    return;
  }
  // uniforms are bit-major, [batch][ustride][R]: level t of consecutive shots is contiguous
  const double *U = uni + (int64_t)b * ustride * R + s;
  const double2 *Yg = Eg + (int64_t)(n_max + 1) * RS * RS;
  double2 v[RM], w[RM];
#pragma unroll
  for (int a = 0; a < RM; ++a) v[a] = cmk(0.0, 0.0);
  v[0] = cmk(1.0, 0.0);
  double q = q_all;
  int64_t idx = 0;
  for (int t = 0; t < n; ++t) {
    const int pa = pad_bond(rk[t], WHOLE<RM>), pb = pad_bond(rk[t + 1], WHOLE<RM>);
    const double ut = U[(int64_t)t * R];
    const double2 *Y = Yg + (int64_t)t * 2 * RS * RS;
    const double2 *E = Eg + (int64_t)(t + 1) * RS * RS;
    // up to 16 one copy of the products' code serves both bits, as the sizes that fill most of a
    // chain (both bonds the largest or the next even one) have copies of their own: without
    // branches between the blocks the scalar loads run ahead of the products. Lanes that keep bit 0
    // sit out the second pass.
    const double lim = ut * q;
    bool more = true;
#pragma unroll(RM > PAD2_MAX ? 2 : 1)
    for (int bit = 0; bit < 2; ++bit) {
      if (more) {
        const double2 *Yb = Y + bit * pb;
        if (RM <= PAD2_MAX && pa == RM - 2 && pb == RM - 2) q = continuation<RM>(v, Yb, E, RM - 2, RM - 2, w);
        else if (RM <= PAD2_MAX && pa == RM && pb == RM) q = continuation<RM>(v, Yb, E, RM, RM, w);
        else q = continuation<RM>(v, Yb, E, pa, pb, w);
        if (bit) idx |= (int64_t)1 << t;
        more = lim >= q;
      }
    }
#pragma unroll
    for (int a = 0; a < RM; ++a) v[a] = w[a];
  }
  out[(int64_t)b * R + s] = idx;
}

// slot edge: the bond bound rounded up to a multiple of 4 (the padded blocks fit)
int env_rs(int cap_rank) { return pad4(cap_rank < SMP_RS ? cap_rank : SMP_RS); }

}  // namespace

// environments (n_max + 1) RS^2 plus padded FP64 cores 2 n_max RS^2 per instance
extern "C" size_t cm_sample_ws_bytes(int batch, int n_max, int cap_rank) {
  const int RS = env_rs(cap_rank);
  return (size_t)batch * (size_t)(3 * n_max + 1) * RS * RS * sizeof(double2);
}

extern "C" cm_status cm_sample_outcomes(const cm_tt_batch *y, const double *uniforms, int R, int64_t *out,
                                        double *norm2, int32_t *status, void *ws, size_t ws_bytes, void *stream) {
  if (!y || !norm2 || R < 0) return CM_E_INVALID;
  if (y->d_out != 2 || y->d_in != 1 || y->batch < 0) return CM_E_INVALID;
  if (y->dtype != CM_C64 && y->dtype != CM_C128) return CM_E_INVALID;
  if (y->cap_rank < 1 || y->cap_rank > 256 || y->n_max < 1 || y->n_max > CM_MAX_N) return CM_E_INVALID;
  if (y->batch == 0) return CM_OK;
  if (y->batch > 65535) return CM_E_UNSUPPORTED;
  if (R > 0 && (!uniforms || !out)) return CM_E_INVALID;
  const int RS = env_rs(y->cap_rank);
  const int64_t inst_stride = (int64_t)(3 * y->n_max + 1) * RS * RS;
  if (!ws || ws_bytes < cm_sample_ws_bytes(y->batch, y->n_max, y->cap_rank)) return CM_E_INVALID;
  hipStream_t s = (hipStream_t)stream;
  TTView v = tt_view(y);
  double2 *slab = (double2 *)ws;
  const int nm = y->n_max;
  const size_t env_lds = (size_t)6 * RS * RS * sizeof(double2);
  if (y->dtype == CM_C64) {
    CM_HIP_CHECK(cm_allow_lds(k_envs<float2>, env_lds));
    hipLaunchKernelGGL(k_envs<float2>, dim3((unsigned)y->batch), dim3(SMP_WG), env_lds, s, v, RS, nm, inst_stride,
                       slab, norm2, status);
  } else {
    CM_HIP_CHECK(cm_allow_lds(k_envs<double2>, env_lds));
    hipLaunchKernelGGL(k_envs<double2>, dim3((unsigned)y->batch), dim3(SMP_WG), env_lds, s, v, RS, nm, inst_stride,
                       slab, norm2, status);
  }
  CM_LAUNCH_CHECK();
  if (R == 0) return CM_OK;
  const dim3 grid((unsigned)((R + SMP_WG - 1) / SMP_WG), (unsigned)y->batch);
  const int us = y->n_max;
#define CM_SAMPLE_LAUNCH(RM, LO)                                                                         \
  hipLaunchKernelGGL((k_sample<RM>), grid, dim3(SMP_WG), 0, s, v, slab, RS, nm, inst_stride, norm2, uniforms, us, R, \
                     out, LO)
  CM_SAMPLE_LAUNCH(4, 0);
  if (y->cap_rank > 4) CM_SAMPLE_LAUNCH(8, 4);
  if (y->cap_rank > 8) CM_SAMPLE_LAUNCH(12, 8);
  if (y->cap_rank > 12) CM_SAMPLE_LAUNCH(16, 12);
  if (y->cap_rank > 16) CM_SAMPLE_LAUNCH(32, 16);
#undef CM_SAMPLE_LAUNCH
  CM_LAUNCH_CHECK();
  return CM_OK;
}
