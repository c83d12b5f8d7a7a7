// cm_fft_price: dense Carr–Madan baseline (Section 2.1, Eqs. x, dft, discretization_dft).
//
// Only the real part of ro (+-1)^u y_u is a price, so the transform is of half length. With
// z_j = ro x_{(j + jmid) mod M} (jmid the index of v = 0, which absorbs the sign (+-1)^u) the
// prices' f_u = Re sum_j z_j w^{ju}, w = exp(-2 pi i / M), are a real sequence, and
//   g_v = f_{2v} + i f_{2v+1} = sum_{j < h} G_j exp(-2 pi i j v / h),   h = M / 2,
//   G_j = ((1 + i w^j) (z_j + conj z_{M-j}) + (1 - i w^j) (z_{j+h} + conj z_{h-j})) / 2
// (indices of z mod M): one complex DFT of N = h points gives two neighbouring strikes per
// point, with half the arithmetic and half the bytes of the M-point DFT.
//
// Mixed-radix Stockham FFT (decimation in time, autosorting). Pass p with radix R_p and
// stride p_len = R_1 ... R_{p-1} maps work item i in [0, N/R_p), k = i mod p_len, as
//   u[r] = G[i + r N/R_p] * exp(-2 pi i r k / (R_p p_len)),  u <- DFT_{R_p}(u),
//   y[(i - k) R_p + k + r p_len] = u[r].
// Inside a workgroup each R_p-point DFT is itself a Stockham FFT in LDS with register radix
// 16 for CM_C64 and 8 for CM_C128 (smaller radices for the remaining bits): a thread reads its
// butterflies' points into registers, the workgroup synchronises, and the thread writes the
// transformed points back, so one LDS buffer suffices. A thread holds 16 (CM_C64) or 8 points, so
// small transforms take small workgroups. LDS indices carry one pad slot per 16 against bank
// conflicts.
//   - Pass 1 (p_len = 1, one work item per workgroup, radix up to 2^14 for CM_C64 and 2^13 for
//     CM_C128) generates G on the fly, so it reads nothing from HBM. x is set to exactly zero
//     where |psi| has decayed below a per-problem cutoff far under the storage precision (found
//     once per problem by k_fft_prepare), which skips the characteristic function outside the
//     integrand's numerical support and the stages that would only spread zeros.
//   - Later passes handle 16 consecutive work items per workgroup up to 2^9 points (CM_C64) or 2^8, 8 and
//     then 4 at the two radices above, so a load or store moves 128 (CM_C64) or 256 consecutive bytes,
//     32 or 64 at the largest radix.
//   - The last pass multiplies by the readout scalars and stores prices; in FP64 each price
//     takes its log-strike from the error-free grid sum (1e-15 NRMSE on the paper grid up
//     to n = 30). When strikes are chosen it stores g, and the gather prices those alone.
// Characteristic functions run in the storage precision (FP32 for CM_C64); every phase that
// grows with j or u is reduced exactly in FP64 first.
#include <array>
#include <utility>
#include <type_traits>

#include "cm_cf.h"
#include "cm_tt.h"

namespace {

constexpr int NT_MAX = 1024;   // threads per FFT workgroup (at most)
constexpr size_t DENSE_PROB_BYTES = 512;  // workspace slot per problem
constexpr int MAX_CHUNK = 32768;
constexpr int CUS = 256;
constexpr int PREP_ONE = 3000;

template <typename T> struct fr;
template <> struct fr<float2> {
  using R = float;
  __device__ __forceinline__ static float2 mk(double a, double b) { return make_float2((float)a, (float)b); }
  __device__ __forceinline__ static float2 mk2(float a, float b) { return make_float2(a, b); }
  __device__ __forceinline__ static float2 mul(float2 a, float2 b) { return fmulc(a, b); }
  __device__ __forceinline__ static float2 add(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
  __device__ __forceinline__ static float2 sub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
  // exp(-2 pi i f), f a turn fraction
  __device__ __forceinline__ static float2 cis_neg(double f) {
    // the argument's rounding (up to 2^-24 of a half turn) is put back as a small rotation
    const double x = -2.0 * (f - rint(f));
    const float xf = (float)x, d = (float)(M_PI * (x - (double)xf));
    float s, c;
    sincospif(xf, &s, &c);
    return make_float2(fmaf(-s, d, c), fmaf(c, d, s));
  }
};
template <> struct fr<double2> {
  using R = double;
  __device__ __forceinline__ static double2 mk(double a, double b) { return cmk(a, b); }
  __device__ __forceinline__ static double2 mk2(double a, double b) { return cmk(a, b); }
  __device__ __forceinline__ static double2 mul(double2 a, double2 b) { return cmul(a, b); }
  __device__ __forceinline__ static double2 add(double2 a, double2 b) { return cadd(a, b); }
  __device__ __forceinline__ static double2 sub(double2 a, double2 b) { return csub(a, b); }
  __device__ __forceinline__ static double2 cis_neg(double f) {
    double s, c;
    sincospi(-2.0 * f, &s, &c);
    return cmk(c, s);
  }
};

// cos(2 pi m / 16) for any integer m
__host__ __device__ constexpr double cos16(int m) {
  m &= 15;
  if (m > 8) m = 16 - m;
  return m == 0 ? 1.0 : m == 1 ? 0.92387953251128676 : m == 2 ? 0.70710678118654752 : m == 3 ? 0.38268343236508977
       : m == 4 ? 0.0 : m == 5 ? -0.38268343236508977 : m == 6 ? -0.70710678118654752 : m == 7 ? -0.92387953251128676
       : -1.0;
}

struct FftPlan {
  int n, npass;    // the transform has 2^(n-1) points
  int logr[4];     // radix bits per pass
  int bufs;        // pass buffers of one instance
  int chunk;       // instances per launch group
};

__host__ __device__ constexpr int first_radix_bits(int dtype) { return dtype == CM_C64 ? 14 : 13; }
__host__ __device__ constexpr int later_radix_bits(int dtype) { return dtype == CM_C64 ? 11 : 10; }
constexpr int LATER_MIN_BITS = 5;   // make_plan leaves later passes 5 (CM_C128) or 6 bits at least
// work items per workgroup after the first pass: 16, fewer where two workgroups could not share a
// CU (2^13 points of CM_C64, 2^12 of CM_C128 are 70 KB of LDS)
__host__ __device__ constexpr int log_cols(int dtype, int logr) {
  const int most = (dtype == CM_C64 ? 13 : 12) - logr;
  return most < 4 ? most : 4;
}

__host__ inline size_t al256f(size_t x) { return (x + 255) & ~(size_t)255; }

// Bytes a call must bring: a pass buffer of M points per instance of a group of 2^22 points,
// two where M takes more than two passes of 2^first and 2^(later-1) points, half of one more
// to gather from.
__host__ inline size_t fft_min_ws_bytes(int n, int dtype, bool gather, int batch) {
  const size_t es = dtype == CM_C64 ? 8 : 16;
  const size_t M = (size_t)1 << n;
  size_t ch = n < 22 ? (size_t)1 << (22 - n) : 1;
  if (ch > (size_t)MAX_CHUNK) ch = MAX_CHUNK;
  if ((size_t)batch < ch) ch = batch;
  size_t o = al256f(DENSE_PROB_BYTES * (size_t)batch);   // per-problem constants
  o += al256f(es * M * ch);
  if (n > first_radix_bits(dtype) + later_radix_bits(dtype) - 1) o += al256f(es * M * ch);
  if (gather) o += al256f(es / 2 * M * ch);
  return o;
}

// Passes. The first takes as much as leaves the others 6 bits (a radix-2 pass moves as many bytes as
// any other: the third pass of n = 26 was one of two bits and took 950 of 1370 us), up to 11 bits, and
// beyond them no more than bring the next pass down to 8 bits (CM_C64) or 9; the rest is split
// evenly. A larger first pass is a workgroup of up to 1024 threads with a CU to itself, few of them,
// and evaluates its share of G in 128 registers a thread (at 2^13 points of CM_C128 112 of them spill):
// where G fills the grid, that is most of the call. 16 grids, 300 strikes, as large a first pass as
// leaves 6 bits -> this rule (the full-length transform in brackets): Variance Gamma n = 20 CM_C128
// 1029 -> 529 us (603), n = 21 1963 -> 886 (1141), n = 22 3395 -> 1903 (2176), CM_C64 n = 20 233 -> 162
// (270), n = 21 421 -> 280 (382); where G is a sliver, Heston n = 20 CM_C128 178 -> 186 (350), n = 21
// CM_C64 231 -> 236 (358). n = 24 CM_C128 needs 13 and 10 bits for two passes and keeps 2^13.
// A grid of the largest single pass takes two while there are fewer grids than CUs: one Variance Gamma
// grid of n = 14 in CM_C128 takes 47 us (141 in one pass, 84 of the full-length transform in two),
// 1000 Black-Scholes grids 90 us in one and 250 in two.
// A group's instances are what fits the workspace.
__host__ inline FftPlan make_plan(int n, int dtype, bool gather, int batch, size_t ws_bytes) {
  FftPlan p;
  p.n = n;
  const int nb = n - 1, f = first_radix_bits(dtype), g = later_radix_bits(dtype);
  int b0 = nb;
  if (nb > f || (nb == f && batch < CUS)) {
    b0 = nb <= 18 ? (nb - 6 < 11 ? nb - 6 : 11) : nb - (dtype == CM_C64 ? 8 : 9);
    if (b0 > f) b0 = f;
  }
  p.logr[0] = b0;
  int rem = nb - b0;
  const int k = rem == 0 ? 0 : rem <= g ? 1 : (rem + g - 2) / (g - 1);
  p.npass = 1 + k;
  for (int i = 0; i < k; ++i) {
    const int b = (rem + (k - i) - 1) / (k - i);
    p.logr[1 + i] = b;
    rem -= b;
  }
  const size_t es = dtype == CM_C64 ? 8 : 16;
  // every pass but a last one that writes prices stores into a buffer; they alternate
  const int stores = p.npass - (gather ? 0 : 1);
  p.bufs = stores < 2 ? stores : 2;
  const size_t fixed = al256f(DENSE_PROB_BYTES * (size_t)batch), buf = es << nb;
  size_t ch = batch < MAX_CHUNK ? batch : MAX_CHUNK;
  if (p.bufs) {
    const size_t fit = (ws_bytes - fixed) / (buf * p.bufs);
    if (fit < ch) ch = fit;
    while (ch > 1 && fixed + (p.bufs - 1) * al256f(buf * ch) + buf * ch > ws_bytes) --ch;
  }
  p.chunk = (int)(ch < 1 ? 1 : ch);
  return p;
}

// one pad slot per 16 elements: stride-16 accesses of 8- and 16-byte elements spread over
// all banks
__host__ __device__ inline int pidx(int x) { return x + (x >> 4); }
__host__ __device__ inline int col_stride(int logL) { return pidx(1 << logL) + 1; }
__host__ inline size_t lds_bytes(int logL, int ncol, size_t es) { return es * (size_t)col_stride(logL) * ncol; }

// u <- w u for the constant twiddle w = exp(-2 pi i m / 16)
template <typename T, int m>
__device__ __forceinline__ T tw16(T u) {
  if constexpr (m == 0) return u;
  else if constexpr (m == 4) return fr<T>::mk(u.y, -u.x);    // -i u
  else {
    using R = typename fr<T>::R;
    const R c = (R)cos16(m), s = (R)cos16((m + 12) & 15);   // sin(2 pi m/16) = cos(2 pi (m-4)/16)
    // (c - i s)(x + i y) = (c x + s y) + i (c y - s x)
    T r;
    r.x = c * u.x + s * u.y;
    r.y = c * u.y - s * u.x;
    return r;
  }
}

template <typename T, int R, int S, int G, int Q>
__device__ __forceinline__ void bfly(T *u) {
  constexpr int m = Q * (8 / S);
  const T t = tw16<T, m>(u[G + Q + S]);
  u[G + Q + S] = fr<T>::sub(u[G + Q], t);
  u[G + Q] = fr<T>::add(u[G + Q], t);
}

template <typename T, int R, int S, int G, int Q>
__device__ __forceinline__ void bfly_q(T *u) {
  if constexpr (Q < S) {
    bfly<T, R, S, G, Q>(u);
    bfly_q<T, R, S, G, Q + 1>(u);
  }
}
template <typename T, int R, int S, int G>
__device__ __forceinline__ void bfly_g(T *u) {
  if constexpr (G < R) {
    bfly_q<T, R, S, G, 0>(u);
    bfly_g<T, R, S, G + 2 * S>(u);
  }
}
template <typename T, int R, int S>
__device__ __forceinline__ void bfly_s(T *u) {
  if constexpr (S < R) {
    bfly_g<T, R, S, 0>(u);
    bfly_s<T, R, 2 * S>(u);
  }
}

__host__ __device__ constexpr int brev_c(int i, int R) {
  int rb = 0;
  for (int b = 1; b < R; b <<= 1, i >>= 1) rb = (rb << 1) | (i & 1);
  return rb;
}

// In-register DFT of R points with the minus sign, R in {2, 4, 8, 16}.
template <typename T, int R>
__device__ __forceinline__ void dft_reg(T *v) {
  T u[R];
#pragma unroll
  for (int i = 0; i < R; ++i) u[brev_c(i, R)] = v[i];
  bfly_s<T, R, 1>(u);
#pragma unroll
  for (int i = 0; i < R; ++i) v[i] = u[i];
}

template <typename T> struct price_t;
template <> struct price_t<float2> { using type = float; };
template <> struct price_t<double2> { using type = double; };

// One Stockham stage of radix R over 2^logc columns of L = 2^logL points, current
// sub-transform length Ls. Butterfly g -> column col = g mod 2^logc (fastest, so that global
// loads and stores of neighbouring lanes touch neighbouring work items), i = g / 2^logc,
// k = i mod Ls: reads element i + r L/R, twiddles by exp(-2 pi i r k / (Ls R)), transforms,
// writes element (i - k) R + k + r Ls. Elements come from LDS (column stride Lp, padded
// indices) or, in the first stage, from src(col, i, L/R, v); they go to LDS or, in the last
// stage, to dst(col, (i - k) R + k, Ls, v). Needs L 2^logc <= pts_per_thread<T> NT.
template <typename T> constexpr int pts_per_thread = sizeof(T) == 8 ? 16 : 8;
// threads of a workgroup of 2^b points
template <typename T> constexpr int fft_threads(int b) {
  const int t = (1 << b) / pts_per_thread<T>;
  return t < 64 ? 64 : t > NT_MAX ? NT_MAX : t;
}
// of pass 1 with 2^b points: eight points a thread at most, for the evaluation of G; 2^8 points of
// CM_C64 a pair of inputs a thread (4000 Heston grids of n = 9 139 us, with two or three pairs 152; 119 with
// one wave per problem in k_fft_prepare as well)
template <typename T> constexpr int first_threads(int b) {
  if (sizeof(T) == 8 && b == 8) return 192;
  const int t = (1 << b) / 8;
  return t < 64 ? 64 : t > NT_MAX ? NT_MAX : t;
}
// Up to WIDE_GRIDS grids of 2^8 to 2^10 points in one pass are bound by the latency of the few
// evaluations in turn on each thread (16 values of the integrand at 2^9 points): their workgroups
// have a thread per value, as far as 1024 go, four of them to a pair of inputs.
constexpr int WIDE_B0 = 8, WIDE_B = 10, WIDE_GRIDS = 512;
constexpr int wide_threads(int b) {
  const int t = 2 * (1 << b) + 64;
  return t > NT_MAX ? NT_MAX : t;
}

// Twiddles t w^r, r < R, with w = exp(-2 pi i f) and t = exp(-2 pi i f0) (f, f0 turn fractions;
// HAS_T false: t = 1), in FP64 and rounded once at the end. The r-th power of a rounded w is off
// by r ulps, and the integrand's negative frequencies sit at the largest r, so the upper half goes
// down from w^R, which has a fraction of its own (powers in FP32 tripled the error of a Heston grid of
// n = 26). FP64 multiplies issue at the rate of FP32 ones. Error of all prices against FP64 (relative,
// 2-norm; geometric mean over 10 to 16 Heston grids within a factor e^pi of the spot, the full-length
// transform in brackets): n = 16 7.9e-7 (8.5e-7), n = 20 8.0e-7 (8.5e-7), n = 24 8.2e-7 (8.6e-7), n = 26
// 9.6e-7 (9.3e-7); one grid may be a quarter above or below the other transform's.
template <typename T, int R, bool HAS_T> __device__ __forceinline__ void twiddles(double f, double f0, T *tw) {
  double2 pw[R / 2 + 1];
  pw[0] = cmk(1.0, 0.0);
  pw[1] = fr<double2>::cis_neg(f);
#pragma unroll
  for (int r = 2; r <= R / 2; ++r) pw[r] = cmul(pw[r / 2], pw[r - r / 2]);
  const double2 t = HAS_T ? fr<double2>::cis_neg(f0) : cmk(1.0, 0.0);
  double2 tr = t;
  if constexpr (R > 2) tr = fr<double2>::cis_neg(f0 + R * f);   // t w^R
#pragma unroll
  for (int r = 0; r < R; ++r) {
    double2 x = pw[r <= R / 2 ? r : R - r];
    if (r > R / 2) x = cmul(tr, cconj(x));
    else if (HAS_T) x = cmul(t, x);
    tw[r] = fr<T>::mk(x.x, x.y);
  }
}

template <typename T, int R, int NT, bool FROM_LDS, bool TO_LDS, class Src, class Dst>
__device__ __forceinline__ void fft_stage(T *a, int logL, int logc, int Lp, int Ls, const Src &src, const Dst &dst) {
  constexpr int PT = pts_per_thread<T>;
  constexpr int NB = PT / R;  // butterflies per thread (at most)
  constexpr int LOGR = R == 16 ? 4 : R == 8 ? 3 : R == 4 ? 2 : 1;
  const int logLR = logL - LOGR;
  const int nbut = 1 << (logLR + logc);
  const int cmask = (1 << logc) - 1;
  T v[PT];
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    const int g = threadIdx.x + t * NT;
    if (g < nbut) {
      const int col = g & cmask, i = g >> logc;
      if constexpr (FROM_LDS) {
        const T *c = a + col * Lp;
#pragma unroll
        for (int r = 0; r < R; ++r) v[t * R + r] = c[pidx(i + (r << logLR))];
      } else {
        src.template load<R>(col, i, 1 << logLR, v + t * R);
      }
    }
  }
  if constexpr (FROM_LDS && TO_LDS) __syncthreads();
#pragma unroll
  for (int t = 0; t < NB; ++t) {
    const int g = threadIdx.x + t * NT;
    if (g < nbut) {
      const int col = g & cmask, i = g >> logc;
      const int k = i & (Ls - 1);
      if (k) {
        T tw[R];
        twiddles<T, R, false>((double)k * (1.0 / ((double)Ls * R)), 0.0, tw);
#pragma unroll
        for (int r = 1; r < R; ++r) v[t * R + r] = fr<T>::mul(v[t * R + r], tw[r]);
      }
      dft_reg<T, R>(v + t * R);
      const int base = (i - k) * R + k;
      if constexpr (TO_LDS) {
        T *c = a + col * Lp;
#pragma unroll
        for (int r = 0; r < R; ++r) c[pidx(base + r * Ls)] = v[t * R + r];
      } else {
        dst.template store<R>(col, base, Ls, v + t * R);
      }
    }
  }
  if constexpr (TO_LDS) __syncthreads();
}

// DFT of 2^logc columns of 2^LOGL points from stage 2^LOGLS on, inputs from src (or from LDS if
// GEN_LDS: the caller has already written them there), outputs to dst, LDS in between. Register
// radix 16 for CM_C64 and 8 for CM_C128; the remaining bits go last. The stage sequence is fixed
// at compile time.
template <typename T, int LOGL, int LOGLS, int NT, bool GEN_LDS, class Src, class Dst>
__device__ __forceinline__ void fft_block(T *a, int logc, int Lp, const Src &src, const Dst &dst) {
  constexpr int RB = pts_per_thread<T> >= 16 ? 4 : 3;
  constexpr int rem = LOGL - LOGLS;
  if constexpr (rem > 0) {
    constexpr int b = rem >= RB ? RB : rem;
    constexpr bool last = b == rem;
    fft_stage<T, (1 << b), NT, GEN_LDS, !last>(a, LOGL, logc, Lp, 1 << LOGLS, src, dst);
    fft_block<T, LOGL, LOGLS + b, NT, true>(a, logc, Lp, src, dst);
  }
}

}  // namespace

// Per-problem constants of the integrand and readout.
struct DenseConst {
  double eta, v0;
  int64_t jmid;            // index of v = 0: 2^(n-1) for the symmetric rule, else 0
  double th_hi, th_lo;     // theta / (2 pi) as double-double, theta = eta (m_f - k0)
  double2 g0;              // exp(i v0 (m_f - k0)): the integrand's and the read-out's constant phases
  double k0, nalog2e, lsf; // log2 of the readout scale e^{-alpha k_u} / (s pi) is nalog2e k_u + lsf
  double dz, zorg;         // its step per unit of u and its value at u = us (single-precision outputs)
  int64_t us;              // k_u = k0 + lambda (u - us): the default grid is centred on ln S0
  StrikeStep step;         // 2 pi / eta
  int n;
  int simpson;
};

// Everything a dense FFT workgroup needs about its problem, computed once per problem.
template <typename T> struct DenseProb {
  DenseConst c;
  CfModel<typename fr<T>::R> m;
  int64_t jlo, jhi;        // x_j may be non-zero only for jlo <= j < jhi
  int64_t side;            // G_j may be non-zero only for j < side and j > N - side
  int32_t bad;             // the problem failed its checks: prices are NaN
};
static_assert(sizeof(DenseProb<double2>) <= DENSE_PROB_BYTES, "DenseProb too large");
static_assert(sizeof(DenseProb<float2>) <= DENSE_PROB_BYTES, "DenseProb too large");

__device__ inline DenseConst dense_const(const cm_problem &pr) {
  DenseConst c;
  const int n = pr.n;
  c.eta = pr.eta;
  c.simpson = pr.quad == CM_QUAD_SIMPSON1;
  c.v0 = c.simpson ? 0.0 : -ldexp(pr.eta, n - 1);
  c.jmid = c.simpson ? 0 : ((int64_t)1 << (n - 1));
  const double rq = (pr.r - pr.q) * pr.T;
  double p, e;
  if (k0_is_default(pr)) {
    two_prod(pr.eta, rq, p, e);
    // theta/(2 pi) = eta rq / (2 pi) + 1/2
    double ch = p * CM_INV2PI_HI;
    double cl = fma(p, CM_INV2PI_HI, -ch) + p * CM_INV2PI_LO + e * CM_INV2PI_HI;
    // (ch + 0.5) may round; keep its rounding error in th_lo
    double s, err;
    two_sum(ch, 0.5, s, err);
    c.th_hi = s; c.th_lo = cl + err;
  } else {
    drift_angle(pr.eta, log(pr.S0), pr.k0, rq, p, e);
    c.th_hi = p * CM_INV2PI_HI;
    c.th_lo = fma(p, CM_INV2PI_HI, -c.th_hi) + p * CM_INV2PI_LO + e * CM_INV2PI_HI;
  }
  if (c.simpson) c.g0 = cmk(1.0, 0.0);
  else {
    double f = prod_cycles_frac(c.v0, log(pr.S0), 0) + prod_cycles_frac(c.v0, rq, 0);
    c.g0 = turn(f - floor(f));
  }
  // the default k0 = ln S0 - pi/eta is ln S0 - lambda M/2 exactly: strikes from ln S0 and an
  // exact integer offset
  const double k0 = k0_is_default(pr) ? log(pr.S0) : pr.k0;
  c.us = k0_is_default(pr) ? ((int64_t)1 << (n - 1)) : 0;
  const double sfac = c.simpson ? 1.0 / M_PI : 0.5 / M_PI;
  c.k0 = k0;
  c.n = n;
  c.nalog2e = -pr.alpha * M_LOG2E;
  c.dz = c.nalog2e * (2.0 * M_PI / (ldexp(1.0, n) * pr.eta));
  c.lsf = log2(sfac);
  c.zorg = fma(c.nalog2e, k0, c.lsf);
  c.step = strike_step(pr.eta);
  if (!c.simpson) {
    // -v0 k0 = eta 2^(n-1) k0; with the default k0 = ln S0 - pi/eta the pi part is a whole
    // number of turns for n >= 2
    double f;
    if (k0_is_default(pr)) {
      f = prod_cycles_frac(pr.eta, log(pr.S0), n - 1);
      if (n == 1) { f += 0.5; f -= floor(f); }
    } else {
      f = prod_cycles_frac(pr.eta, pr.k0, n - 1);
    }
    c.g0 = cmul(c.g0, turn(f));   // exp(-i v0 k0)
  }
  return c;
}

// z_j = ro x_{(j + jmid) mod M} (zero outside the support): the characteristic function in the
// storage precision, its phase and weight in FP64
template <typename T>
__device__ __forceinline__ double2 z_at(const DenseProb<T> &d, int64_t i) {
  using R = typename fr<T>::R;
  const DenseConst &c = d.c;
  const int64_t j = (i + c.jmid) & (((int64_t)1 << c.n) - 1);
  if (j < d.jlo || j >= d.jhi) return cmk(0.0, 0.0);
  // v_j = v0 + j eta formed from the exact offset j - jmid: adding v0 to j eta would cancel
  // to an absolute error of |v0| ulp near v = 0 on large symmetric grids
  const double v = (double)(j - c.jmid) * c.eta;
  const cx<R> h = h_centered<R>(d.m, (R)v);
  // exp(i j theta): fraction of j * (th_hi + th_lo)
  double p, e;
  two_prod((double)j, c.th_hi, p, e);
  double f = frac2(p, e + (double)j * c.th_lo);
  double w;
  if (c.simpson) w = c.eta / 3.0 * ((j & 1) ? 4.0 : (j == 0 ? 1.0 : 2.0));
  else w = c.eta;
  const double2 ph = fr<double2>::cis_neg(-f);   // exp(+2 pi i f)
  return cmul(cmul(cmk((double)h.x, (double)h.y), ph), cscale(c.g0, w));
}

// G_j, 0 <= j <= h = 2^(n-1) (see the head of the file), rounded once, and G_{h-j}, which takes
// the same four values of z. Outside the support nothing is evaluated.
template <typename T>
__device__ __forceinline__ T g_pair(const DenseProb<T> &d, int64_t j, T *other) {
  const int64_t h = (int64_t)1 << (d.c.n - 1), M = 2 * h;
  if (j >= d.side && j <= h - d.side) {
    if (other) *other = fr<T>::mk(0.0, 0.0);
    return fr<T>::mk(0.0, 0.0);
  }
  const double2 a = cadd(z_at<T>(d, j), cconj(z_at<T>(d, M - j)));
  const double2 b = cadd(z_at<T>(d, j + h), cconj(z_at<T>(d, h - j)));
  // w^j from the smaller of j and h - j (w^{h-m} = -conj w^m): near h/M = 1/2 turn a rounded
  // fraction would lose the low bits of m
  const bool far = 2 * j > h;
  double2 w = fr<double2>::cis_neg(ldexp((double)(far ? h - j : j), -d.c.n));
  if (far) w.x = -w.x;
  const double2 e = cmul(cmk(-w.y, w.x), csub(a, b)), s = cadd(a, b);
  // G_{h-j}: conj(b) and conj(a) for a and b, and i w^{h-j} = -i conj(w^j) = conj(i w^j)
  if (other) *other = fr<T>::mk(0.5 * (s.x - e.x), 0.5 * (e.y - s.y));
  return fr<T>::mk(0.5 * (s.x + e.x), 0.5 * (s.y + e.y));
}
// The same on four neighbouring lanes, one value of z each (q = lane mod 4): lane 0 returns G_j, lane 1
// G_{h-j}. Every lane of the wave takes part, with the j of its four.
template <typename T>
__device__ __forceinline__ T g_quad(const DenseProb<T> &d, int64_t j, int q) {
  const int64_t h = (int64_t)1 << (d.c.n - 1), M = 2 * h;
  const bool out = j >= d.side && j <= h - d.side;
  double2 z = cmk(0.0, 0.0);
  if (!out) z = z_at<T>(d, q == 0 ? j : q == 1 ? M - j : q == 2 ? j + h : h - j);
  if (q & 1) z = cconj(z);
  const double2 o = cmk(__shfl_xor(z.x, 1, 64), __shfl_xor(z.y, 1, 64));
  const double2 ab = cadd(z, o);   // a on lanes 0 and 1, b on 2 and 3
  const double2 c = cmk(__shfl_xor(ab.x, 2, 64), __shfl_xor(ab.y, 2, 64));
  const double2 a = q < 2 ? ab : c, b = q < 2 ? c : ab;
  const bool far = 2 * j > h;
  double2 w = fr<double2>::cis_neg(ldexp((double)(far ? h - j : j), -d.c.n));
  if (far) w.x = -w.x;
  const double2 e = cmul(cmk(-w.y, w.x), csub(a, b)), s = cadd(a, b);
  if (out) return fr<T>::mk(0.0, 0.0);
  return q & 1 ? fr<T>::mk(0.5 * (s.x - e.x), 0.5 * (e.y - s.y)) : fr<T>::mk(0.5 * (s.x + e.x), 0.5 * (s.y + e.y));
}
template <typename T> __device__ __forceinline__ T g_at(const DenseProb<T> &d, int64_t j) {
  return g_pair<T>(d, j, nullptr);
}

// Prices C(k_u) = e^{-alpha k_u}/(s pi) f_u: the scale is 2^z with the exponent kept in FP64.
// z, the log2 of the scale, is passed in: formed from the accurate log-strike (strike_log) in FP64
// and as zorg + dz (u - us) in FP32.
__device__ __forceinline__ float price_at(double z, float f) {
  const double zi = floor(z);
  return ldexpf(f * exp2f((float)(z - zi)), (int)zi);
}
__device__ __forceinline__ double price_at(double z, double f) { return exp2(z) * f; }
template <typename T> __device__ __forceinline__ double scale_log2(const DenseConst &c, int64_t u) {
  if constexpr (sizeof(T) == sizeof(double2))
    return fma(c.nalog2e, strike_log(c.k0, c.step, c.n, (double)(u - c.us)), c.lsf);
  else
    return fma(c.dz, (double)(u - c.us), c.zorg);
}

// Sources and sinks of a pass. Work item of column col is item0 + col; a pass with radix R
// and stride plen reads x[item + e N/R] (element e of the item's DFT) and writes
// y[(item - k) R + k + q plen] (output q), k = item mod plen.
struct NoSrc {
  template <int R, typename T> __device__ __forceinline__ void load(int, int, int, T *) const {}
};

template <typename T> struct BufSrc {     // later passes: read the previous pass, apply its twiddle
  const T *src;
  int64_t item0, T_items, plen;
  int twl_bits;                          // log2(R plen)
  template <int R> __device__ __forceinline__ void load(int col, int e0, int de, T *v) const {
    const int64_t item = item0 + col;
    const int64_t k = item & (plen - 1);
    const int64_t mask = ((int64_t)1 << twl_bits) - 1;
    T tw[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = src[item + (int64_t)(e0 + r * de) * T_items];
    twiddles<T, R, true>(ldexp((double)(((int64_t)de * k) & mask), -twl_bits),
                         ldexp((double)(((int64_t)e0 * k) & mask), -twl_bits), tw);
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = fr<T>::mul(v[r], tw[r]);
  }
};

template <typename T> struct BufDst {     // intermediate passes
  T *dst;
  int64_t item0, plen;
  int logR;
  template <int R> __device__ __forceinline__ void store(int col, int q0, int dq, const T *v) const {
    const int64_t item = item0 + col;
    const int64_t k = item & (plen - 1);
    T *o = dst + ((item - k) << logR) + k;
#pragma unroll
    for (int r = 0; r < R; ++r) o[(int64_t)(q0 + r * dq) * plen] = v[r];
  }
};

template <typename T> struct PriceDst {   // last pass: readout scalars, two prices per point
  typename price_t<T>::type *prices;
  const DenseConst *c;
  int64_t item0, plen;
  int logR, bad;
  template <int R> __device__ __forceinline__ void store(int col, int q0, int dq, const T *v) const {
    const int64_t item = item0 + col;
    const int64_t k = item & (plen - 1);
    const int64_t v0 = ((item - k) << logR) + k + (int64_t)q0 * plen, dv = (int64_t)dq * plen;
    if constexpr (std::is_same<T, double2>::value) {
      // every output from its accurate log-strike: the outputs of one call lie up to M apart,
      // where steps of a rounded lambda would be off by the whole strike range times ulp(1)
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int64_t u = 2 * (v0 + r * dv);
        T pr = fr<T>::mk2(price_at(scale_log2<T>(*c, u), v[r].x), price_at(scale_log2<T>(*c, u + 1), v[r].y));
        if (bad) pr = fr<T>::mk2(NAN, NAN);
        prices[u] = pr.x;
        prices[u + 1] = pr.y;
      }
    } else {
      // single-precision prices: the scale's exponent as z_org + dz (u - us) in FP64, one FMA per
      // call and steps for its outputs (the FP64 error of a rounded lambda, at most the strike
      // range times ulp(1), stays far below the FP32 rounding of the price)
      const double z0 = scale_log2<T>(*c, 2 * v0), dz = c->dz * (double)(2 * dv);
#pragma unroll
      for (int r = 0; r < R; ++r) {
        const int64_t u = 2 * (v0 + r * dv);
        const double z = fma((double)r, dz, z0);
        T pr = fr<T>::mk2(price_at(z, v[r].x), price_at(z + c->dz, v[r].y));
        if (bad) pr = fr<T>::mk2(NAN, NAN);
        prices[u] = pr.x;
        prices[u + 1] = pr.y;
      }
    }
  }
};

// Per problem: constants, and the numerical support of x. W wavefronts per problem evaluate |h| at
// v = +-2^{q/4 - 4}, q < 256, find the first q from which five consecutive points lie below
// thr |h(0)|, and keep indices with |v| < 2 v_q. A problem that fails its checks keeps the whole
// range and is marked bad. Four waves, where one takes their quarters in turn (24 us of a small call);
// one from PREP_ONE problems on, which fill the chip either way (4000 grids of n = 4: 1.18 times as fast).
template <typename T, int W>
__global__ __launch_bounds__(64 * W) void k_fft_prepare(const cm_problem *__restrict__ prob, int batch, int n, double thr,
                                                     DenseProb<T> *__restrict__ out, int32_t *__restrict__ status) {
  __shared__ uint64_t below[4];
  const int b = blockIdx.x;
  if (b >= batch) return;
  const cm_problem pr = prob[b];
  int code = check_problem(pr);
  if (code == CM_OK && pr.n != n) code = CM_E_INVALID;
  const int64_t M = (int64_t)1 << n;
  int64_t jlo = 0, jhi = M;
  if (code == CM_OK) {   // the same for all threads of the problem
    const CfModel<double> m = make_model<double>(pr);
    const cx<double> h0 = h_centered<double>(m, 0.0);
    const double lim = thr * sqrt(h0.x * h0.x + h0.y * h0.y);
    auto scan = [&](int w, int q) {
      const double v = exp2(0.25 * q - 4.0);
      const cx<double> hp = h_centered<double>(m, v), hm = h_centered<double>(m, -v);
      const double a = fmax(sqrt(hp.x * hp.x + hp.y * hp.y), sqrt(hm.x * hm.x + hm.y * hm.y));
      const uint64_t mask = __ballot(a < lim);
      if ((threadIdx.x & 63) == 0) below[w] = mask;
    };
    if constexpr (W == 4) {
      scan(threadIdx.x >> 6, threadIdx.x);
    } else {
#pragma unroll
      for (int w = 0; w < 4; ++w) scan(w, 64 * w + (int)(threadIdx.x & 63));
    }
    __syncthreads();
    // the first q whose five points from q on all lie below: shifted masks, word by word (q + 4 <= 255)
    int qcut = -1;
#pragma unroll
    for (int w = 3; w >= 0; --w) {
      const uint64_t lo = below[w], up = w < 3 ? below[w + 1] : 0;
      uint64_t all = lo;
#pragma unroll
      for (int t = 1; t < 5; ++t) all &= (lo >> t) | (up << (64 - t));
      if (all) qcut = 64 * w + (int)__builtin_ctzll(all);
    }
    if (qcut >= 0) {
      const double half = 2.0 * exp2(0.25 * qcut - 4.0) / pr.eta;
      if (pr.quad == CM_QUAD_SIMPSON1) {
        jhi = (int64_t)fmin((double)M, ceil(half) + 1.0);
      } else {
        const double c0 = (double)(M / 2);
        jlo = (int64_t)fmax(0.0, floor(c0 - half) - 1.0);
        jhi = (int64_t)fmin((double)M, ceil(c0 + half) + 1.0);
      }
    }
  }
  if (threadIdx.x == 0) {
    DenseProb<T> d;
    d.c = dense_const(pr);
    d.m = make_model<typename fr<T>::R>(pr);
    d.jlo = jlo;
    d.jhi = jhi;
    // G_j takes x_j at |v| = j eta and (h - j) eta; both sides vanish from `side` on
    const int64_t h = M / 2;
    int64_t side = pr.quad == CM_QUAD_SIMPSON1 ? jhi : (h - jlo > jhi - h ? h - jlo : jhi - h) + 1;
    d.side = side < h ? side : h + 1;
    d.bad = code != CM_OK;
    out[b] = d;
    if (status) status[b] = code;
  }
}

// Pass 1 from stage 2^SB on. Of the L = 2^LOGR inputs of a work item only the first and last
// E = ceil(side / items) may be non-zero. With P = 2^SB and E <= L / P, the P-point DFTs that the
// first SB bits' stages form have two non-zero inputs at most, their first and last, so the array
// after those stages is y[P i + q] = a_i + b_i exp(2 pi i q / P), i < L / P, with a_i, b_i the
// inputs i and L - L / P + i. a and b are evaluated once into LDS (behind the FFT buffer) and
// the first stage that is run reads them there.
template <typename T> struct PrunedSrc {
  const T *ab;          // a, then b
  int logP, logL;
  template <int R> __device__ __forceinline__ void load(int, int i, int, T *v) const {
    const int n = 1 << (logL - logP), q = i & ((1 << logP) - 1), i0 = i >> logP;
    const double2 t = fr<double2>::cis_neg(-ldexp((double)q, -logP));
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const int e = i0 + r * (n / R);
      const T a = ab[e], b = ab[n + e];
      const double2 y = cadd(cmk(a.x, a.y), cmul(cmk(b.x, b.y), t));
      v[r] = fr<T>::mk(y.x, y.y);
    }
  }
};

// inputs of either side that a pruned start keeps in LDS, at most
template <typename T> constexpr int PRUNE_MAX = sizeof(T) == 8 ? 1024 : 512;

template <typename T, int LOGR, int REM, int NT, class Dst>
__device__ __forceinline__ void first_pass_pruned(T *a, const DenseProb<T> &d, int64_t item, int64_t T_items,
                                                  const Dst &dst) {
  constexpr int n = 1 << REM, L = 1 << LOGR;
  static_assert(n <= PRUNE_MAX<T>, "LDS behind the FFT buffer");
  T *ab = a + pidx(L) + 1;
  if (T_items == 1) {   // input L - e is input e's partner
    for (int e = threadIdx.x; e <= n; e += NT) {
      T o;
      const T g = g_pair<T>(d, e, &o);
      if (e < n) ab[e] = g;
      if (e > 0) ab[2 * n - e] = o;
    }
  } else {
    for (int e = threadIdx.x; e < 2 * n; e += NT)
      ab[e] = g_at<T>(d, item + (int64_t)(e < n ? e : L - 2 * n + e) * T_items);
  }
  __syncthreads();
  fft_block<T, LOGR, LOGR - REM, NT, false>(a, 0, 0, PrunedSrc<T>{ab, LOGR - REM, LOGR}, dst);
}

// Chooses the latest start that the problem's support allows, counted in remaining bits: one, two
// or three register stages.
template <typename T, int LOGR, bool WIDE, class Dst>
__device__ __forceinline__ void first_pass(T *a, const DenseProb<T> &d, int64_t item, int64_t T_items, const Dst &dst) {
  constexpr int RB = pts_per_thread<T> >= 16 ? 4 : 3, NT = WIDE ? wide_threads(LOGR) : first_threads<T>(LOGR);
  if constexpr (LOGR == 0) {
    if (threadIdx.x == 0) {
      const T g = g_at<T>(d, 0);
      dst.template store<1>(0, 0, 1, &g);
    }
    return;
  } else {
    const int64_t E = (d.side + T_items - 1) / T_items;   // more than L / 2 when nothing is known
    constexpr int R1 = RB, R2 = 2 * RB - 2, R3 = 2 * RB, R4 = RB == 4 ? 10 : 9;
    if constexpr (LOGR > R1)
      if (E <= (1 << R1)) return first_pass_pruned<T, LOGR, R1, NT>(a, d, item, T_items, dst);
    if constexpr (LOGR >= 12)
      if (E <= (1 << R2)) return first_pass_pruned<T, LOGR, R2, NT>(a, d, item, T_items, dst);
    if constexpr (LOGR > R3)
      if (E <= (1 << R3)) return first_pass_pruned<T, LOGR, R3, NT>(a, d, item, T_items, dst);
    if constexpr (LOGR > R4)
      if (E <= (1 << R4)) return first_pass_pruned<T, LOGR, R4, NT>(a, d, item, T_items, dst);
    if constexpr (WIDE) {   // one pass
      constexpr int L = 1 << LOGR;
      const int q = threadIdx.x & 3;
      for (int e0 = 0; e0 <= L / 2; e0 += NT / 4) {
        const int e = e0 + (int)(threadIdx.x >> 2);
        const T v = g_quad<T>(d, e <= L / 2 ? e : 0, q);
        if (q == 0 && e <= L / 2) a[pidx(e)] = v;
        if (q == 1 && e > 0 && e < L / 2) a[pidx(L - e)] = v;
      }
    } else if (T_items == 1) {
      constexpr int L = 1 << LOGR;
      for (int e = threadIdx.x; e <= L / 2; e += NT) {
        T o;
        a[pidx(e)] = g_pair<T>(d, e, &o);
        if (e > 0 && e < L / 2) a[pidx(L - e)] = o;
      }
    } else {
      for (int e = threadIdx.x; e < (1 << LOGR); e += NT) a[pidx(e)] = g_at<T>(d, item + (int64_t)e * T_items);
    }
    __syncthreads();
    fft_block<T, LOGR, 0, NT, true>(a, 0, 0, NoSrc{}, dst);
  }
}

// LDS bytes of pass 1: the FFT buffer and the inputs of a pruned start
template <typename T> __host__ inline size_t first_lds_bytes(int logr) {
  const size_t keep = logr > 0 ? (size_t)1 << (logr - 1) : 0;
  return sizeof(T) * ((size_t)col_stride(logr) + 2 * (keep < PRUNE_MAX<T> ? keep : PRUNE_MAX<T>));
}

// Either sink, chosen per launch (one instance of the transform's code serves both).
template <typename T> struct PassDst {
  BufDst<T> buf;
  PriceDst<T> price;
  template <int R> __device__ __forceinline__ void store(int col, int q0, int dq, const T *v) const {
    if (price.prices) price.template store<R>(col, q0, dq, v);
    else buf.template store<R>(col, q0, dq, v);
  }
};

// Pass 1: one work item (blockIdx.x) per workgroup; G is generated (only lanes inside the support
// evaluate the characteristic function), then transformed. Prices go out at once when this is
// the only pass and no strikes are chosen.
template <typename T, int LOGR, bool WIDE>
__global__ __launch_bounds__(WIDE ? wide_threads(LOGR) : first_threads<T>(LOGR)) void k_fft_first(
    const DenseProb<T> *__restrict__ dprob, int inst0, int n, T *__restrict__ out,
    typename price_t<T>::type *__restrict__ prices) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  T *a = (T *)lds_raw;
  const int64_t N = (int64_t)1 << (n - 1);
  const DenseProb<T> *d = dprob + inst0 + blockIdx.y;
  const int64_t item = blockIdx.x, T_items = N >> LOGR;
  const PassDst<T> dst{{out + (int64_t)blockIdx.y * N, item, 1, LOGR},
                       {prices ? prices + (int64_t)blockIdx.y * 2 * N : nullptr, &d->c, item, 1, LOGR, d->bad}};
  first_pass<T, LOGR, WIDE>(a, *d, item, T_items, dst);
}

// Later passes: 16, 8 or 4 consecutive work items per workgroup, loaded straight into the
// first stage's registers.
template <typename T, int LOGR>
__global__ __launch_bounds__(fft_threads<T>(LOGR + log_cols(sizeof(T) == 8 ? CM_C64 : CM_C128, LOGR))) void k_fft_next(
    const DenseProb<T> *__restrict__ dprob, int inst0, int n, int64_t plen, const T *__restrict__ in,
    T *__restrict__ out, typename price_t<T>::type *__restrict__ prices) {
  extern __shared__ __align__(16) unsigned char lds_raw[];
  T *a = (T *)lds_raw;
  constexpr int LC = log_cols(sizeof(T) == 8 ? CM_C64 : CM_C128, LOGR), NT = fft_threads<T>(LOGR + LC);
  const int64_t N = (int64_t)1 << (n - 1);
  // Workgroups go to the eight XCDs in turn: numbered so that each XCD takes neighbouring items,
  // whose loads and stores share cache lines when a workgroup covers less than a line
  const unsigned nb = gridDim.x, blk = nb % 8 == 0 ? blockIdx.x % 8 * (nb / 8) + blockIdx.x / 8 : blockIdx.x;
  const int64_t item0 = (int64_t)blk << LC;
  const int twl_bits = LOGR + (int)__builtin_ctzll(plen);
  BufSrc<T> src{in + (int64_t)blockIdx.y * N, item0, N >> LOGR, plen, twl_bits};
  const int Lp = col_stride(LOGR);
  const DenseProb<T> *d = dprob + inst0 + blockIdx.y;
  const PassDst<T> dst{{out + (int64_t)blockIdx.y * N, item0, plen, LOGR},
                       {prices ? prices + (int64_t)blockIdx.y * 2 * N : nullptr, &d->c, item0, plen, LOGR, d->bad}};
  fft_block<T, LOGR, 0, NT, false>(a, LC, Lp, src, dst);
}

// Host-side tables of the instantiations, indexed by radix bits.
template <typename T, int... B>
static constexpr std::array<decltype(&k_fft_first<T, 1, false>), sizeof...(B)> first_table(std::integer_sequence<int, B...>) {
  return {&k_fft_first<T, B, false>...};
}
template <typename T, int... B>
static constexpr std::array<decltype(&k_fft_first<T, WIDE_B, true>), sizeof...(B)> wide_table(std::integer_sequence<int, B...>) {
  return {&k_fft_first<T, WIDE_B0 + B, true>...};
}
template <typename T, int... B>
static constexpr std::array<decltype(&k_fft_next<T, LATER_MIN_BITS>), sizeof...(B)> next_table(std::integer_sequence<int, B...>) {
  return {&k_fft_next<T, LATER_MIN_BITS + B>...};
}

// Prices of the chosen strikes from the transform: price u = 2 v + c is component c of g_v.
template <typename T>
__global__ void k_gather(const DenseProb<T> *__restrict__ dprob, const T *__restrict__ g, int n,
                         const int64_t *__restrict__ idx, int nk, int inst0, int cnt,
                         typename price_t<T>::type *__restrict__ out, int32_t *__restrict__ status) {
  const int64_t M = (int64_t)1 << n;
  const int64_t total = (int64_t)cnt * nk;
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
    const int b = (int)(e / nk), s = (int)(e % nk);
    const int64_t u = idx[(int64_t)(inst0 + b) * nk + s];
    typename price_t<T>::type v = NAN;
    if (u < 0 || u >= M) {
      set_status(status, inst0 + b, CM_E_INVALID);
    } else {
      const DenseProb<T> &d = dprob[inst0 + b];
      const T gv = g[(int64_t)b * (M / 2) + (u >> 1)];
      if (!d.bad) v = price_at(scale_log2<T>(d.c, u), (u & 1) ? gv.y : gv.x);
    }
    out[(int64_t)(inst0 + b) * nk + s] = v;
  }
}

extern "C" size_t cm_fft_ws_bytes(int batch, int n, int dtype, int gather) {
  if (n < 1 || n > 30 || batch < 1) return 0;
  return fft_min_ws_bytes(n, dtype, gather != 0, batch);
}

template <typename T>
static cm_status fft_run(const cm_problem *prob, int batch, int n, const int64_t *strike_idx, int nk, void *prices,
                         int32_t *status, void *ws, size_t ws_bytes, hipStream_t s) {
  using P = typename price_t<T>::type;
  constexpr int dtype = sizeof(T) == 8 ? CM_C64 : CM_C128;
  const bool gather = strike_idx != nullptr;
  const FftPlan p = make_plan(n, dtype, gather, batch, ws_bytes);
  const int64_t M = (int64_t)1 << n, N = M / 2;
  char *w = (char *)ws;
  DenseProb<T> *dp = (DenseProb<T> *)w;
  w += al256f(DENSE_PROB_BYTES * (size_t)batch);
  T *buf[2] = {(T *)w, nullptr};
  if (p.bufs > 1) buf[1] = (T *)(w + al256f(sizeof(T) * (size_t)N * p.chunk));
  // cut-off of |psi| relative to |psi(0)|, far below the storage precision
  const double thr = dtype == CM_C64 ? 1e-16 : 1e-32;
  if (batch < PREP_ONE)
    hipLaunchKernelGGL((k_fft_prepare<T, 4>), dim3(batch), dim3(256), 0, s, prob, batch, n, thr, dp, status);
  else
    hipLaunchKernelGGL((k_fft_prepare<T, 1>), dim3(batch), dim3(64), 0, s, prob, batch, n, thr, dp, status);
  CM_LAUNCH_CHECK();
  constexpr int FB = first_radix_bits(dtype), NB = later_radix_bits(dtype);
  static constexpr auto kfirst = first_table<T>(std::make_integer_sequence<int, FB + 1>{});
  static constexpr auto kwide = wide_table<T>(std::make_integer_sequence<int, WIDE_B - WIDE_B0 + 1>{});
  static constexpr auto knext = next_table<T>(std::make_integer_sequence<int, NB - LATER_MIN_BITS + 1>{});
  const int lr0 = p.logr[0];
  if (lr0 < 0 || lr0 > FB) return CM_E_UNSUPPORTED;
  for (int ps = 1; ps < p.npass; ++ps)
    if (p.logr[ps] < LATER_MIN_BITS || p.logr[ps] > NB) return CM_E_UNSUPPORTED;
  const size_t lds0 = first_lds_bytes<T>(lr0);
  const bool wide = p.npass == 1 && lr0 >= WIDE_B0 && lr0 <= WIDE_B && batch <= WIDE_GRIDS;
  const auto first = wide ? kwide[lr0 - WIDE_B0] : kfirst[lr0];
  const int nt0 = wide ? wide_threads(lr0) : first_threads<T>(lr0);
  CM_HIP_CHECK(cm_allow_lds(first, lds0));
  for (int ps = 1; ps < p.npass; ++ps)
    CM_HIP_CHECK(cm_allow_lds(knext[p.logr[ps] - LATER_MIN_BITS], lds_bytes(p.logr[ps], 1 << log_cols(dtype, p.logr[ps]), sizeof(T))));
  for (int inst0 = 0; inst0 < batch; inst0 += p.chunk) {
    const int cnt = (batch - inst0) < p.chunk ? (batch - inst0) : p.chunk;
    P *dstp = (P *)prices + (int64_t)inst0 * M;   // where the last pass writes prices
    hipLaunchKernelGGL(first, dim3((unsigned)(N >> lr0), cnt), dim3(nt0), lds0, s, dp, inst0, n,
                       buf[0], p.npass == 1 && !gather ? dstp : (P *)nullptr);
    CM_LAUNCH_CHECK();
    int64_t plen = (int64_t)1 << lr0;
    int cur = 0;
    for (int ps = 1; ps < p.npass; ++ps) {
      const int lr = p.logr[ps], lc = log_cols(dtype, lr);
      const bool to_prices = ps == p.npass - 1 && !gather;
      hipLaunchKernelGGL(knext[lr - LATER_MIN_BITS], dim3((unsigned)((N >> lr) >> lc), cnt), dim3(fft_threads<T>(lr + lc)),
                         lds_bytes(lr, 1 << lc, sizeof(T)), s, dp, inst0, n, plen, buf[cur], buf[cur ^ 1],
                         to_prices ? dstp : (P *)nullptr);
      CM_LAUNCH_CHECK();
      cur ^= 1;
      plen <<= lr;
    }
    if (gather) {
      const int64_t gb = ((int64_t)cnt * nk + 255) / 256;
      hipLaunchKernelGGL(k_gather<T>, dim3((unsigned)(gb < 4096 ? gb : 4096)), dim3(256), 0, s, dp, buf[cur], n, strike_idx, nk, inst0, cnt,
                         (P *)prices, status);
      CM_LAUNCH_CHECK();
    }
  }
  return CM_OK;
}

extern "C" cm_status cm_fft_price(const cm_problem *prob, int batch, int n, int dtype, const int64_t *strike_idx,
                                  int nk, void *prices, int32_t *status, void *ws, size_t ws_bytes, void *stream) {
  if (!prob || !prices || batch < 0 || n < 1) return CM_E_INVALID;
  if (n > 30) return CM_E_UNSUPPORTED;
  if (dtype != CM_C64 && dtype != CM_C128) return CM_E_INVALID;
  if (strike_idx && nk < 1) return CM_E_INVALID;
  if (batch == 0) return CM_OK;
  if (batch > 65535) return CM_E_UNSUPPORTED;
  const size_t need = cm_fft_ws_bytes(batch, n, dtype, strike_idx != nullptr);
  if (!ws || ws_bytes < need) return CM_E_INVALID;
  hipStream_t s = (hipStream_t)stream;
  if (dtype == CM_C64) return fft_run<float2>(prob, batch, n, strike_idx, nk, prices, status, ws, ws_bytes, s);
  return fft_run<double2>(prob, batch, n, strike_idx, nk, prices, status, ws, ws_bytes, s);
}
