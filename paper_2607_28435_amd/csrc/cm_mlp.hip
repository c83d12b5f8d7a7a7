// Pricing surrogate network (a project addition; the paper has no learned component):
// forward, backward, MSE, Adam and the gate. Layer equations and the parameter layout are
// in cm.h.
//
// The 256 x 256 layers are GEMMs on BF16 MFMA (v_mfma_f32_32x32x16_bf16) with FP32
// accumulation. An operand that comes from FP32 activations is split into hi + lo BF16 parts
// (two MFMAs per step), so its rounding error is ~2^-16 instead of 2^-8. Operand lane layout
// (32x32x16): lane l holds A[l % 32][8 (l / 32) + i] and B[8 (l / 32) + i][l % 32], i < 8;
// accumulator v of lane l is C[8 (v / 4) + 4 (l / 32) + v % 4][l % 32].
//   k_mlp_fused  inference over many queries: five layers per tile of 64, two tiles in flight
//   k_mlp_tile   five layers per tile of 32: small inference batches, and the training forward
//                (which also stores the pre-activations)
//   k_mlp_bwd    the backward-data chain per tile of 32, with the first layer's gradients
//   k_wgrad      the other layers' gradients: sums over the batch of delta^T silu(Z)
#include "cm_internal.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int NW = CM_MLP_WIDTH;
constexpr int NIN = CM_MLP_NIN;
constexpr int OFF_W1 = 0, OFF_B1 = 1792, OFF_W5 = 199424, OFF_B5 = 199680;
__host__ __device__ constexpr int off_w(int l) { return l == 2 ? 2048 : l == 3 ? 67840 : 133632; }
__host__ __device__ constexpr int off_b(int l) { return l == 2 ? 67584 : l == 3 ? 133376 : 199168; }
static_assert(OFF_B5 + 1 == CM_MLP_NPARAMS, "parameter layout");

// The BF16 copies of W2..W4 (w_bf16) are kept in MFMA fragment order: the eight weights
// W_l[n][k8 .. k8 + 7] (k8 a multiple of 8) are lane 32 ((k8 / 8) mod 2) + n mod 32 of the
// 64-lane, 1 KB block (n / 32) 16 + k8 / 16, which is what lane of a 32 x 32 x 16 MFMA
// A fragment holds them. One neuron block's fragment for one K step is then one contiguous
// 1 KB read (eight full cache lines) rather than 32 pieces of 32 rows.
constexpr int WFB = 512;   // weights per fragment block
__host__ __device__ constexpr int wfrag(int n, int k) {
  return ((((n >> 5) * 16 + (k >> 4)) * 64 + ((k >> 3) & 1) * 32 + (n & 31)) << 3) + (k & 7);
}

// sigmoid(z) = 1 / (1 + e^-z) and silu(z) = z sigmoid(z), as exact as expf and an IEEE division give
// them in half the instructions: e^-|z| from the hardware exp2 with the argument's rounding put back
// (log2 e as two FP32 numbers), the quotient by the hardware reciprocal and one correction, which
// for silu also takes the roundings of 1 + e^-|z| and z e^-|z|.
struct Sig {
  float u, d, r;   // e^-|z|, 1 + u, about 1 / d
  bool neg;
  __device__ __forceinline__ explicit Sig(float z) {
    const float a = fminf(fabsf(z), 200.0f);   // beyond, e^-a is 0
    const float t = -1.44269502f * a;
    const float lo = fmaf(-1.92596299e-8f, a, fmaf(-1.44269502f, a, -t));
    const float e = __builtin_amdgcn_exp2f(t);
    u = fmaf(e, 0.693147181f * lo, e);
    d = 1.0f + u;
    r = __builtin_amdgcn_rcpf(d);
    neg = z < 0.0f;
  }
  __device__ __forceinline__ float sigmoid() const {
    const float n = neg ? u : 1.0f, q = n * r;
    return fmaf(r, fmaf(-d, q, n), q);
  }
  __device__ __forceinline__ float silu(float z) const {
    const float m = neg ? u : 1.0f, n = z * m, q = n * r;
    return fmaf(r, fmaf(-d, q, n) + fmaf((d - 1.0f) - u, q, fmaf(z, m, -n)), q);
  }
  __device__ __forceinline__ float silu_grad(float z) const {
    const float s = sigmoid();
    return s * (1.0f + z * (1.0f - s));
  }
};
__device__ __forceinline__ float silu_f(float z) { return Sig(z).silu(z); }
// SiLU from the hardware exp2 and reciprocal: for the activation operands of the layer products, of
// which one BF16 part or two keep 2^-8 or 2^-16, and for inference. Its relative error grows with |z|
// (the exponent's argument is rounded: 40 units of 2^-24 at z = -80), so what training keeps in
// FP32 (predictions, deltas, the gradients of W5) takes silu_f. Large |z| behave:
// exp2 overflows to inf and the reciprocal to 0 (z -> -inf), or exp2 goes to 0 (z -> +inf).
__device__ __forceinline__ float silu_fast(float z) {
  return z * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-1.4426950408889634f * z));
}
// float -> bf16 bits, round to nearest even (NaN stays NaN)
__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40);
  u += 0x7fffu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// ------------------------------------------------------------------ fused inference
// The whole network for tiles of FM = 64 queries, with no activation leaving the CU. Each
// layer is computed transposed, Z^T = W A^T: the weights are the MFMA's A operand (32 output
// neurons x 16 inputs per fragment, 16-byte loads of W rows from L2, where the three
// 256 x 256 BF16 matrices stay) and the activations its B operand, read from LDS, where a
// tile's activations live as their hi and lo BF16 parts (Ah, Al: [query][neuron], 68 KB per
// tile). A wave computes neurons 64 w .. 64 w + 63 for all 64 queries of its tile: four
// 32 x 32 accumulators, K in steps of 16, the A fragments loaded a few steps ahead, all hi
// products of a step before the lo products. An accumulator lane holds four consecutive
// neurons of one query per group, so the epilogue (bias, SiLU, hi / lo split) converts in
// pairs and stores eight-byte packets. The first layer (7 -> 256, FP32 weights) is three
// MFMAs per block with both operands split into hi and lo parts (W_hi x_hi + W_hi x_lo +
// W_lo x_hi: relative error ~2^-16, below the hidden layers' own); the last folds
// W5 silu(z4) into per-query partial sums.
//
// A workgroup is two groups of four waves, each with a tile of its own, and a tile goes
// through six phases: (0) the previous tile's output fold, then layer 1 and its epilogue,
// (1) layer 2's MFMAs, (2) its epilogue, (3) layer 3's MFMAs, (4) its epilogue, (5) layer
// 4's MFMAs. Group 1 runs one phase behind group 0 and one barrier of the whole workgroup
// ends every phase, so the two waves that share a SIMD (wave w of each group) alternate:
// one issues MFMAs while the other runs its VALU epilogue. The barrier also orders each
// group's own LDS traffic: a phase's epilogue writes the activations the next phase's MFMAs
// read, after every wave of the group has read the previous layer's.
constexpr int FM = 64;               // queries per tile
constexpr int FQB = FM / 32;         // query blocks
constexpr int FP = NW + 8;           // LDS row pitch (bf16): 528 bytes, 16-byte aligned
constexpr size_t FUSED_LDS = sizeof(uint16_t) * 2 * 2 * FM * FP;   // two tiles, hi and lo
constexpr int FPD = 3;               // K steps between a weight fragment's load and its use
constexpr int FPH = 6;               // phases per tile

__device__ __forceinline__ void split8(const float *v, s16x8 &hi, s16x8 &lo) {
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint16_t h = __builtin_bit_cast(uint16_t, (__bf16)v[i]);
    hi[i] = (short)h;
    lo[i] = (short)__builtin_bit_cast(uint16_t, (__bf16)(v[i] - bf2f(h)));
  }
}

__global__ __launch_bounds__(512, 1) void k_mlp_fused(const float *__restrict__ x, int B, const float *__restrict__ p,
                                                   const uint16_t *__restrict__ wbf, cm_mlp net,
                                                   float *__restrict__ y) {
  extern __shared__ __align__(16) uint16_t fl[];
  __shared__ float bsh[4][NW];   // b1..b4
  __shared__ float w5s[NW];
  __shared__ float ys[2][4][FM];  // per-group, per-wave partial outputs
  const int tid = threadIdx.x, lane = tid & 63;
  const int grp = tid >> 8, w = (tid >> 6) & 3, gtid = tid & 255;
  const int l32 = lane & 31, hi32 = lane >> 5;
  uint16_t *Ah = fl + grp * 2 * FM * FP, *Al = Ah + FM * FP;
  for (int e = tid; e < NW; e += 512) {
    bsh[0][e] = p[OFF_B1 + e];
    bsh[1][e] = p[off_b(2) + e];
    bsh[2][e] = p[off_b(3) + e];
    bsh[3][e] = p[off_b(4) + e];
    w5s[e] = p[OFF_W5 + e];
  }
  // first-layer A fragments: W1[n][k], n = 64 w + 32 mb + l32, k = 8 hi32 + i (k < 7; zero
  // beyond), split into hi and lo
  bf16x8 w1h[2], w1l[2];
#pragma unroll
  for (int mb = 0; mb < 2; ++mb) {
    float v[8];
    const int n = 64 * w + 32 * mb + l32;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int k = 8 * hi32 + i;
      v[i] = k < NIN ? p[OFF_W1 + n * NIN + k] : 0.0f;
    }
    s16x8 h, l;
    split8(v, h, l);
    w1h[mb] = __builtin_bit_cast(bf16x8, h);
    w1l[mb] = __builtin_bit_cast(bf16x8, l);
  }
  __syncthreads();
  // the tiles of group g are 2 blockIdx.x + g + i stride, i = 0, 1, ...
  const int ntiles = (B + FM - 1) / FM;
  const int stride = 2 * gridDim.x;
  const int f0 = 2 * blockIdx.x, f1 = f0 + 1;
  const int n0 = f0 < ntiles ? (ntiles - 1 - f0) / stride + 1 : 0;
  const int n1 = f1 < ntiles ? (ntiles - 1 - f1) / stride + 1 : 0;
  const int nmine = grp ? n1 : n0;
  // a group's own steps: FPH per tile, then the last tile's fold (phase 0) and output
  // (phase 1); group 1 starts one step late. Every wave runs the same number of barriers.
  const int last0 = n0 ? FPH * n0 + 2 : 0, last1 = n1 ? 1 + FPH * n1 + 2 : 0;
  const int nsteps = last0 > last1 ? last0 : last1;
  f32x16 acc[2][FQB];
  s16x8 ar0[FPD], ar1[FPD];
  // accumulators start at the layer's bias: element v of block mb is neuron
  // 64 w + 32 mb + 8 (v / 4) + 4 hi32 + v mod 4, the same for both query blocks
  auto bias_init = [&](const float *bias) {
#pragma unroll
    for (int mb = 0; mb < 2; ++mb) {
      f32x16 bz;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const float4 b4 = *(const float4 *)&bias[64 * w + 32 * mb + 8 * g + 4 * hi32];
        bz[4 * g] = b4.x;
        bz[4 * g + 1] = b4.y;
        bz[4 * g + 2] = b4.z;
        bz[4 * g + 3] = b4.w;
      }
#pragma unroll
      for (int qb = 0; qb < FQB; ++qb) acc[mb][qb] = bz;
    }
  };
  for (int st = 0; st < nsteps; ++st) {
    const int ls = st - grp;
    if (ls >= 0 && ls < FPH * nmine + 2) {
      const int i = ls / FPH, ph = ls - FPH * i;
      const int q0 = (f0 + grp + i * stride) * FM;   // this step's tile (while i < nmine)
      if (ph & 1) {
        if (ph == 1 && i > 0 && gtid < FM && q0 - stride * FM + gtid < B) {
          const int t = gtid;
          y[q0 - stride * FM + t] = ((ys[grp][0][t] + ys[grp][1][t]) + (ys[grp][2][t] + ys[grp][3][t])) + p[OFF_B5];
        }
        if (i < nmine) {
          // layers 2, 3, 4 at phases 1, 3, 5
          const uint16_t *W = wbf + (int64_t)(ph >> 1) * NW * NW;
          bias_init(bsh[1 + (ph >> 1)]);
          // A fragment of neuron block 2 w + mb at K step ks: W[n][16 ks + 8 hi32 .. +7],
          // n = 64 w + 32 mb + l32, one contiguous 1 KB block of the fragment-ordered copy,
          // read from L2 FPD steps ahead into a ring indexed statically by the unrolled K loop
          const uint16_t *wrow0 = W + (int64_t)(2 * w) * 16 * WFB + 8 * lane;
          const uint16_t *wrow1 = wrow0 + 16 * WFB;
          // B fragments of query block qb at K step kk: Ah / Al[q][kk + 8 hi32 .. +7], q = 32 qb + l32
          const int boff = l32 * FP + 8 * hi32;
          s16x8 bhn[FQB], bln[FQB];
#pragma unroll
          for (int qb = 0; qb < FQB; ++qb) {
            bhn[qb] = *(const s16x8 *)&Ah[boff + 32 * qb * FP];
            bln[qb] = *(const s16x8 *)&Al[boff + 32 * qb * FP];
          }
#pragma unroll
          for (int ks = 0; ks < NW / 16; ++ks) {
            const int kk = 16 * ks;
            const bf16x8 A0 = __builtin_bit_cast(bf16x8, ar0[ks % FPD]), A1 = __builtin_bit_cast(bf16x8, ar1[ks % FPD]);
            if (ks + FPD < NW / 16) {
              ar0[ks % FPD] = *(const s16x8 *)(wrow0 + (ks + FPD) * WFB);
              ar1[ks % FPD] = *(const s16x8 *)(wrow1 + (ks + FPD) * WFB);
            }
            s16x8 bh[FQB], bl[FQB];
#pragma unroll
            for (int qb = 0; qb < FQB; ++qb) {
              bh[qb] = bhn[qb];
              bl[qb] = bln[qb];
            }
            if (kk + 16 < NW) {   // next step's activations, in flight during this step's MFMAs
#pragma unroll
              for (int qb = 0; qb < FQB; ++qb) {
                bhn[qb] = *(const s16x8 *)&Ah[boff + 32 * qb * FP + kk + 16];
                bln[qb] = *(const s16x8 *)&Al[boff + 32 * qb * FP + kk + 16];
              }
            }
#pragma unroll
            for (int qb = 0; qb < FQB; ++qb) {
              const bf16x8 BH = __builtin_bit_cast(bf16x8, bh[qb]);
              acc[0][qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A0, BH, acc[0][qb], 0, 0, 0);
              acc[1][qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A1, BH, acc[1][qb], 0, 0, 0);
            }
#pragma unroll
            for (int qb = 0; qb < FQB; ++qb) {
              const bf16x8 BL = __builtin_bit_cast(bf16x8, bl[qb]);
              acc[0][qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A0, BL, acc[0][qb], 0, 0, 0);
              acc[1][qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A1, BL, acc[1][qb], 0, 0, 0);
            }
          }
        }
      } else {
        if (ph == 0) {
          if (i > 0) {
            // the previous tile's y[q] = b5 + sum_n W5[n] silu(z4[n][q]) over this lane's 32
            // neurons; the two half waves hold the same queries' other neurons
#pragma unroll
            for (int qb = 0; qb < FQB; ++qb) {
              float sacc = 0.0f;
#pragma unroll
              for (int mb = 0; mb < 2; ++mb)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                  const int n = 64 * w + 32 * mb + 8 * (v >> 2) + 4 * hi32 + (v & 3);
                  sacc += w5s[n] * silu_fast(acc[mb][qb][v]);
                }
              const float s2 = sacc + __shfl_xor(sacc, 32, 64);
              if (hi32 == 0) ys[grp][w][32 * qb + l32] = s2;
            }
          }
          if (i < nmine) {
            // layer 1: B fragments xn[q][k], q = 32 qb + l32, k = 8 hi32 + i
            bf16x8 xh[FQB], xl[FQB];
#pragma unroll
            for (int qb = 0; qb < FQB; ++qb) {
              const int q = q0 + 32 * qb + l32;
              float v[8];
#pragma unroll
              for (int j = 0; j < 8; ++j) {
                const int k = 8 * hi32 + j;
                v[j] = (k < NIN && q < B) ? (x[(int64_t)q * NIN + k] - net.shift[k]) * net.scale[k] : 0.0f;
              }
              s16x8 h, l;
              split8(v, h, l);
              xh[qb] = __builtin_bit_cast(bf16x8, h);
              xl[qb] = __builtin_bit_cast(bf16x8, l);
            }
            bias_init(bsh[0]);
#pragma unroll
            for (int mb = 0; mb < 2; ++mb)
#pragma unroll
              for (int qb = 0; qb < FQB; ++qb) {
                acc[mb][qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1h[mb], xh[qb], acc[mb][qb], 0, 0, 0);
                acc[mb][qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1h[mb], xl[qb], acc[mb][qb], 0, 0, 0);
                acc[mb][qb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1l[mb], xh[qb], acc[mb][qb], 0, 0, 0);
              }
          }
        }
        if (i < nmine) {
          {
            // the next phase's first weight fragments, in flight during this epilogue
            const uint16_t *wrow0 = wbf + (int64_t)(ph >> 1) * NW * NW + (int64_t)(2 * w) * 16 * WFB + 8 * lane;
            const uint16_t *wrow1 = wrow0 + 16 * WFB;
#pragma unroll
            for (int s = 0; s < FPD; ++s) {
              ar0[s] = *(const s16x8 *)(wrow0 + s * WFB);
              ar1[s] = *(const s16x8 *)(wrow1 + s * WFB);
            }
          }
          // epilogue of layers 1, 2, 3 at phases 0, 2, 4: neurons 64 w + 32 mb + 8 g + 4 hi32 + j
          // (j < 4) of query 32 qb + l32 are acc[mb][qb][4 g + j], bias included
#pragma unroll
          for (int mb = 0; mb < 2; ++mb)
#pragma unroll
            for (int qb = 0; qb < FQB; ++qb)
#pragma unroll
              for (int g = 0; g < 4; ++g) {
                const int n = 64 * w + 32 * mb + 8 * g + 4 * hi32;
                float v[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) v[j] = silu_fast(acc[mb][qb][4 * g + j]);
                uint16_t h[4], lo[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                  h[j] = __builtin_bit_cast(uint16_t, (__bf16)v[j]);
                  lo[j] = __builtin_bit_cast(uint16_t, (__bf16)(v[j] - bf2f(h[j])));
                }
                const int off = (32 * qb + l32) * FP + n;
                *(uint2 *)&Ah[off] = make_uint2(h[0] | ((uint32_t)h[1] << 16), h[2] | ((uint32_t)h[3] << 16));
                *(uint2 *)&Al[off] = make_uint2(lo[0] | ((uint32_t)lo[1] << 16), lo[2] | ((uint32_t)lo[3] << 16));
              }
        }
      }
    }
    __syncthreads();
  }
}

// ------------------------------------------------------------------ tiles of 32 rows
// One workgroup of eight waves takes 32 rows through a chain of 256 x 256 products; wave w
// owns neurons 32 w .. 32 w + 31 of every layer (one 32 x 32 accumulator per operand part).
// As in k_mlp_fused the products are transposed (weights are the A operand, in fragment order;
// the rows' values the B operand, hi and lo parts in LDS). All 16 weight fragments of the next
// layer are loaded while the present one finishes, and the values alternate between two LDS
// buffers, so a layer costs one barrier. 8192 rows are 256 tiles, one per CU; a launch per layer
// with the weights staged in LDS put one 32-row tile on two of sixteen waves behind 128 KB of
// staging. 8192 rows: forward with the pre-activations stored 21 us (58 before), backward
// chain 33 us (107 before, its first-layer gradients included); 777 rows of inference 9.6 us
// (27 with tiles of 64). Bound by the latency of a layer (fragments, products, epilogue): at 8192
// rows two waves a SIMD, 17 % of its cycles issuing VALU instructions.
constexpr int TM = 32;
constexpr int TWG = 512;
constexpr int TKS = NW / 16;                                        // K steps per layer
constexpr size_t TILE_BUF = (size_t)2 * TM * FP;                    // hi and lo parts (uint16)
constexpr size_t TILE_LDS = sizeof(uint16_t) * 2 * TILE_BUF;

// hi + lo parts of four consecutive neurons' values of row r into a tile buffer
__device__ __forceinline__ void put4(uint16_t *buf, int r, int n, const float *v) {
  uint16_t h[4], lo[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    h[j] = __builtin_bit_cast(uint16_t, (__bf16)v[j]);
    lo[j] = __builtin_bit_cast(uint16_t, (__bf16)(v[j] - bf2f(h[j])));
  }
  const int off = r * FP + n;
  *(uint2 *)&buf[off] = make_uint2(h[0] | ((uint32_t)h[1] << 16), h[2] | ((uint32_t)h[3] << 16));
  *(uint2 *)&buf[TM * FP + off] = make_uint2(lo[0] | ((uint32_t)lo[1] << 16), lo[2] | ((uint32_t)lo[3] << 16));
}

// the 16 weight fragments of neuron block w (fragment-ordered matrix W)
__device__ __forceinline__ void load_frags(const uint16_t *__restrict__ W, int w, int lane, s16x8 *f) {
  const uint16_t *src = W + (int64_t)w * TKS * WFB + 8 * lane;
#pragma unroll
  for (int ks = 0; ks < TKS; ++ks) f[ks] = *(const s16x8 *)(src + ks * WFB);
}

// acc[0] += W_block hi(values), acc[1] += W_block lo(values) over all K: two independent chains
__device__ __forceinline__ void tile_product(const uint16_t *buf, int lane, const s16x8 *f, f32x16 *acc) {
  const uint16_t *src = buf + (lane & 31) * FP + 8 * (lane >> 5);
#pragma unroll
  for (int ks = 0; ks < TKS; ++ks) {
    const bf16x8 A = __builtin_bit_cast(bf16x8, f[ks]);
    const s16x8 bh = *(const s16x8 *)(src + 16 * ks), bl = *(const s16x8 *)(src + TM * FP + 16 * ks);
    acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A, __builtin_bit_cast(bf16x8, bh), acc[0], 0, 0, 0);
    acc[1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A, __builtin_bit_cast(bf16x8, bl), acc[1], 0, 0, 0);
  }
}

// The same with one chain, hi before lo in every K step, as k_mlp_fused adds.
__device__ __forceinline__ void tile_product_1(const uint16_t *buf, int lane, const s16x8 *f, f32x16 &acc) {
  const uint16_t *src = buf + (lane & 31) * FP + 8 * (lane >> 5);
#pragma unroll
  for (int ks = 0; ks < TKS; ++ks) {
    const bf16x8 A = __builtin_bit_cast(bf16x8, f[ks]);
    const s16x8 bh = *(const s16x8 *)(src + 16 * ks), bl = *(const s16x8 *)(src + TM * FP + 16 * ks);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A, __builtin_bit_cast(bf16x8, bh), acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(A, __builtin_bit_cast(bf16x8, bl), acc, 0, 0, 0);
  }
}

// y[b] = network(x[b]). With KEEP (training) the pre-activations Z1..Z4 go to Z ([4][B][256]), layer 1
// is summed in FP32 and the two operand parts in chains of their own. Without it (inference) every
// sum is formed by k_mlp_fused's operations in its order, so that a row's output does not depend
// on the batch it came in: with sums of its own this kernel was off by 6.6e-8 of the outputs'
// norm where k_mlp_fused is by 4.7e-8 (777 to 24000 rows, against FP64).
template <bool KEEP>
__global__ __launch_bounds__(TWG) void k_mlp_tile(const float *__restrict__ x, int B, const float *__restrict__ p,
                                                  const uint16_t *__restrict__ wbf, cm_mlp net,
                                                  float *__restrict__ y, float *__restrict__ Z) {
  extern __shared__ __align__(16) uint16_t tl[];
  __shared__ __align__(16) float w1s[KEEP ? NW * NIN : 4], bsh[4][NW], w5s[NW];
  __shared__ float xs[KEEP ? TM : 1][NIN + 1], ys[8][TM], half[4][64];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int l32 = lane & 31, hi32 = lane >> 5;
  const int q0 = blockIdx.x * TM, q = q0 + l32;
  s16x8 f[TKS];
  load_frags(wbf, w, lane, f);
  bf16x8 w1h, w1l, xh, xl;   // layer 1's operands (inference)
  if constexpr (KEEP) {
    for (int e = tid; e < NW * NIN; e += TWG) w1s[e] = p[OFF_W1 + e];
    if (tid < TM * NIN) {
      const int r = tid / NIN, i = tid % NIN;
      xs[r][i] = q0 + r < B ? (x[(int64_t)(q0 + r) * NIN + i] - net.shift[i]) * net.scale[i] : 0.0f;
    }
  } else {
    float a[8], b[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int k = 8 * hi32 + i;
      a[i] = k < NIN ? p[OFF_W1 + (32 * w + l32) * NIN + k] : 0.0f;
      b[i] = (k < NIN && q < B) ? (x[(int64_t)q * NIN + k] - net.shift[k]) * net.scale[k] : 0.0f;
    }
    s16x8 h, l;
    split8(a, h, l);
    w1h = __builtin_bit_cast(bf16x8, h);
    w1l = __builtin_bit_cast(bf16x8, l);
    split8(b, h, l);
    xh = __builtin_bit_cast(bf16x8, h);
    xl = __builtin_bit_cast(bf16x8, l);
  }
  for (int e = tid; e < NW; e += TWG) {
    bsh[0][e] = p[OFF_B1 + e];
    bsh[1][e] = p[off_b(2) + e];
    bsh[2][e] = p[off_b(3) + e];
    bsh[3][e] = p[off_b(4) + e];
    w5s[e] = p[OFF_W5 + e];
  }
  __syncthreads();
  f32x16 acc[2];
  // accumulator v of this lane: neuron 32 w + 8 (v / 4) + 4 hi32 + v mod 4 of row l32
  auto bias_init = [&](const float *bias) {
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 b4 = *(const float4 *)&bias[32 * w + 8 * g + 4 * hi32];
      acc[0][4 * g] = b4.x; acc[0][4 * g + 1] = b4.y; acc[0][4 * g + 2] = b4.z; acc[0][4 * g + 3] = b4.w;
    }
  };
  if constexpr (KEEP) {
    float xr[NIN];
#pragma unroll
    for (int i = 0; i < NIN; ++i) xr[i] = xs[l32][i];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int n = 32 * w + 8 * g + 4 * hi32;
      float wv[4 * NIN];   // rows n .. n + 3 of W1, contiguous
#pragma unroll
      for (int c = 0; c < NIN; ++c) {
        const float4 t = *(const float4 *)&w1s[n * NIN + 4 * c];
        wv[4 * c] = t.x; wv[4 * c + 1] = t.y; wv[4 * c + 2] = t.z; wv[4 * c + 3] = t.w;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float s = bsh[0][n + j];
#pragma unroll
        for (int i = 0; i < NIN; ++i) s += wv[j * NIN + i] * xr[i];
        acc[0][4 * g + j] = s;
      }
    }
  } else {
    bias_init(bsh[0]);
    acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1h, xh, acc[0], 0, 0, 0);
    acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1h, xl, acc[0], 0, 0, 0);
    acc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(w1l, xh, acc[0], 0, 0, 0);
  }
#pragma unroll
  for (int l = 2; l <= 5; ++l) {
    // acc[0] holds z_{l-1}: store it, then either the output fold or the next product
    float v[16];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int n = 32 * w + 8 * g + 4 * hi32;
      if (KEEP && q < B)
        *(float4 *)&Z[((int64_t)(l - 2) * B + q) * NW + n] =
            make_float4(acc[0][4 * g], acc[0][4 * g + 1], acc[0][4 * g + 2], acc[0][4 * g + 3]);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        v[4 * g + j] = KEEP && l == 5 ? silu_f(acc[0][4 * g + j]) : silu_fast(acc[0][4 * g + j]);
    }
    if (l == 5) {
      float s = 0.0f;
      auto fold = [&]() {
#pragma unroll
        for (int k = 0; k < 16; ++k) s += w5s[32 * w + 8 * (k >> 2) + 4 * hi32 + (k & 3)] * v[k];
      };
      if (KEEP || !(w & 1)) fold();
      if constexpr (!KEEP) {   // a lane of k_mlp_fused adds the neurons of two waves here, the even one's first
        if (!(w & 1)) half[w >> 1][lane] = s;
        __syncthreads();
        if (w & 1) {
          s = half[w >> 1][lane];
          fold();
        }
      }
      s += __shfl_xor(s, 32, 64);
      if (hi32 == 0) ys[w][l32] = s;
    } else {
      uint16_t *buf = tl + (l & 1) * TILE_BUF;
#pragma unroll
      for (int g = 0; g < 4; ++g) put4(buf, l32, 32 * w + 8 * g + 4 * hi32, v + 4 * g);
      bias_init(bsh[l - 1]);
#pragma unroll
      for (int k = 0; k < 16; ++k) acc[1][k] = 0.0f;
      __syncthreads();
      if constexpr (KEEP) tile_product(buf, lane, f, acc);
      else tile_product_1(buf, lane, f, acc[0]);
      if (l < 4) load_frags(wbf + (int64_t)(l - 1) * NW * NW, w, lane, f);
      if constexpr (KEEP) {
#pragma unroll
        for (int k = 0; k < 16; ++k) acc[0][k] += acc[1][k];
      }
    }
  }
  __syncthreads();
  if (tid < TM && q0 + tid < B) {
    if constexpr (KEEP) {
      float s = p[OFF_B5];
#pragma unroll
      for (int k = 0; k < 8; ++k) s += ys[k][tid];
      y[q0 + tid] = s;
    } else {
      y[q0 + tid] = ((ys[1][tid] + ys[3][tid]) + (ys[5][tid] + ys[7][tid])) + p[OFF_B5];
    }
  }
}

// ------------------------------------------------------------------ backward
// Where the transposed weight copies W4^T, W3^T, W2^T (fragment order) live during the backward
// chain: in the gradient buffer, inside W3's and W4's gradients, which are only accumulated
// after it. 16-byte aligned whatever the buffer's own alignment.
__host__ __device__ inline uint16_t *grad_scratch(float *grad) {
  return (uint16_t *)(((uintptr_t)(grad + off_w(3)) + 15) & ~(uintptr_t)15);
}
// Behind them, copies of the first layer's gradients (W1, b1), which the tiles of k_mlp_bwd add
// to by turns: 256 tiles adding to each address serialised (59 us against 31 us at 8192 rows).
// k_bwd_mid sums them and clears the space.
constexpr int FIRST_COPIES = 16, FIRST_OFF = off_w(3) + 4 + 3 * NW * NW / 2, FIRST_N = off_w(2);
static_assert(FIRST_OFF + FIRST_COPIES * FIRST_N <= OFF_W5, "the scratch fits before W5's gradient");

// Transposes the BF16 copies (one 8 x 8 piece per thread) and clears the copies of the first
// layer's gradients.
__global__ __launch_bounds__(256) void k_bwd_prep(const uint16_t *__restrict__ wbf, uint16_t *__restrict__ wt,
                                                  float *__restrict__ grad) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e >= 3 * NW * NW / 64) {   // 3 * 1024 pieces, then the copies
    const int c = e - 3 * NW * NW / 64;
    if (c < FIRST_COPIES * FIRST_N) grad[FIRST_OFF + c] = 0.0f;
    return;
  }
  const int l = e >> 10, n0 = 8 * ((e >> 5) & 31), k0 = 8 * (e & 31);
  s16x8 r[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) r[i] = *(const s16x8 *)&wbf[l * NW * NW + wfrag(n0 + i, k0)];
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    s16x8 c;
#pragma unroll
    for (int i = 0; i < 8; ++i) c[i] = r[i][j];
    *(s16x8 *)&wt[l * NW * NW + wfrag(k0 + j, n0)] = c;
  }
}

// Between the backward chain and k_wgrad: the first layer's gradients from their copies, and
// zeros in every other gradient (each copy's element is cleared by the thread that read it).
__global__ __launch_bounds__(256) void k_bwd_mid(float *__restrict__ grad) {
  const int e = blockIdx.x * 256 + threadIdx.x;
  if (e < FIRST_N) {
    float s = 0.0f;
#pragma unroll
    for (int c = 0; c < FIRST_COPIES; ++c) s += grad[FIRST_OFF + c * FIRST_N + e];
#pragma unroll
    for (int c = 0; c < FIRST_COPIES; ++c) grad[FIRST_OFF + c * FIRST_N + e] = 0.0f;
    grad[e] = s;
  } else if (e < CM_MLP_NPARAMS && (e < FIRST_OFF || e >= FIRST_OFF + FIRST_COPIES * FIRST_N)) {
    grad[e] = 0.0f;
  }
}

// delta_4 = dy W5 silu'(Z4), delta_{l-1} = (delta_l W_l) silu'(Z_{l-1}) for a tile of 32 rows;
// delta_3 and delta_2 go to D ([2][B][256]), delta_1 stays on chip and is summed into W1's and
// b1's gradients (FP32, one atomic per gradient and tile, to one of their copies).
__global__ __launch_bounds__(TWG) void k_mlp_bwd(const float *__restrict__ x, const float *__restrict__ Z,
                                                 const float *__restrict__ dy, int B, const float *__restrict__ p,
                                                 const uint16_t *__restrict__ wt, cm_mlp net, float *__restrict__ D,
                                                 float *__restrict__ grad) {
  extern __shared__ __align__(16) uint16_t tl[];
  __shared__ float xs[TM][8];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int l32 = lane & 31, hi32 = lane >> 5;
  const int q0 = blockIdx.x * TM, q = q0 + l32;
  const bool ok = q < B;
  const int64_t zrow = (int64_t)(ok ? q : 0) * NW, BN = (int64_t)B * NW;
  s16x8 f[TKS];
  load_frags(wt + 2 * NW * NW, w, lane, f);
  if (tid < TM * 8) {
    const int r = tid >> 3, i = tid & 7;
    xs[r][i] = q0 + r >= B ? 0.0f : i == NIN ? 1.0f : (x[(int64_t)(q0 + r) * NIN + i] - net.shift[i]) * net.scale[i];
  }
  float v[16];
  {
    const float d = ok ? dy[q] : 0.0f;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int n = 32 * w + 8 * g + 4 * hi32;
      const float4 z = *(const float4 *)&Z[3 * BN + zrow + n];
      v[4 * g] = d * p[OFF_W5 + n] * Sig(z.x).silu_grad(z.x);
      v[4 * g + 1] = d * p[OFF_W5 + n + 1] * Sig(z.y).silu_grad(z.y);
      v[4 * g + 2] = d * p[OFF_W5 + n + 2] * Sig(z.z).silu_grad(z.z);
      v[4 * g + 3] = d * p[OFF_W5 + n + 3] * Sig(z.w).silu_grad(z.w);
      put4(tl, l32, n, v + 4 * g);
    }
  }
#pragma unroll
  for (int l = 4; l >= 2; --l) {
    const uint16_t *buf = tl + (l & 1) * TILE_BUF;
    float4 z[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) z[g] = *(const float4 *)&Z[(l - 2) * BN + zrow + 32 * w + 8 * g + 4 * hi32];
    f32x16 acc[2];
#pragma unroll
    for (int k = 0; k < 16; ++k) acc[0][k] = acc[1][k] = 0.0f;
    __syncthreads();
    tile_product(buf, lane, f, acc);
    if (l > 2) load_frags(wt + (int64_t)(l - 3) * NW * NW, w, lane, f);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      v[4 * g] = (acc[0][4 * g] + acc[1][4 * g]) * Sig(z[g].x).silu_grad(z[g].x);
      v[4 * g + 1] = (acc[0][4 * g + 1] + acc[1][4 * g + 1]) * Sig(z[g].y).silu_grad(z[g].y);
      v[4 * g + 2] = (acc[0][4 * g + 2] + acc[1][4 * g + 2]) * Sig(z[g].z).silu_grad(z[g].z);
      v[4 * g + 3] = (acc[0][4 * g + 3] + acc[1][4 * g + 3]) * Sig(z[g].w).silu_grad(z[g].w);
      const int n = 32 * w + 8 * g + 4 * hi32;
      if (l > 2) {
        put4(tl + ((l - 1) & 1) * TILE_BUF, l32, n, v + 4 * g);
        if (ok) *(float4 *)&D[(4 - l) * BN + zrow + n] = make_float4(v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]);
      }
    }
  }
  // delta_1 as FP32 rows of 260 in LDS (over both buffers, once every wave has read the last)
  constexpr int DP = NW + 4;
  static_assert(sizeof(float) * (TM * DP + 8 * NW) <= TILE_LDS, "delta_1 and the half sums fit the tile buffers");
  float *d1 = (float *)tl, *half = d1 + TM * DP;
  __syncthreads();
#pragma unroll
  for (int g = 0; g < 4; ++g) *(float4 *)&d1[l32 * DP + 32 * w + 8 * g + 4 * hi32] =
      make_float4(v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]);
  __syncthreads();
  const int n = tid & (NW - 1), r0 = (tid >> 8) * (TM / 2);
  float gs[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) gs[i] = 0.0f;
#pragma unroll
  for (int r = 0; r < TM / 2; ++r) {
    const float d = d1[(r0 + r) * DP + n];
#pragma unroll
    for (int i = 0; i < 8; ++i) gs[i] += d * xs[r0 + r][i];
  }
  if (tid >= NW) {
#pragma unroll
    for (int i = 0; i < 8; ++i) half[i * NW + n] = gs[i];
  }
  __syncthreads();
  if (tid < NW) {
    float *first = grad + FIRST_OFF + (blockIdx.x % FIRST_COPIES) * FIRST_N;
#pragma unroll
    for (int i = 0; i < 8; ++i)
      atomicAdd(first + (i < NIN ? OFF_W1 + n * NIN + i : OFF_B1 + n), gs[i] + half[i * NW + n]);
  }
}

// Gradients of layers 2..5 from the batch: gW_l[m][n] += sum_b delta_l[b][m] silu(Z_{l-1}[b][n])
// (delta split into hi + lo parts, the activation rounded to BF16), gb_l += sum_b delta_l[b],
// gW5 += sum_b dy[b] silu(Z4[b]), gb5 += sum_b dy[b]. A workgroup takes one span of rows for one
// layer and 128 x 128 tile. Workgroups go to the eight XCDs in turn, so the twelve tiles of a span
// are numbered eight apart: they read the same rows and share one L2. The batch is the K dimension, so a lane's fragment is eight rows
// of one column: eight dword loads whose lanes run along the row (128-byte segments), converted
// in registers. Each wave converts one of the four 32-column blocks of either operand and
// shares the fragments through LDS, so nothing is loaded or converted twice in a workgroup; the
// next rows' loads are in flight during the products. delta_4 is formed here from dy and Z4.
// 8192 rows take 39 us for all layers (35 with the fast SiLU also in W5's gradient and the deltas),
// about 10 of them the 6.3 M atomics of 32 spans (16 spans 53 us against those 35: too few workgroups;
// 64 about 10 us more atomics); it is bound by the latency of a step's loads. It replaces, per layer,
// a 64 x 64-tile kernel that converted each element in four workgroups (44 us) and a column sum
// (19 us).
constexpr int GWT = 128;                  // tile edge
constexpr int GKR = 32;                   // rows per step
constexpr int WG_SPANS = 32;              // spans of rows (see cm_mlp_backward)
constexpr int XCDS = 8;
__global__ __launch_bounds__(256) void k_wgrad(const float *__restrict__ Z, const float *__restrict__ dy,
                                               const float *__restrict__ D, int B, int span,
                                               const float *__restrict__ p, float *__restrict__ grad) {
  __shared__ __align__(16) uint16_t fr[2][3][2][4][64 * 8];   // [buffer][A hi, A lo, B][K half][block][lane]
  const int tid = threadIdx.x, lane = tid & 63, wv = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l32 = lane & 31, hi32 = lane >> 5;
  const int slot = blockIdx.x / XCDS, tile = slot % 12;
  const int rbeg = (blockIdx.x % XCDS + XCDS * (slot / 12)) * span;
  if (rbeg >= B) return;
  const int layer = 4 - (tile >> 2);                          // 4, 3, 2
  const int m0 = ((tile >> 1) & 1) * GWT, n0 = (tile & 1) * GWT;
  const int64_t BN = (int64_t)B * NW;
  const int rend = min(B, rbeg + span);
  const int ca = m0 + 32 * wv + l32, cb = n0 + 32 * wv + l32;   // this lane's columns
  const float *Asrc = layer == 4 ? Z + 3 * BN : D + (3 - layer) * BN;
  const float *Bsrc = Z + (layer - 2) * BN;
  const float w5 = layer == 4 ? p[OFF_W5 + ca] : 0.0f;
  const bool sums = n0 == 0;              // these workgroups also add the bias gradients
  float gb = 0.0f, g5 = 0.0f, gd = 0.0f;
  struct Rows {
    float a[2][8], b[2][8], d[2][8];
  };
  auto load = [&](int r0, Rows &t) {
    if (r0 + GKR <= rend) {   // uniform: whole steps address their rows by constant offsets
      const int64_t o = (int64_t)(r0 + 8 * hi32) * NW;
      const float *pa = Asrc + o + ca, *pb = Bsrc + o + cb, *pd = dy + r0 + 8 * hi32;
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          t.a[h][i] = pa[(16 * h + i) * NW];
          t.b[h][i] = pb[(16 * h + i) * NW];
          t.d[h][i] = layer == 4 ? pd[16 * h + i] : 1.0f;
        }
      return;
    }
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int r = r0 + 16 * h + 8 * hi32 + i;
        const bool in = r < rend;
        const int64_t o = (int64_t)(in ? r : rbeg) * NW;
        t.a[h][i] = in ? Asrc[o + ca] : 0.0f;
        t.b[h][i] = Bsrc[o + cb];
        t.d[h][i] = !in ? 0.0f : layer == 4 ? dy[r] : 1.0f;
      }
  };
  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int k = 0; k < 16; ++k) acc[i][j][k] = 0.0f;
  Rows cur, nxt;
  load(rbeg, cur);
  int b = 0;
  for (int r0 = rbeg; r0 < rend; r0 += GKR, b ^= 1) {
    // the next step's rows are in flight during this step's conversions and products
    if (r0 + GKR < rend) load(r0 + GKR, nxt);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      float a[8], s[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        // rows past the span carry zeros in a and d
        a[i] = cur.a[h][i];
        if (layer == 4) {
          const float z = a[i];
          const Sig sg(z);
          a[i] = cur.d[h][i] * w5 * sg.silu_grad(z);
          g5 += cur.d[h][i] * sg.silu(z);
          gd += cur.d[h][i];
        }
        gb += a[i];
        s[i] = silu_fast(cur.b[h][i]);   // rounded to BF16 next
      }
      s16x8 hi, lo, sb;
      split8(a, hi, lo);
#pragma unroll
      for (int i = 0; i < 8; ++i) sb[i] = (short)__builtin_bit_cast(uint16_t, (__bf16)s[i]);
      *(s16x8 *)&fr[b][0][h][wv][8 * lane] = hi;
      *(s16x8 *)&fr[b][1][h][wv][8 * lane] = lo;
      *(s16x8 *)&fr[b][2][h][wv][8 * lane] = sb;
    }
    cur = nxt;
    // one barrier per step: a wave writes the other buffer next, which every wave has finished
    // reading once it arrives here again
    __syncthreads();
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      bf16x8 Ah[2], Al[2], Bf[2];
#pragma unroll
      for (int i = 0; i < 2; ++i) {
        Ah[i] = __builtin_bit_cast(bf16x8, *(const s16x8 *)&fr[b][0][h][2 * (wv >> 1) + i][8 * lane]);
        Al[i] = __builtin_bit_cast(bf16x8, *(const s16x8 *)&fr[b][1][h][2 * (wv >> 1) + i][8 * lane]);
        Bf[i] = __builtin_bit_cast(bf16x8, *(const s16x8 *)&fr[b][2][h][2 * (wv & 1) + i][8 * lane]);
      }
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Ah[i], Bf[j], acc[i][j], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(Al[i], Bf[j], acc[i][j], 0, 0, 0);
    }
  }
  float *gw = grad + off_w(layer);
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        const int m = m0 + 64 * (wv >> 1) + 32 * i + 8 * (k >> 2) + 4 * hi32 + (k & 3);
        atomicAdd(gw + m * NW + n0 + 64 * (wv & 1) + 32 * j + l32, acc[i][j][k]);
      }
  if (sums) {
    gb += __shfl_xor(gb, 32, 64);
    g5 += __shfl_xor(g5, 32, 64);
    gd += __shfl_xor(gd, 32, 64);
    if (hi32 == 0) {
      atomicAdd(grad + off_b(layer) + ca, gb);
      if (layer == 4) {
        atomicAdd(grad + OFF_W5 + ca, g5);
        if (m0 == 0 && wv == 0 && l32 == 0) atomicAdd(grad + OFF_B5, gd);
      }
    }
  }
}

__global__ void k_mse(const float *__restrict__ y, const float *__restrict__ t, int B, float *__restrict__ dy,
                      float *__restrict__ loss) {
  float acc = 0.0f;
  const float inv = 1.0f / (float)B;
  for (int b = blockIdx.x * blockDim.x + threadIdx.x; b < B; b += gridDim.x * blockDim.x) {
    const float r = y[b] - t[b];
    dy[b] = 2.0f * r * inv;
    acc += r * r * inv;
  }
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_xor(acc, o, 64);
  if ((threadIdx.x & 63) == 0 && loss) atomicAdd(loss, acc);
}

// BF16 copies of W2..W4 live contiguously in w_bf16, layer l's copy at (l - 2) * 65536 in
// fragment order
__device__ __forceinline__ int bf16_slot(int i) {
  for (int l = 2; l <= 4; ++l)
    if (i >= off_w(l) && i < off_w(l) + NW * NW) {
      const int j = i - off_w(l);
      return (l - 2) * NW * NW + wfrag(j / NW, j % NW);
    }
  return -1;
}

__global__ void k_adam(float *__restrict__ p, const float *__restrict__ g, float *__restrict__ m, float *__restrict__ v,
                       int n, float lr, float b1, float b2, float eps, float bc1, float bc2,
                       uint16_t *__restrict__ wbf) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const float gi = g[i];
    const float mi = b1 * m[i] + (1.0f - b1) * gi;
    const float vi = b2 * v[i] + (1.0f - b2) * gi * gi;
    m[i] = mi;
    v[i] = vi;
    const float pi = p[i] - lr * (mi / bc1) / (sqrtf(vi / bc2) + eps);
    p[i] = pi;
    const int s = bf16_slot(i);
    if (s >= 0) wbf[s] = f2bf(pi);
  }
}

__global__ void k_sync_bf16(const float *__restrict__ p, uint16_t *__restrict__ wbf) {
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < 3 * NW * NW; e += gridDim.x * blockDim.x) {
    const int l = 2 + e / (NW * NW), i = e % (NW * NW);
    wbf[(l - 2) * NW * NW + wfrag(i / NW, i % NW)] = f2bf(p[off_w(l) + i]);
  }
}

struct GateBox {
  float lo[NIN], hi[NIN];
};

// Validation error table of the gate: cell (iT, ik) of an nT x nk grid over the trusted
// box's (T, k) rectangle holds the largest |network - SFFT| / S0 seen there.
struct GateCells {
  const float *err;
  int nT, nk;
  float tol;
};

__global__ void k_gate(const float *__restrict__ x, const float *__restrict__ z, int B, GateBox box, float r,
                       float tol, float out_eps, GateCells cells, float *__restrict__ price,
                       int32_t *__restrict__ accept) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  bool ok = true;
#pragma unroll
  for (int i = 0; i < NIN; ++i) {
    const float xi = x[(int64_t)b * NIN + i];
    ok = ok && (xi >= box.lo[i]) && (xi <= box.hi[i]);
  }
  const float T = x[(int64_t)b * NIN + 5], k = x[(int64_t)b * NIN + 6];
  const float lower = fmaxf(0.0f, 1.0f - expf(k - r * T));
  const float yb = out_eps > 0.0f ? expf(z[b]) - out_eps : z[b];
  const float res = fmaxf(fmaxf(lower - yb, yb - 1.0f), 0.0f);
  if (ok && cells.err) {
    // the query's (T, k) cell; in-box queries map into [0, n) (the upper edges clamp)
    const float fT = (T - box.lo[5]) / (box.hi[5] - box.lo[5]), fk = (k - box.lo[6]) / (box.hi[6] - box.lo[6]);
    const int iT = min(cells.nT - 1, max(0, (int)(fT * (float)cells.nT)));
    const int ik = min(cells.nk - 1, max(0, (int)(fk * (float)cells.nk)));
    ok = cells.err[iT * cells.nk + ik] <= cells.tol;
  }
  if (price) price[b] = yb;
  accept[b] = (ok && res <= tol && yb == yb) ? 1 : 0;
}

inline unsigned grid_for(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

}  // namespace

extern "C" size_t cm_mlp_act_bytes(int B) { return B > 0 ? (size_t)4 * B * NW * sizeof(float) : 0; }

static bool net_ok(const cm_mlp *net) { return net && net->params && net->w_bf16; }

extern "C" cm_status cm_mlp_sync_bf16(const cm_mlp *net, void *stream) {
  if (!net_ok(net)) return CM_E_INVALID;
  hipLaunchKernelGGL(k_sync_bf16, dim3(256), dim3(256), 0, (hipStream_t)stream, net->params, net->w_bf16);
  CM_LAUNCH_CHECK();
  return CM_OK;
}

// Inference batches up to this many rows go through tiles of 32 (one workgroup each, 256 at a
// time), larger ones through the kernel with two tiles of 64 in flight per CU: 777 rows take 9.6
// against 27 us, 8192 11.5 against 28, 16384 19 against 29, 24576 28 against 31, 32768 37 against 33.
constexpr int TILE_ROWS_MAX = 24576;

extern "C" cm_status cm_mlp_forward(const cm_mlp *net, const float *x, int B, float *y, float *acts,
                                    size_t acts_bytes, void *stream) {
  if (!net_ok(net) || !x || !y || B < 0) return CM_E_INVALID;
  if (B == 0) return CM_OK;
  if ((int64_t)B * NW > INT32_MAX) return CM_E_UNSUPPORTED;
  const bool keep = acts && acts_bytes >= cm_mlp_act_bytes(B);
  hipStream_t s = (hipStream_t)stream;
  if (keep || B <= TILE_ROWS_MAX) {
    const dim3 grid((B + TM - 1) / TM);
    if (keep) {
      CM_HIP_CHECK(cm_allow_lds(k_mlp_tile<true>, TILE_LDS));
      hipLaunchKernelGGL(k_mlp_tile<true>, grid, dim3(TWG), TILE_LDS, s, x, B, net->params, net->w_bf16, *net, y, acts);
    } else {
      CM_HIP_CHECK(cm_allow_lds(k_mlp_tile<false>, TILE_LDS));
      hipLaunchKernelGGL(k_mlp_tile<false>, grid, dim3(TWG), TILE_LDS, s, x, B, net->params, net->w_bf16, *net, y,
                         (float *)nullptr);
    }
    CM_LAUNCH_CHECK();
    return CM_OK;
  }
  // one persistent workgroup (two tiles in flight) per CU
  CM_HIP_CHECK(cm_allow_lds(k_mlp_fused, FUSED_LDS));
  const int ntiles = (B + FM - 1) / FM;
  int cus = 0;
  int dev = 0;
  CM_HIP_CHECK(hipGetDevice(&dev));
  CM_HIP_CHECK(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
  const int pairs = (ntiles + 1) / 2;
  const int grid = pairs < cus ? pairs : cus;
  hipLaunchKernelGGL(k_mlp_fused, dim3(grid), dim3(512), FUSED_LDS, s, x, B, net->params, net->w_bf16, *net, y);
  CM_LAUNCH_CHECK();
  return CM_OK;
}

extern "C" cm_status cm_mlp_backward(const cm_mlp *net, const float *x, const float *acts, const float *dy, int B,
                                     float *grad, void *ws, size_t ws_bytes, void *stream) {
  if (!net_ok(net) || !x || !acts || !dy || !grad || B < 0) return CM_E_INVALID;
  if (B == 0) return CM_OK;
  if (!ws || ws_bytes < cm_mlp_act_bytes(B) / 2) return CM_E_INVALID;
  hipStream_t s = (hipStream_t)stream;
  float *D = (float *)ws;   // delta_3, delta_2
  uint16_t *wt = grad_scratch(grad);
  CM_HIP_CHECK(cm_allow_lds(k_mlp_bwd, TILE_LDS));
  hipLaunchKernelGGL(k_bwd_prep, dim3((3 * NW * NW / 64 + FIRST_COPIES * FIRST_N) / 256), dim3(256), 0, s, net->w_bf16, wt, grad);
  hipLaunchKernelGGL(k_mlp_bwd, dim3((B + TM - 1) / TM), dim3(TWG), TILE_LDS, s, x, acts, dy, B, net->params, wt, *net,
                     D, grad);
  hipLaunchKernelGGL(k_bwd_mid, dim3(grid_for(CM_MLP_NPARAMS, 256)), dim3(256), 0, s, grad);
  // spans of at least 128 rows, at most WG_SPANS of them: each adds 3 x 65536 gradients by atomics
  int span = (B + WG_SPANS - 1) / WG_SPANS;
  if (span < 128) span = 128;
  span = (span + GKR - 1) / GKR * GKR;
  const int spans = (B + span - 1) / span;
  hipLaunchKernelGGL(k_wgrad, dim3(12 * XCDS * ((spans + XCDS - 1) / XCDS)), dim3(256), 0, s, acts, dy, D, B, span, net->params, grad);
  CM_LAUNCH_CHECK();
  return CM_OK;
}

extern "C" cm_status cm_mlp_mse(const float *y, const float *t, int B, float *dy, float *loss, void *stream) {
  if (!y || !t || !dy || B < 0) return CM_E_INVALID;
  if (B == 0) return CM_OK;
  hipLaunchKernelGGL(k_mse, dim3(grid_for(B, 256) < 1024 ? grid_for(B, 256) : 1024), dim3(256), 0,
                     (hipStream_t)stream, y, t, B, dy, loss);
  CM_LAUNCH_CHECK();
  return CM_OK;
}

extern "C" cm_status cm_adam_step(const cm_mlp *net, const float *grad, float *m, float *v, int step, float lr,
                                  float beta1, float beta2, float eps, void *stream) {
  if (!net_ok(net) || !grad || !m || !v || step < 1) return CM_E_INVALID;
  if (!(beta1 >= 0.0f && beta1 < 1.0f && beta2 >= 0.0f && beta2 < 1.0f && eps > 0.0f)) return CM_E_INVALID;
  const float bc1 = 1.0f - powf(beta1, (float)step), bc2 = 1.0f - powf(beta2, (float)step);
  hipLaunchKernelGGL(k_adam, dim3(grid_for(CM_MLP_NPARAMS, 256)), dim3(256), 0, (hipStream_t)stream, net->params,
                     grad, m, v, (int)CM_MLP_NPARAMS, lr, beta1, beta2, eps, bc1, bc2, net->w_bf16);
  CM_LAUNCH_CHECK();
  return CM_OK;
}

extern "C" cm_status cm_surrogate_gate(const float *x, const float *z, int B, const float *lo, const float *hi,
                                       float r, float res_tol, float out_eps, const float *cell_err, int nT, int nk,
                                       float err_tol, float *price, int32_t *accept, void *stream) {
  if (!x || !z || !lo || !hi || !accept || B < 0 || !(out_eps >= 0.0f)) return CM_E_INVALID;
  if (cell_err && (nT < 1 || nk < 1 || nT > 4096 || nk > 4096 || !(err_tol >= 0.0f))) return CM_E_INVALID;
  if (B == 0) return CM_OK;
  GateBox box;
  for (int i = 0; i < NIN; ++i) {
    box.lo[i] = lo[i];
    box.hi[i] = hi[i];
  }
  if (cell_err && !(box.hi[5] > box.lo[5] && box.hi[6] > box.lo[6])) return CM_E_INVALID;
  GateCells cells{cell_err, nT, nk, err_tol};
  hipLaunchKernelGGL(k_gate, dim3(grid_for(B, 256)), dim3(256), 0, (hipStream_t)stream, x, z, B, box, r, res_tol,
                     out_eps, cells, price, accept);
  CM_LAUNCH_CHECK();
  return CM_OK;
}
