// kernels_block.h -- the rest of one AFNO transformer block around the spectral filter:
// per-token LayerNorm, the channel-mixing MLP (C -> 4C -> C, shared by all tokens, "Model
// Innovations" and "Implementation Details" (c)) as two bf16 matrix-core GEMMs with fused
// epilogues, and the residual adds.  Tokens are the rows of x [B H W][C] (row-major).
//
//   t   = LN1(x)                         layer_norm_kernel (and the weights' transposes)
//   u   = filter(t)  (= t + y(t))         the filter's kernels
//   v   = u + x,  w = LN2(v)              add_layer_norm_kernel
//   h   = GELU(w Wa + ba)                 gemm_dma<kEpiGelu>, or gemm_bf16 for other shapes
//   out = v + h Wb + bb                   gemm_dma<kEpiResidual>
#pragma once
#include "kernel_common.h"
#include "kernels_mfma.h"

namespace afno {

constexpr int kLnMaxPerLane = 32;  // values a lane holds: C <= 64 * 32
constexpr float kLnEps = 1e-6f;

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// LayerNorm of one token's C channels held as vals[0 .. n) by this lane (channels
// 8 (lane + 64 i) .. + 7 for chunk i), two passes over registers; writes bf16.
template <int NCH>
__device__ __forceinline__ void ln_token(float (&vals)[NCH][8], int nchunk, int C, int lane,
                                         const bf16* __restrict__ gamma,
                                         const bf16* __restrict__ beta, bf16* __restrict__ y) {
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i)
    if (lane + 64 * i < nchunk) {
#pragma unroll
      for (int e = 0; e < 8; ++e) s += vals[i][e];
    }
  const float mean = wave_sum(s) / (float)C;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i)
    if (lane + 64 * i < nchunk) {
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const float d = vals[i][e] - mean;
        q += d * d;
      }
    }
  const float rstd = rsqrtf(wave_sum(q) / (float)C + kLnEps);
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int ch = lane + 64 * i;
    if (ch < nchunk) {
      const uint4 gw = *reinterpret_cast<const uint4*>(gamma + 8 * ch);
      const uint4 bw = *reinterpret_cast<const uint4*>(beta + 8 * ch);
      const uint32_t* gu = reinterpret_cast<const uint32_t*>(&gw);
      const uint32_t* bu = reinterpret_cast<const uint32_t*>(&bw);
      uint32_t o[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const float g0 = __uint_as_float(gu[p] << 16), g1 = __uint_as_float(gu[p] & 0xffff0000u);
        const float b0 = __uint_as_float(bu[p] << 16), b1 = __uint_as_float(bu[p] & 0xffff0000u);
        o[p] = cvt_pk((vals[i][2 * p] - mean) * rstd * g0 + b0,
                      (vals[i][2 * p + 1] - mean) * rstd * g1 + b1);
      }
      *reinterpret_cast<uint4*>(y + 8 * ch) = make_uint4(o[0], o[1], o[2], o[3]);
    }
  }
}

__device__ __forceinline__ void unpack8(uint4 w, float (&v)[8]) {
  const uint32_t* u = reinterpret_cast<const uint32_t*>(&w);
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    v[2 * p] = __uint_as_float(u[p] << 16);
    v[2 * p + 1] = __uint_as_float(u[p] & 0xffff0000u);
  }
}

// One 64 x 64 tile of dst[c][r] = src[r][c] for a rows x cols bf16 matrix, both multiples of 64
// (the MLP weights to the GEMM's [N][K] form), by 256 threads.  src may be 2-byte aligned, so it
// is read a value a lane, a whole 128-byte row a wave and 16 rows in flight; dst is written in
// 16-byte words.
__device__ __forceinline__ void transpose_tile(const bf16* __restrict__ src, bf16* __restrict__ dst,
                                               int rows, int cols, int r0, int c0) {
  __shared__ uint16_t t[64][66];
  const uint16_t* s = reinterpret_cast<const uint16_t*>(src);
  const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
  uint16_t v[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) v[i] = s[(int64_t)(r0 + ty + 4 * i) * cols + c0 + tx];
#pragma unroll
  for (int i = 0; i < 16; ++i) t[ty + 4 * i][tx] = v[i];
  __syncthreads();
  const int r = 8 * (threadIdx.x & 7);
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int c = (threadIdx.x >> 3) + 32 * i;
    uint32_t o[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) o[p] = t[r + 2 * p][c] | (uint32_t)t[r + 2 * p + 1][c] << 16;
    *reinterpret_cast<uint4*>(dst + (int64_t)(c0 + c) * rows + r0 + r) = make_uint4(o[0], o[1], o[2], o[3]);
  }
}

// y = LN(x) per token; one wave per token, 4 tokens per 256-thread workgroup.  C a multiple
// of 8, at most 64 * kLnMaxPerLane.  The first 2 ntile workgroups transpose the MLP's weights
// instead, wa [C][4 C] to wat and wb [4 C][C] to wbt, ntile tiles each (C a multiple of 64):
// the weights' 18.9 MB at C = 768 move beside the tokens' 199 MB, both bound by HBM, and the
// launch takes 47.6 us where 41.4 and two transposing launches of 7.2 were (32 x 32 tiles, 2-byte
// stores): the 64,800-token block 980.4 -> 971.8 us, both builds in turn on one card.  First
// rather than last, so that the tokens' workgroups cover the transposes' latency.
__global__ void __launch_bounds__(256) layer_norm_kernel(const bf16* __restrict__ x,
                                                         const bf16* __restrict__ gamma,
                                                         const bf16* __restrict__ beta,
                                                         bf16* __restrict__ y, int64_t M, int C,
                                                         const bf16* __restrict__ wa,
                                                         const bf16* __restrict__ wb,
                                                         bf16* __restrict__ wat,
                                                         bf16* __restrict__ wbt, int ntile) {
  constexpr int NCH = kLnMaxPerLane / 8;
  int g = blockIdx.x;
  if (g < 2 * ntile) {
    const bool second = g >= ntile;
    if (second) g -= ntile;
    const int rows = second ? 4 * C : C, cols = second ? C : 4 * C;
    const int tr = g / (cols / 64), tc = g - tr * (cols / 64);
    transpose_tile(second ? wb : wa, second ? wbt : wat, rows, cols, 64 * tr, 64 * tc);
    return;
  }
  const int lane = threadIdx.x & 63;
  const int64_t tok = (int64_t)(g - 2 * ntile) * 4 + (threadIdx.x >> 6);
  if (tok >= M) return;
  const int nchunk = C / 8;
  const bf16* xr = x + tok * C;
  float vals[NCH][8];
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int ch = lane + 64 * i;
    if (ch < nchunk) unpack8(*reinterpret_cast<const uint4*>(xr + 8 * ch), vals[i]);
  }
  ln_token<NCH>(vals, nchunk, C, lane, gamma, beta, y + tok * C);
}

// v = u + x (rounded to bf16 and stored), w = LN(v) of the stored v; as layer_norm_kernel.
__global__ void __launch_bounds__(256) add_layer_norm_kernel(const bf16* __restrict__ u,
                                                             const bf16* __restrict__ x,
                                                             const bf16* __restrict__ gamma,
                                                             const bf16* __restrict__ beta,
                                                             bf16* __restrict__ v,
                                                             bf16* __restrict__ w, int64_t M, int C) {
  constexpr int NCH = kLnMaxPerLane / 8;
  const int lane = threadIdx.x & 63;
  const int64_t tok = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (tok >= M) return;
  const int nchunk = C / 8;
  float vals[NCH][8];
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int ch = lane + 64 * i;
    if (ch < nchunk) {
      float a[8], b[8];
      unpack8(*reinterpret_cast<const uint4*>(u + tok * C + 8 * ch), a);
      unpack8(*reinterpret_cast<const uint4*>(x + tok * C + 8 * ch), b);
      uint32_t o[4];
#pragma unroll
      for (int p = 0; p < 4; ++p) o[p] = cvt_pk(a[2 * p] + b[2 * p], a[2 * p + 1] + b[2 * p + 1]);
      const uint4 ow = make_uint4(o[0], o[1], o[2], o[3]);
      *reinterpret_cast<uint4*>(v + tok * C + 8 * ch) = ow;
      unpack8(ow, vals[i]);  // LN of the stored (rounded) v
    }
  }
  ln_token<NCH>(vals, nchunk, C, lane, gamma, beta, w + tok * C);
}

enum { kEpiGelu = 0, kEpiResidual = 1 };
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// GELU(z) = z Phi(z).  The lower tail u = Phi(-|z|) = t Q(t) exp(-z^2 / 2), t = 1 / (1 + 0.3 |z|),
// with Q a degree-7 fit to erfcx(|z| / sqrt 2) / (2 t) on |z| <= 9 (least squares reweighted to a
// minimax relative error of 5e-8); then z - |z| u above zero and z u below.  Against float64 the
// result, in single precision, is within 7e-7 of its own size for z > -3 and 7e-6 from there to
// -12.9 (a model in float32 of every step: 4.4e-7 and 6.7e-6; the fit reaches past its 9), and within
// 2e-37 below, where the exponential leaves the normal numbers; 0.5 z (1 + erf) has 1e-7 to 2e-7
// for |z| < 1, and below loses all digits by z = -6 to the subtraction.  About 25 issue slots a value where erff takes over 60: the epilogue's
// values are the exposed part of the first product (64,800 x 3072 x 768: 426 us with erff, 387
// with this, 320 without any).  |z| is bounded in the tail only (z = +inf gives +inf; -inf and NaN
// give NaN, as z Phi(z) does).
__device__ __forceinline__ float gelu(float z) {
  const float a = fminf(fabsf(z), 16.f);
  const float t = __builtin_amdgcn_rcpf(__builtin_fmaf(0.3f, a, 1.f));
  float q = 0.037535712f;
  q = __builtin_fmaf(q, t, -0.16501968f);
  q = __builtin_fmaf(q, t, 0.21997128f);
  q = __builtin_fmaf(q, t, -0.06640263f);
  q = __builtin_fmaf(q, t, 0.13542020f);
  q = __builtin_fmaf(q, t, 0.097783938f);
  q = __builtin_fmaf(q, t, 0.1211057f);
  q = __builtin_fmaf(q, t, 0.11960549f);
  const float e = __builtin_amdgcn_exp2f(a * a * -0.72134752f);  // exp(-a^2 / 2)
  const float u = t * q * e;
  return z > 0.f ? __builtin_fmaf(-a, u, z) : z * u;
}

// GEMM geometry of the register-staged kernel (column counts N that are not a multiple of
// 256): workgroup tile 256 x BN (rows x columns of D), k-stage 64 (two MFMA k-steps per
// barrier); 4 x (BN / 64) waves, each 64 x 64 (4 x 4 MFMA tiles of 16 x 16).  LDS: two stages
// of the A (256 x 64) and B (BN x 64) slabs, rows padded to 72 elements; the epilogue reuses
// it for 64 rows of fp32 at a time.
template <int BN>
struct GemmGeo {
  static constexpr int BM = 256, BK = 64, LDK = BK + 8;
  static constexpr int NWN = BN / 64, NT = 64 * 4 * NWN;    // threads
  static constexpr int ASLAB = BM * LDK, BSLAB = BN * LDK;
  static constexpr int STAGE = ASLAB + BSLAB;               // elements
  static constexpr int LDC = BN + 4;                         // epilogue stride, floats
  static constexpr int kLA = BM * (BK / 8) / NT, kLB = BN * (BK / 8) / NT;  // words per thread
  static constexpr int kBytes = 2 * STAGE * 2 > 64 * LDC * 4 ? 2 * STAGE * 2 : 64 * LDC * 4;
  static_assert(BM * (BK / 8) % NT == 0 && BN * (BK / 8) % NT == 0, "whole words per thread");
};

// D[M][N] = epi(A[M][K] Bt[N][K]^T + bias[N]) in bf16, fp32 accumulation on the matrix cores.
// The next k-stage's global loads are in flight during the current stage's products.
// Epilogue: + bias staged through LDS in fp32 (64 rows at a time), then, on the way out to
// row-contiguous stores, GELU (kEpiGelu) or + R[M][N] (kEpiResidual).  Rows of A past M are read clamped and never
// stored.  Tiles go XCD-aware: workgroup g runs on XCD g % 8 and the workgroups of one XCD
// take all column tiles of a row tile in turn, so that row tile's A stays in that XCD's L2.
// N a multiple of BN, K a multiple of 64; grid 8 ceil(MB / 8) (N / BN) with MB = ceil(M / 256);
// GemmGeo<BN>::NT threads; dynamic LDS GemmGeo<BN>::kBytes.
template <int EPI, int BN>
__global__ void __launch_bounds__(GemmGeo<BN>::NT) gemm_bf16(const bf16* __restrict__ A,
                                                             const bf16* __restrict__ Bt,
                                                             const bf16* __restrict__ bias,
                                                             const bf16* __restrict__ R,
                                                             bf16* __restrict__ D, int M, int N,
                                                             int K) {
  typedef GemmGeo<BN> G;
  extern __shared__ uint4 gemm_smem[];
  bf16* S = reinterpret_cast<bf16*>(gemm_smem);           // [2][STAGE]: A slab, then B slab
  float* sC = reinterpret_cast<float*>(gemm_smem);        // [64][LDC] in the epilogue

  const int nbn = N / BN;
  const int g = blockIdx.x, xcd = g & 7, i = g >> 3;
  const int mb = (i / nbn) * 8 + xcd, nbk = i - (i / nbn) * nbn;
  const int m0 = mb * G::BM, n0 = nbk * BN;
  if (m0 >= M) return;  // padding workgroups: the whole group leaves before any barrier

  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, gq = lane >> 4;
  const int wave = tid >> 6, wm = wave / G::NWN, wn = wave % G::NWN;
  // global -> LDS: thread tid moves k-word tid % 8 of rows tid / 8 + RS j (A: kLA rows, B: kLB)
  constexpr int WPR = G::BK / 8, RS = G::NT / WPR;
  const int r4 = tid / WPR, kc = 8 * (tid % WPR);
  const bf16* srcB = Bt + (int64_t)(n0 + r4) * K + kc;
  int64_t aoff[G::kLA];
#pragma unroll
  for (int j = 0; j < G::kLA; ++j) aoff[j] = (int64_t)min(m0 + r4 + RS * j, M - 1) * K + kc;
  const int dA = r4 * G::LDK + kc, dB = G::ASLAB + r4 * G::LDK + kc;
  f32x4 acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};

  const int stages = K / G::BK;
  {
    uint4 ra[G::kLA], rb[G::kLB];
#pragma unroll
    for (int j = 0; j < G::kLA; ++j) ra[j] = *reinterpret_cast<const uint4*>(A + aoff[j]);
#pragma unroll
    for (int j = 0; j < G::kLB; ++j)
      rb[j] = *reinterpret_cast<const uint4*>(srcB + (int64_t)RS * j * K);
#pragma unroll
    for (int j = 0; j < G::kLA; ++j) *reinterpret_cast<uint4*>(S + dA + RS * j * G::LDK) = ra[j];
#pragma unroll
    for (int j = 0; j < G::kLB; ++j) *reinterpret_cast<uint4*>(S + dB + RS * j * G::LDK) = rb[j];
  }
  __syncthreads();
  for (int s = 0; s < stages; ++s) {
    const int buf = s & 1;
    // the next stage's words (the last stage reloads its own: loads and stores unconditional)
    const int kn = (s + 1 < stages ? s + 1 : s) * G::BK;
    uint4 na[G::kLA], nb_[G::kLB];
#pragma unroll
    for (int j = 0; j < G::kLA; ++j) na[j] = *reinterpret_cast<const uint4*>(A + aoff[j] + kn);
#pragma unroll
    for (int j = 0; j < G::kLB; ++j)
      nb_[j] = *reinterpret_cast<const uint4*>(srcB + (int64_t)RS * j * K + kn);
    const bf16* cA = S + buf * G::STAGE + (64 * wm + l16) * G::LDK + 8 * gq;
    const bf16* cB = S + buf * G::STAGE + G::ASLAB + (64 * wn + l16) * G::LDK + 8 * gq;
#pragma unroll
    for (int kk = 0; kk < G::BK; kk += 32) {
      uint4 fa[4], fb[4];
#pragma unroll
      for (int a = 0; a < 4; ++a)
        fa[a] = *reinterpret_cast<const uint4*>(cA + 16 * a * G::LDK + kk);
#pragma unroll
      for (int b = 0; b < 4; ++b)
        fb[b] = *reinterpret_cast<const uint4*>(cB + 16 * b * G::LDK + kk);
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) acc[a][b] = mma_bf16(fa[a], fb[b], acc[a][b]);
    }
    bf16* nS = S + (buf ^ 1) * G::STAGE;
#pragma unroll
    for (int j = 0; j < G::kLA; ++j) *reinterpret_cast<uint4*>(nS + dA + RS * j * G::LDK) = na[j];
#pragma unroll
    for (int j = 0; j < G::kLB; ++j) *reinterpret_cast<uint4*>(nS + dB + RS * j * G::LDK) = nb_[j];
    __syncthreads();
  }

  // ---- epilogue, one wave row (64 rows) at a time
  float bv[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) bv[b] = (float)bias[n0 + 64 * wn + 16 * b + l16];
  constexpr int C4 = BN / 4;              // groups of 4 columns per row
  constexpr int PER = 64 * C4 / G::NT;    // groups per thread
#pragma unroll 1
  for (int part = 0; part < 4; ++part) {
    if (wm == part) {
#pragma unroll
      for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            sC[(16 * a + 4 * gq + q) * G::LDC + 64 * wn + 16 * b + l16] = acc[a][b][q] + bv[b];
          }
    }
    __syncthreads();
#pragma unroll 1
    for (int j = 0; j < PER; ++j) {
      const int c = tid + G::NT * j;
      const int r = c / C4, c4 = 4 * (c - (c / C4) * C4);
      const int row = m0 + 64 * part + r;
      if (row < M) {
        const float4 z = *reinterpret_cast<const float4*>(sC + r * G::LDC + c4);
        float o0 = z.x, o1 = z.y, o2 = z.z, o3 = z.w;
        if constexpr (EPI == kEpiGelu) {
          o0 = gelu(o0);
          o1 = gelu(o1);
          o2 = gelu(o2);
          o3 = gelu(o3);
        }
        const int64_t off = (int64_t)row * N + n0 + c4;
        if constexpr (EPI == kEpiResidual) {
          const uint2 rw = *reinterpret_cast<const uint2*>(R + off);
          o0 += __uint_as_float(rw.x << 16);
          o1 += __uint_as_float(rw.x & 0xffff0000u);
          o2 += __uint_as_float(rw.y << 16);
          o3 += __uint_as_float(rw.y & 0xffff0000u);
        }
        *reinterpret_cast<uint2*>(D + off) = make_uint2(cvt_pk(o0, o1), cvt_pk(o2, o3));
      }
    }
    __syncthreads();
  }
}

// The same product with the k-stages moved by the direct-to-LDS loads (global_load_lds_dwordx4:
// each lane's 16 bytes go straight into the LDS, no registers or LDS store instructions in
// between), so that three stages can be in flight during the current one's products.
// Workgroup tile 256 x 256, 32-deep k-stages in a ring of four LDS stages (A slab 256 x 32,
// then B slab 256 x 32, 32 KB each), 16 waves as 4 x 4 of 64 x 64.  Slab rows are 64 bytes
// (four 16-byte chunks) without padding; chunk c of row r sits at position c ^ 2((r / 8) % 2) in
// the A slab and c ^ ((r / 8) % 4) in the B slab, so that the rows a pass of ds_read_b128 takes
// (A: 16 consecutive ones; B: four groups of four, eight apart) cover the banks once.  A wave's
// load moves 16 consecutive rows (lane i: row i / 4, position i % 4).
// The four stages are separate arrays: the compiler then sees that a stage being read is not
// one whose loads are still in flight, and the loop waits on exactly the current stage's loads
// (per wave: two loads per stage, in issue order).  The loads of the last stages' successors
// re-read the last stage into a buffer nobody reads, so every wait counts the same.
// The products are taken transposed and B's rows are dealt to the tiles so that a lane ends up
// with eight consecutive columns of a row twice: the epilogue needs no LDS and no barrier, each
// wave adds the bias, applies GELU or the residual and stores 64 contiguous bytes of 16 rows at
// a time (staged in LDS, 64 rows of the workgroup after each other: 438 us for the first product
// of 64,800 tokens at C = 768, direct 426; 32-byte pieces 488; without the non-temporal hint
// 448).  Measured and not kept: one persistent workgroup per compute unit with the next tile's
// first stages loaded under the epilogue (390 against 387 us).
// N a multiple of 256, K a multiple of 128; grid 8 ceil(MB / 8) (N / 256), 1024 threads, no
// dynamic LDS.
__shared__ uint4 gd_stage0[2048];
__shared__ uint4 gd_stage1[2048];
__shared__ uint4 gd_stage2[2048];
__shared__ uint4 gd_stage3[2048];

template <int EPI>
__global__ void __launch_bounds__(1024) gemm_dma(const bf16* __restrict__ A,
                                                 const bf16* __restrict__ Bt,
                                                 const bf16* __restrict__ bias,
                                                 const bf16* __restrict__ R,
                                                 bf16* __restrict__ D, int M, int N, int K) {
  constexpr int BM = 256, BN = 256, BK = 32;
  const int nbn = N / BN;
  const int g = blockIdx.x, xcd = g & 7, i = g >> 3;
  const int mb = (i / nbn) * 8 + xcd, nbk = i - (i / nbn) * nbn;
  const int m0 = mb * BM, n0 = nbk * BN;
  if (m0 >= M) return;  // padding workgroups: the whole group leaves before any barrier

  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, gq = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), wm = wave >> 2, wn = wave & 3;
  const int S = K / BK;
  // this lane's loads: row 16 wave + lane / 4 of both slabs, the chunk that belongs at
  // position lane % 4 there (A: swizzle 2 ((r / 8) % 2); B: (r / 8) % 4)
  const int lr = lane >> 2;
  const int lca = (lane & 3) ^ (2 * ((lr >> 3) & 1)), lcb = (lane & 3) ^ ((2 * wave + (lr >> 3)) & 3);
  const bf16* ga = A + (int64_t)min(m0 + 16 * wave + lr, M - 1) * K + 8 * lca;
  const bf16* gb = Bt + (int64_t)(n0 + 16 * wave + lr) * K + 8 * lcb;
  // this lane's operand slots: A row l16 of a 16-row group; B row 8 (l16 / 4) + l16 % 4 of the
  // wave's 64, to which tile b adds 32 (b / 2) + 4 (b % 2); chunk gq of each
  const int fa_s = 4 * l16 + (gq ^ (2 * ((l16 >> 3) & 1)));
  const int fb_s = 4 * (8 * (l16 >> 2) + (l16 & 3)) + (gq ^ (l16 >> 2));

  auto issue = [&](uint4* st, int s) {
    const int64_t kk = (int64_t)(s < S ? s : S - 1) * BK;
    __builtin_amdgcn_global_load_lds(ga + kk, st + 64 * wave, 16, 0, 0);
    __builtin_amdgcn_global_load_lds(gb + kk, st + 1024 + 64 * wave, 16, 0, 0);
  };
  f32x4 acc[4][4];
#pragma unroll
  for (int a = 0; a < 4; ++a)
#pragma unroll
    for (int b = 0; b < 4; ++b) acc[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](const uint4* st) {
    uint4 fa[4], fb[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) fa[a] = st[(4 * wm + a) * 64 + fa_s];
#pragma unroll
    for (int b = 0; b < 4; ++b) fb[b] = st[1024 + 256 * wn + 128 * (b / 2) + 16 * (b % 2) + fb_s];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
      for (int b = 0; b < 4; ++b) acc[a][b] = mma_bf16(fb[b], fa[a], acc[a][b]);
  };
  // this wave's loads of the current stage done (the two later stages' four loads may still
  // be in flight), then every wave's: the barrier also tells that the stage read last is free
  auto sync = [&]() {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0x0f74);  // vmcnt(4), no wait on the other counters
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  issue(gd_stage0, 0);
  issue(gd_stage1, 1);
  issue(gd_stage2, 2);
  for (int s = 0; s < S; s += 4) {
    sync();
    issue(gd_stage3, s + 3);
    compute(gd_stage0);
    sync();
    issue(gd_stage0, s + 4);
    compute(gd_stage1);
    sync();
    issue(gd_stage1, s + 5);
    compute(gd_stage2);
    sync();
    issue(gd_stage2, s + 6);
    compute(gd_stage3);
  }
  // the three surplus loads land before the workgroup's LDS can pass to another
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
  asm volatile("" ::: "memory");

  // ---- epilogue, each wave on its own: this lane's columns n .. n + 7 and
  //      n + 32 .. n + 39 of rows m0 + .. + l16 (a store covers 64 bytes of each row)
  const int n = n0 + 64 * wn + 8 * gq;
  float bv[16];
#pragma unroll
  for (int e = 0; e < 16; ++e) bv[e] = (float)bias[n + 32 * (e / 8) + e % 8];
#pragma unroll
  for (int a = 0; a < 4; ++a) {
    const int row = m0 + 64 * wm + 16 * a + l16;
    if (row >= M) continue;
    const int64_t off = (int64_t)row * N + n;
    // streamed once: non-temporal, so that the output and residual streams do not push the
    // operands' k-slices out of the caches
    u32x4 rv[2];
    if constexpr (EPI == kEpiResidual) {
      rv[0] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(R + off));
      rv[1] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(R + off + 32));
    }
#pragma unroll
    for (int h = 0; h < 2; ++h) {  // eight columns: tiles 2 h and 2 h + 1
      float o[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        o[e] = acc[a][2 * h + e / 4][e % 4] + bv[8 * h + e];
        if constexpr (EPI == kEpiGelu)
          o[e] = gelu(o[e]);
        if constexpr (EPI == kEpiResidual)
          o[e] += e % 2 ? __uint_as_float(rv[h][e / 2] & 0xffff0000u) : __uint_as_float(rv[h][e / 2] << 16);
      }
      const u32x4 w = {cvt_pk(o[0], o[1]), cvt_pk(o[2], o[3]), cvt_pk(o[4], o[5]), cvt_pk(o[6], o[7])};
      __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(D + off + 32 * h));
    }
  }
}

}  // namespace afno
