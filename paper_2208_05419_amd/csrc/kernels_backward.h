// kernels_backward.h -- the AFNO filter's backward pass on gfx950.
//
// For an upstream gradient g = dL/dout the filter's transpose runs the forward steps in
// reverse ("Model Innovations", steps 1-3; the paper trains through them, "Implementation
// Details" (a), (e)).  With F the 2-D real DFT (W-axis R2C then H-axis DFT, ortho), G its
// half-spectrum inverse (H-axis inverse DFT then W-axis C2R with weights c_kw = 1 at kw = 0
// and W/2, else 2) and the per-mode block MLP v = X W1 + b1, h = relu(v), o = h W2 + b2,
// z = S_lam(o) (componentwise on re and im, zero outside the cutoff), y = G(z):
//
//   dz  = c_kw F(g)                       (G's transpose: the weighted C2R's is c_kw R2C,
//                                          the unitary inverse H-DFT's the forward H-DFT)
//   do  = dz where |o| > lam and the mode is kept, else 0   (componentwise)
//   dh  = do W2^H,   dv = dh where v > 0, else 0
//   dX  = dv W1^H
//   dx  = g + G(dX / c_kw)                (F's transpose: C2R with unit weights)
//   dW1 = sum over modes conj(X)^T dv,  db1 = sum dv;  dW2 = sum conj(h)^T do,  db2 = sum do
//
// Passes: the forward W-axis kernel on x and on g (spectra Sx, Sg); a backward column kernel
// per (b, kw, block) recomputes X, h and both masks, transforms the gradient column and runs
// the two conjugate-transposed products, writing dX's inverse back into Sg and the per-mode
// factors X, h, do, dv to HBM in 8-mode groups; a weight-product kernel (wgrad_slab for bf16
// with 2 bs in {64, 128, 192}, else wgrad_kernel) forms the weight and bias gradients from the
// factors on the matrix cores as chunk sums, which wgrad_finalize_parts adds in a fixed order
// (no floating-point atomics: repeated calls give the same bits); the forward W-axis inverse kernel
// with g as its residual gives dx.  This header
// holds the weight products; kernels_column.h the size-generic column kernel (any dtype,
// H <= 192), kernels_backward_mfma.h the bf16 one for H <= 96 with the H transforms on the
// matrix cores.
#pragma once
#include "kernels_column.h"
#include "kernels_mfma.h"

namespace afno {

template <typename T>
__global__ void __launch_bounds__(256) fill_zero_f32(float* __restrict__ p, int64_t n) {
  for (int64_t t = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; t < n;
       t += (int64_t)gridDim.x * blockDim.x)
    p[t] = 0.f;
}

// Weight-gradient products over all modes: for layer 0 (dW1) A = X, B = dv; for layer 1
// (dW2) A = h, B = do; part[chunk][layer][blk][r][s] = sum over the chunk's modes of
// A[r][m] B[s][m] (r, s the 2 bs real entries, (c, rho) interleaved), and
// bpart[chunk][layer][blk][s] = sum of B[s][m] (the bias gradients db1, db2): plain stores,
// one wave per output value and chunk, summed over the chunks by wgrad_finalize_parts in
// chunk order, so repeated calls give the same bits.
//
// A wave owns a 32 x 32 output tile (2 bs is a multiple of 32: no ragged tile) over one chunk
// of kchunk modes (a multiple of 32), 32 modes a step, the next step's words in flight during
// the current products; there is no barrier, so waves only wait for their own loads.  Every
// load is 16 bytes per lane.  In fp32 lane group g loads modes 4 g .. 4 g + 3 of 16 and feeds
// value j of the four to the j-th matrix instruction: the product sums over the modes, so any
// order serves as long as both operands take the same one.  What bounds it is the operands'
// trip through the caches (each is read by 2 bs / 32 waves) and, with few chunks, latency:
// 72 x 144 x 384 fp32 (8 blocks of 48, 7,008 modes): 400 us as 128 workgroups of 64 x 64 tiles
// with 4-byte loads and 2 chunks, 32 us as 4,032 waves in 28 chunks.
// grid (ceil(2 nb (2 bs / 32)^2 / 4), nchunk = ceil(mpad / kchunk)), 256 threads.
template <typename T>
__global__ void __launch_bounds__(256) wgrad_kernel(const T* __restrict__ modes, int64_t mpad,
                                                    int nb, int bs, int kchunk,
                                                    float* __restrict__ part,
                                                    float* __restrict__ bpart) {
  typedef Mma<T> M;
  constexpr int LD = sizeof(T) == 2 ? 1 : 2;  // 16-byte loads per 16 entries and 32 modes
  const int nb2 = 2 * bs, nt = nb2 / 32;
  int g = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (g >= 2 * nb * nt * nt) return;
  const int ts = g % nt; g /= nt;
  const int tr = g % nt; g /= nt;
  const int blk = g % nb;
  const int layer = g / nb;  // 0: dW1, 1: dW2
  const int lane = threadIdx.x & 63, l16 = lane & 15, gq = lane >> 4;
  const int r0 = 32 * tr, s0 = 32 * ts;
  const int64_t k0 = (int64_t)blockIdx.y * kchunk;
  const int64_t k1 = k0 + kchunk < mpad ? k0 + kchunk : mpad;
  // this lane's word of step 0: bf16 the eight modes of group gq; fp32 half gq % 2 of group
  // gq / 2 (its second load: two groups on)
  const int64_t grp = (k0 >> 3) + (sizeof(T) == 2 ? gq : gq >> 1);
  const int half = sizeof(T) == 2 ? 0 : 4 * (gq & 1);
  const T* A = modes + (((int64_t)(layer ? kModeH : kModeX) * nb + blk) * mpad / 8 + grp) * nb2 * 8 +
               (r0 + l16) * 8 + half;
  const T* Bm = modes + (((int64_t)(layer ? kModeDo : kModeDv) * nb + blk) * mpad / 8 + grp) * nb2 * 8 +
                (s0 + l16) * 8 + half;
  const int64_t step = (int64_t)4 * nb2 * 8;  // 32 modes
  const int sub = 2 * nb2 * 8;                // fp32: the second 16 modes
  f32x4 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  float bsum[2] = {0.f, 0.f};
  V16 a[2][LD], b[2][LD];
  auto load = [&](V16 (&pa)[2][LD], V16 (&pb)[2][LD]) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < LD; ++q) {
        pa[i][q].u = *reinterpret_cast<const uint4*>(A + 16 * 8 * i + q * sub);
        pb[i][q].u = *reinterpret_cast<const uint4*>(Bm + 16 * 8 * i + q * sub);
      }
    A += step;
    Bm += step;
  };
  load(a, b);
  for (int64_t k = k0; k < k1; k += 32) {
    V16 an[2][LD], bn[2][LD];
    if (k + 32 < k1) load(an, bn);
#pragma unroll
    for (int q = 0; q < LD; ++q) {
      if constexpr (sizeof(T) == 2) {
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < 2; ++j) acc[i][j] = mma_bf16(a[i][q].u, b[j][q].u, acc[i][j]);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j) acc[i][j] = M::mma(a[i][q].f[e], b[j][q].f[e], acc[i][j]);
      }
      if (tr == 0) {  // the waves of the first row tile also sum their B words
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          float s = 0.f;
          if constexpr (sizeof(T) == 2) {
#pragma unroll
            for (int e = 0; e < 8; ++e) s += (float)b[j][q].h[e];
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) s += b[j][q].f[e];
          }
          bsum[j] += s;
        }
      }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int q = 0; q < LD; ++q) {
        a[i][q] = an[i][q];
        b[i][q] = bn[i][q];
      }
  }
  const int64_t slot = ((int64_t)blockIdx.y * 2 + layer) * nb + blk;
  if (tr == 0) {
    // the four lane groups hold different modes of the same entry: a fixed butterfly
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      float v = bsum[j];
      v += __shfl_xor(v, 16);
      v += __shfl_xor(v, 32);
      if (gq == 0) bpart[slot * nb2 + s0 + 16 * j + l16] = v;
    }
  }
  float* out = part + slot * nb2 * nb2;
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        out[(int64_t)(r0 + 16 * i + 4 * gq + q) * nb2 + s0 + 16 * j + l16] = acc[i][j][q];
}

// bf16 weight-gradient products for 2 bs = NB2 a multiple of 64: one workgroup per (layer,
// block, mode chunk) computes the chunk's whole NB2 x NB2 product, so each per-mode operand is
// read from HBM once.  Per 64-mode step the two operand slabs (8 mode groups x NB2 entries x
// 16 bytes each) stream through LDS, double buffered; the global loads of the two following
// steps are in flight (in registers) during the current step's products, so that a workgroup
// keeps two steps' bytes on the way from HBM.  16 waves as 4 x 4, each (NB2 / 64)^2 output
// tiles of 16 x 16 (one workgroup per compute unit).  Words beyond the chunk's modes read 0
// (buffer range check).  The chunk's sums go to part[chunk][layer][blk][r][s] (plain stores).
// The same pass sums the second operand over the chunk's modes (do for dW2, dv for dW1: the
// bias gradients db2, db1): each thread adds up the words it moves, in step order, and the
// eight mode groups of an entry are added in a fixed order at the end, to
// bpart[chunk][layer][blk][entry] -- so no atomics, and repeated calls give the same bits.
// grid 2 nb nchunk (layer, block, chunk with block fastest), 1024 threads, dynamic LDS
// 2 * 2 * 8 * NB2 * 16 bytes; kchunk a multiple of 64.
template <int NB2>
__global__ void __launch_bounds__(1024) wgrad_slab(const bf16* __restrict__ modes, int64_t mpad,
                                                   int nb, int kchunk, float* __restrict__ part,
                                                   float* __restrict__ bpart) {
  constexpr int T = NB2 / 64;       // output tiles per wave along each axis
  constexpr int SLAB = 8 * NB2;     // 16-byte words per operand and step
  constexpr int LW = 2 * SLAB / 1024;  // words each thread moves per step
  static_assert(SLAB % 64 == 0 && 2 * SLAB % 1024 == 0, "operand uniform per wave, whole words");
  extern __shared__ uint4 slab_lds[];  // [2 buffers][2 operands][SLAB]
  const int tid = threadIdx.x, lane = tid & 63, l16 = lane & 15, gq = lane >> 4;
  const int wave = tid >> 6, wr = wave >> 2, wc = wave & 3;
  int g = blockIdx.x;
  const int blk = g % nb;
  g /= nb;
  const int layer = g & 1;
  const int chunk = g >> 1;
  const int64_t k0 = (int64_t)chunk * kchunk;
  const int64_t k1 = k0 + kchunk < mpad ? k0 + kchunk : mpad;
  const int steps = (int)((k1 - k0 + 63) / 64);
  // the chunk's words of each operand: groups k0 / 8 .. k1 / 8, NB2 words each
  const uint32_t cbytes = buf_bytes((uint64_t)(k1 - k0) / 8 * NB2 * 16);
  const int64_t cw = (k0 >> 3) * NB2;
  const Buf ra(reinterpret_cast<const uint4*>(
                   modes + ((int64_t)(layer ? kModeH : kModeX) * nb + blk) * NB2 * mpad) + cw,
               cbytes);
  const Buf rb(reinterpret_cast<const uint4*>(
                   modes + ((int64_t)(layer ? kModeDo : kModeDv) * nb + blk) * NB2 * mpad) + cw,
               cbytes);
  // word w = tid + 1024 i of a step: operand w / SLAB (uniform per wave), word w % SLAB of
  // that operand's slab, which starts 8 NB2 words further on each step
  uint32_t voff[LW];
  bool opb[LW];
#pragma unroll
  for (int i = 0; i < LW; ++i) {
    const int w = tid + 1024 * i;
    opb[i] = __builtin_amdgcn_readfirstlane(w / SLAB) != 0;
    voff[i] = (uint32_t)(w % SLAB) * 16u;
  }
  auto load = [&](uint4 (&r)[LW], int s) {
    // the step's offset goes into the per-lane offset, which the range check covers; the factors
  // are read once (non-temporal loads keep them from displacing other data in the caches)
    const uint32_t so = (uint32_t)s * (uint32_t)(SLAB * 16);
#pragma unroll
    for (int i = 0; i < LW; ++i) {
      const auto v = __builtin_amdgcn_raw_buffer_load_b128(opb[i] ? rb.r : ra.r, voff[i] + so, 0,
                                                            kNonTemporal);
      r[i] = make_uint4(v[0], v[1], v[2], v[3]);
    }
  };
  // per word moved: the sum of its eight modes, over all steps (used for the second operand)
  float bsum[LW];
#pragma unroll
  for (int i = 0; i < LW; ++i) bsum[i] = 0.f;
  auto stash = [&](const uint4 (&r)[LW], int buf) {
#pragma unroll
    for (int i = 0; i < LW; ++i) {
      slab_lds[buf * 2 * SLAB + tid + 1024 * i] = r[i];
      if (opb[i]) {  // wave-uniform
        const uint32_t v[4] = {r[i].x, r[i].y, r[i].z, r[i].w};
        float s8 = 0.f;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          s8 += __uint_as_float(v[q] << 16) + __uint_as_float(v[q] & 0xffff0000u);
        bsum[i] += s8;
      }
    }
  };
  f32x4 acc[T][T];
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto compute = [&](int buf) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const uint4* LA = slab_lds + buf * 2 * SLAB + (4 * kk + gq) * NB2 + l16;
      const uint4* LB = LA + SLAB;
      uint4 a[T], b[T];
#pragma unroll
      for (int i = 0; i < T; ++i) a[i] = LA[16 * (wr * T + i)];
#pragma unroll
      for (int j = 0; j < T; ++j) b[j] = LB[16 * (wc * T + j)];
#pragma unroll
      for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j) acc[i][j] = mma_bf16(a[i], b[j], acc[i][j]);
    }
  };
  if (steps > 0) {
    // two register sets take turns, so that no step's words are copied between registers;
    // the steps run in pairs (a step past the chunk reads zeros and adds nothing).  The
    // scheduling barriers keep each step's loads issued before the products they overlap.
    uint4 r0[LW], r1[LW];
    load(r0, 0);
    load(r1, 1);
    stash(r0, 0);
    __syncthreads();
    for (int s = 0; s < steps; s += 2) {
      load(r0, s + 2);  // buffer 0 was read last in step s
      __builtin_amdgcn_sched_barrier(0);
      compute(0);
      stash(r1, 1);
      __syncthreads();
      load(r1, s + 3);
      __builtin_amdgcn_sched_barrier(0);
      compute(1);
      stash(r0, 0);
      __syncthreads();
    }
  }
  // bias sums: word (group, entry) of the second operand's slab -> LDS, then per entry the
  // eight groups in order (the slabs are no longer read: every product is behind a barrier)
  __syncthreads();
  float* red = reinterpret_cast<float*>(slab_lds);
#pragma unroll
  for (int i = 0; i < LW; ++i)
    if (opb[i]) red[(tid + 1024 * i) % SLAB] = bsum[i];
  __syncthreads();
  if (tid < NB2) {
    float sb = 0.f;
#pragma unroll
    for (int q = 0; q < 8; ++q) sb += red[q * NB2 + tid];
    bpart[(((int64_t)chunk * 2 + layer) * nb + blk) * NB2 + tid] = sb;
  }
  float* out = part + (((int64_t)chunk * 2 + layer) * nb + blk) * NB2 * NB2;
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j) {
      const int col = 16 * (wc * T + j) + l16;
#pragma unroll
      for (int q = 0; q < 4; ++q) out[(16 * (wr * T + i) + 4 * gq + q) * NB2 + col] = acc[i][j][q];
    }
}

// dW (re, im) from the weight-product kernels' chunk sums part[chunk][2][nb][2 bs][2 bs]: for
// entries r = (i, rho), s = (j, sigma), dW[i][j] = (P[(i,0)][(j,0)] + P[(i,1)][(j,1)],
// P[(i,0)][(j,1)] - P[(i,1)][(j,0)]) (conj(a) b summed); db1, db2 from the chunk bias sums
// bpart[chunk][2][nb][2 bs].  A call has few outputs (37 thousand for 8 blocks of 48) and up to
// 128 chunks, so it is bound by the loads in flight: wave w of a workgroup's four adds up chunks
// w, w + 4, ... of the workgroup's 64 outputs, in that order, and the four sums are added in
// order (28 chunks of 8 blocks of 48: 11.8 us with one thread per output, 6.2 us).  Grid
// 2 nb bs^2 / 64 (bs is a multiple of 16), 256 threads.
__global__ void __launch_bounds__(256) wgrad_finalize_parts(const float* __restrict__ part,
                                                            int nchunk, const float* __restrict__ bpart,
                                                            int nb, int bs, float* __restrict__ dw1,
                                                            float* __restrict__ dw2,
                                                            float* __restrict__ db1,
                                                            float* __restrict__ db2) {
  __shared__ float sre[4][64], sim[4][64], sbias[4][64];
  const int nb2 = 2 * bs;
  const int64_t n = (int64_t)nb * bs * bs;
  const int64_t nbias = (int64_t)nb * nb2;
  const int64_t cstride = (int64_t)2 * nb * nb2 * nb2;
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t t = (int64_t)blockIdx.x * 64 + l;  // < 2 n
  const int layer = t >= n ? 1 : 0;
  const int64_t u = t - layer * n;
  const int64_t k = u / ((int64_t)bs * bs);
  const int r = (int)(u - k * bs * bs), i = r / bs, j = r % bs;
  const float* P = part + ((int64_t)layer * nb + k) * nb2 * nb2 + (2 * i) * nb2 + 2 * j + w * cstride;
  float rr = 0.f, ii = 0.f, ri = 0.f, ir = 0.f;
#pragma unroll 4
  for (int c = w; c < nchunk; c += 4, P += 4 * cstride) {
    const float2 p0 = *reinterpret_cast<const float2*>(P);
    const float2 p1 = *reinterpret_cast<const float2*>(P + nb2);
    rr += p0.x;
    ri += p0.y;
    ir += p1.x;
    ii += p1.y;
  }
  sre[w][l] = rr + ii;
  sim[w][l] = ri - ir;
  if (t < 2 * nbias) {
    float sb = 0.f;
    for (int c = w; c < nchunk; c += 4) sb += bpart[(int64_t)c * 2 * nbias + t];
    sbias[w][l] = sb;
  }
  __syncthreads();
  if (w != 0) return;
  float* d = (layer ? dw2 : dw1) + ((k * bs + i) * bs + j) * 2;
  d[0] = ((sre[0][l] + sre[1][l]) + sre[2][l]) + sre[3][l];
  d[1] = ((sim[0][l] + sim[1][l]) + sim[2][l]) + sim[3][l];
  if (t < 2 * nbias) {
    const float sb = ((sbias[0][l] + sbias[1][l]) + sbias[2][l]) + sbias[3][l];
    (t < nbias ? db1 : db2)[t < nbias ? t : t - nbias] = sb;
  }
}

}  // namespace afno
