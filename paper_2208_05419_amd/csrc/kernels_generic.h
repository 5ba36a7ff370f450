// kernels_generic.h -- size-generic W-axis kernels of the AFNO filter: any W of the form
// 2^a 3^b 5^c within the plan limits.  Transforms run as radix-2/3/4/5 Stockham passes
// over LDS (fft_lds.h); the size-specialised kernels of kernels_fast.h replace them for
// widths from 12 to 576.  The size-generic column kernels are in kernels_column.h.
//
// Three passes over HBM, all on one spectrum workspace S [B][H][KW][C] (complex,
// (re, im) interleaved, stored in the filter's dtype; KW = kept_w columns):
//   row_r2c   x -> S       real-to-complex DFT along W of every (b, h, c) line
//                          (FourCastNet, "Implementation Details" (b): R2C transform
//                          batched over batch and channels), scaled 1/sqrt(W)
//   column    S -> S       per (b, kw, channel block): DFT along H, the block complex
//                          MLP on MFMA with bias/ReLU/bias/softshrink/cutoff in the
//                          epilogues, inverse DFT along H ("Model Innovations" steps
//                          1-3; the MLP weights shared by every mode), in place
//   row_c2r   S, x -> out  complex-to-real inverse along W plus the residual add,
//                          rounded once to the dtype
// Two real channels (c, c+1) travel through the W transforms as one complex signal
// z = x_c + i x_{c+1}; their half spectra are separated (forward) and recombined
// (inverse) through the conjugate symmetry of a real signal's spectrum.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "afno_internal.h"
#include "fft_lds.h"
#include "kernel_common.h"

namespace afno {

// ------------------------------------------------------------------ kernel 1: W-axis R2C

// grid (B * H, C / rc), block kRowThreads.  LDS: W x (rc/2) float2 signals + W twiddles.
template <typename T>
__global__ void __launch_bounds__(kRowThreads)
row_r2c_kernel(const T* __restrict__ x, T* __restrict__ S, RowParams p) {
  extern __shared__ float4 smem_raw[];
  float2* buf = reinterpret_cast<float2*>(smem_raw);
  const int np = p.rc / 2;
  float2* tw = buf + (size_t)p.W * np;
  const int tid = threadIdx.x;
  const int64_t row = blockIdx.x;  // b * H + h
  const int c0 = blockIdx.y * p.rc;

  make_twiddles(tw, p.W);  // synchronises

  // load x[b][h][:][c0 : c0 + rc] as np complex signals of length W
  constexpr int V = Store<T>::kVec;
  const int vpr = p.rc / V;
  const T* xr = x + row * p.W * p.C + c0;
  for (int it = tid; it < p.W * vpr; it += blockDim.x) {
    const int n = it / vpr, cv = it - n * vpr;
    V16 v;
    v.u = *reinterpret_cast<const uint4*>(xr + (int64_t)n * p.C + cv * V);
#pragma unroll
    for (int q = 0; q < V / 2; ++q) {
      float a, b;
      if constexpr (V == 4) { a = v.f[2 * q]; b = v.f[2 * q + 1]; }
      else { a = (float)v.h[2 * q]; b = (float)v.h[2 * q + 1]; }
      buf[n * np + cv * (V / 2) + q] = make_float2(a, b);
    }
  }
  __syncthreads();

  const int sig = tid % np, sub = tid / np, nsub = blockDim.x / np;
  fft_lds<kRowEmax, false>(buf, np, p.rw, sig, sub, nsub, tw);

  // separate the two real channels of each signal and store kw in [0, KW):
  //   X_c = (Z[k] + conj Z[W-k]) / 2,  X_{c+1} = (Z[k] - conj Z[W-k]) / (2i)
  const float sc = 0.5f * p.inv_sqrt_w;
  T* Sr = S + row * (int64_t)p.KW * p.C * 2;
  for (int it = tid; it < p.KW * np; it += blockDim.x) {
    const int k = it / np, q = it - k * np;
    const float2 z = buf[k * np + q];
    const int km = (k == 0) ? 0 : p.W - k;
    const float2 zm = buf[km * np + q];
    const float ar = (z.x + zm.x) * sc, ai = (z.y - zm.y) * sc;
    const float br = (z.y + zm.y) * sc, bi = (zm.x - z.x) * sc;
    T* o = Sr + ((int64_t)k * p.C + c0 + 2 * q) * 2;
    if constexpr (V == 4) {
      *reinterpret_cast<float4*>(o) = make_float4(ar, ai, br, bi);
    } else {
      union { uint2 u; bf16 h[4]; } w;
      w.h[0] = (bf16)ar; w.h[1] = (bf16)ai; w.h[2] = (bf16)br; w.h[3] = (bf16)bi;
      *reinterpret_cast<uint2*>(o) = w.u;
    }
  }
}

// ------------------------------------------------------------------ kernel 3: W-axis C2R + residual

// grid (B * H, C / rc), block kRowThreads.  mode 0: out = x + y in T; mode 1: dst = y (float).
template <typename T>
__global__ void __launch_bounds__(kRowThreads)
row_c2r_kernel(const T* __restrict__ S, const T* __restrict__ x, T* __restrict__ out,
               float* __restrict__ dst, RowParams p, int mode) {
  extern __shared__ float4 smem_raw[];
  float2* buf = reinterpret_cast<float2*>(smem_raw);
  const int np = p.rc / 2;
  float2* tw = buf + (size_t)p.W * np;
  const int tid = threadIdx.x;
  const int64_t row = blockIdx.x;  // b * H + h
  const int c0 = blockIdx.y * p.rc;
  const int half = p.W / 2;

  make_twiddles(tw, p.W);

  // Z[k] = Y_c[k] + i Y_{c+1}[k] over the full length, with Y[W-k] = conj Y[k] and only
  // the real parts of the k = 0 and k = W/2 bins; columns k >= KW are zero.
  const T* Sr = S + row * (int64_t)p.KW * p.C * 2;
  for (int it = tid; it < (half + 1) * np; it += blockDim.x) {
    const int k = it / np, q = it - k * np;
    float ar = 0.f, ai = 0.f, br = 0.f, bi = 0.f;
    if (k < p.KW) {
      const T* s = Sr + ((int64_t)k * p.C + c0 + 2 * q) * 2;
      if constexpr (Store<T>::kVec == 4) {
        const float4 v = *reinterpret_cast<const float4*>(s);
        ar = v.x; ai = v.y; br = v.z; bi = v.w;
      } else {
        union { uint2 u; bf16 h[4]; } w;
        w.u = *reinterpret_cast<const uint2*>(s);
        ar = (float)w.h[0]; ai = (float)w.h[1]; br = (float)w.h[2]; bi = (float)w.h[3];
      }
    }
    if (k == 0 || k == half) {
      buf[k * np + q] = make_float2(ar, br);
    } else {
      buf[k * np + q] = make_float2(ar - bi, ai + br);
      buf[(p.W - k) * np + q] = make_float2(ar + bi, br - ai);
    }
  }
  __syncthreads();

  const int sig = tid % np, sub = tid / np, nsub = blockDim.x / np;
  fft_lds<kRowEmax, true>(buf, np, p.rw, sig, sub, nsub, tw);

  constexpr int V = Store<T>::kVec;
  const int vpr = p.rc / V;
  const float sc = p.inv_sqrt_w;
  const int64_t base = row * p.W * p.C + c0;
  for (int it = tid; it < p.W * vpr; it += blockDim.x) {
    const int n = it / vpr, cv = it - n * vpr;
    const int64_t off = base + (int64_t)n * p.C + cv * V;
    float y[V];
#pragma unroll
    for (int q = 0; q < V / 2; ++q) {
      const float2 z = buf[n * np + cv * (V / 2) + q];
      y[2 * q] = z.x * sc;
      y[2 * q + 1] = z.y * sc;
    }
    if (mode == 1) {
#pragma unroll
      for (int e = 0; e < V; e += 4)
        *reinterpret_cast<float4*>(dst + off + e) = make_float4(y[e], y[e + 1], y[e + 2], y[e + 3]);
      continue;
    }
    V16 xv, ov;
    xv.u = *reinterpret_cast<const uint4*>(x + off);
#pragma unroll
    for (int e = 0; e < V; ++e) {
      if constexpr (V == 4) ov.f[e] = xv.f[e] + y[e];
      else ov.h[e] = (bf16)((float)xv.h[e] + y[e]);
    }
    *reinterpret_cast<uint4*>(out + off) = ov.u;
  }
}

// ------------------------------------------------------------------ diagnostic export

// dst [B][H][Wm][C][2] float from S [B][H][KW][C][2]; columns kw >= KW written as 0.
template <typename T>
__global__ void export_spectrum_kernel(const T* __restrict__ S, float* __restrict__ dst,
                                       int64_t B, int H, int Wm, int KW, int C) {
  const int64_t total = B * H * (int64_t)Wm * C * 2;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t e = i % (2 * C);
    const int64_t r = i / (2 * C);  // (b * H + h) * Wm + kw
    const int kw = (int)(r % Wm);
    const int64_t bh = r / Wm;
    dst[i] = (kw < KW) ? ld_f(S + (bh * KW + kw) * 2 * C + e) : 0.f;
  }
}

}  // namespace afno
