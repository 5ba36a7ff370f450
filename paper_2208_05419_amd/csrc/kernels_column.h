// kernels_column.h -- size-generic column kernels of the AFNO filter, forward and backward:
// any H = 2^a 3^b 5^c <= 192, any block size and hidden size, both storage types.
//
// One workgroup takes one column (b, kw, channel block) and keeps it in one LDS tile
// [H16][ldt] of the storage type (H16 = H rounded up to 16):
//
//  * H transforms: H = n1 n2 (col_split), two register DFTs (dft_reg.h) in fp32 around one LDS
//    exchange, as in kernels_fast.h, chk channels at a time, one task a thread and stage.  The
//    factors come from small sets, so the lengths are a switch over compile-time DFTs rather
//    than a kernel per H.  In fp32 the exchange uses the chunk's own columns of the tile; in
//    bf16, whose tile rows are half as wide, a float buffer [H][chk], which overlays the tiles
//    where one chunk takes all channels.
//  * Block MLP (transposed form): D^T[entry][row] = W^T[entry][k] tile^T[k][row] on the matrix
//    cores, the weights as fragment words prepared once per call (prep_general_words), so that
//    a lane ends up with four consecutive entries of one row: one 8- or 16-byte LDS store.
//    Waves form a wm x wn grid, each mw tiles of 16 rows by nw tiles of 16 entries.  In fp32
//    (16x16x4 matrix instructions) a lane's 16-byte word holds k = 4 g .. 4 g + 3 of 16 for lane
//    group g, and instruction j of four takes value j of both operands: any order of the sum
//    serves as long as both operands agree, and it quarters the LDS reads.
//  * Row tiles of 16 that a cutoff empties are left out of the products (mlist).
//
// Replaces the radix passes over LDS (four or five passes with two barriers each and a copy of
// every channel chunk on both sides) and weights gathered four bytes at a time from their plain
// layout.  Column pass, before and after: forward 2 x 128 x 256 x 512 bf16 (8 blocks of 64) 302 ->
// 81 us; backward 72 x 144 x 384 fp32 (8 of 48) 300 -> 97 us, 180 x 360 x 1024 bf16 (32 of 32)
// 1373 -> 339 us.  What bounds it, from counters: in bf16 the vector ALUs' issue of the fp32
// transforms (forward 54 % of the time busy, 1,758 instructions a wave; backward 63 %, 2,908) and
// the latency of the phases between barriers (waves wait 53 % of their time, two columns of eight
// waves to a compute unit; matrix cores 8 and 4 % busy, LDS 17 and 19 %); in the fp32 backward
// that latency alone (584 columns on 256 compute units, vector ALUs 17 % and matrix cores 25 %
// busy).  The size-specialised kernels of kernels_fast.h, their strides immediate offsets, stay
// ahead at their few sizes (180 x 32 bf16: 90 us against 115).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "afno_internal.h"
#include "dft_reg.h"
#include "kernel_common.h"
#include "kernels_fast.h"
#include "kernels_prep.h"

namespace afno {

// ------------------------------------------------------------------ H transforms

// one task of a stage: N values from ld, their DFT, to st
template <int N, bool INV, class Ld, class Mid, class St>
__device__ __forceinline__ void dft_task(bool act, Ld ld, Mid mid, St st) {
  float2 v[N];
  if (act) {
#pragma unroll
    for (int t = 0; t < N; ++t) v[t] = ld(t);
    DftReg<N, INV>::run(v);
  }
  mid();  // a barrier between the reads and the writes, or nothing
  if (act) {
#pragma unroll
    for (int k = 0; k < N; ++k) st(k, v[k]);
  }
}

// The second factor's sizes (n2) and the first's (n1); every 5-smooth H <= 192 is n1 n2.  Only
// H = 162 and 125 need 18 and 25: a forward kernel with those two beside the others would spill (57
// registers in fp32), so they have instances of their own.  What spills all the same (registers,
// and bytes of scratch a lane): the backward in bf16, 4 and 20, with more than eight tiles a wave
// or H = 162 or 125 15 and 36 (in fp32 8 and 20, the main one none), and the bf16 forward without
// prepared words 102 and 88.  At 180 x 360 x 1024 in 32 blocks the backward writes 747 MB, 44 more
// than the factors and the spectrum: its scratch makes up at most that.
enum { kSizesMain = 0, kSizesBig = 1, kSizesAll = 2 };
#define AFNO_COL_N2(X) X(1) X(2) X(3) X(4) X(5) X(6) X(8) X(9) X(10) X(12) X(15) X(16)
#define AFNO_COL_N2_BIG(X) X(18) X(25)
#define AFNO_COL_N1(X) X(1) X(2) X(3) X(4) X(5) X(6) X(8) X(9) X(10) X(12)
#define AFNO_COL_N1_BIG(X) X(5) X(9)

template <bool INV, int SIZES, class Ld, class Mid, class St>
__device__ __forceinline__ void dft_n2(int n, bool act, Ld ld, Mid mid, St st) {
#define AFNO_CASE(N) case N: dft_task<N, INV>(act, ld, mid, st); break;
  if constexpr (SIZES != kSizesBig) {
    switch (n) { AFNO_COL_N2(AFNO_CASE) }
  }
  if constexpr (SIZES != kSizesMain) {
    switch (n) { AFNO_COL_N2_BIG(AFNO_CASE) }
  }
#undef AFNO_CASE
}
template <bool INV, int SIZES, class Ld, class Mid, class St>
__device__ __forceinline__ void dft_n1(int n, bool act, Ld ld, Mid mid, St st) {
#define AFNO_CASE(N) case N: dft_task<N, INV>(act, ld, mid, st); break;
  if constexpr (SIZES == kSizesBig) {
    switch (n) { AFNO_COL_N1_BIG(AFNO_CASE) }
  } else {
    switch (n) { AFNO_COL_N1(AFNO_CASE) }
  }
#undef AFNO_CASE
}

// LDS of a column workgroup: the tile, the hidden tile (hs != bs), the exchange buffer (bf16),
// the roots
template <typename T>
struct ColMem {
  T* tile;
  T* htile;
  uint32_t base, fbuf, tw;  // LDS addresses of the tile, the exchange buffer and the roots
  __device__ __forceinline__ ColMem(void* smem, const ColParams& p) {
    char* m = reinterpret_cast<char*>(smem);
    tile = reinterpret_cast<T*>(m);
    htile = p.htile_bytes ? reinterpret_cast<T*>(m + p.tile_bytes) : tile;
    base = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)smem;
    fbuf = p.overlay ? base : base + p.tile_bytes + p.htile_bytes;
    tw = base + p.tw_off;
  }
  __device__ __forceinline__ float2* roots(void* smem) const {
    return reinterpret_cast<float2*>(reinterpret_cast<char*>(smem) + (tw - base));
  }
};

// An LDS address that moves by a runtime stride from access to access.  Each step is opaque, so
// one register holds the address; left to itself the compiler forms all of a stage's addresses
// first and keeps them live (40 registers more at 16 points).
struct Walk {
  uint32_t off;
  uint32_t step;
  __device__ __forceinline__ uint32_t next() {
    const uint32_t o = off;
    off = (uint32_t)opq((int)(off + step));
    return o;
  }
};
// the value of type V at LDS address `a`
template <typename V>
__device__ __forceinline__ __attribute__((address_space(3))) V& at(uint32_t a) {
  return *reinterpret_cast<__attribute__((address_space(3))) V*>(a);
}
__device__ __forceinline__ float2 ld_pair_at(uint32_t a, const float*) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  const f2 v = at<f2>(a);
  return make_float2(v.x, v.y);
}
__device__ __forceinline__ float2 ld_pair_at(uint32_t a, const bf16*) { return widen2(at<uint32_t>(a)); }
__device__ __forceinline__ void st_pair_at(uint32_t a, float2 z, const float*) {
  typedef float f2 __attribute__((ext_vector_type(2)));
  at<f2>(a) = f2{z.x, z.y};
}
__device__ __forceinline__ void st_pair_at(uint32_t a, float2 z, const bf16*) {
  at<uint32_t>(a) = pack_c(z, (const bf16*)nullptr);
}

// tile rows h < H = DFT along H of the column at cb (row stride rsb bytes), scaled.  Every
// thread of the workgroup takes part; the caller's barrier ends it.
template <typename T, int SIZES>
__device__ __forceinline__ void column_dft(const CBuf<T>& cb, uint32_t rsb, const ColMem<T>& m,
                                           const ColParams& p, float scale) {
  constexpr bool kOwn = sizeof(T) == 2;  // the exchange buffer is its own
  constexpr uint32_t es = sizeof(T);
  constexpr const float* kF = nullptr;
  const int n1 = p.n1, n2 = p.n2, chk = p.chk, ldt = p.ldt;
  const uint32_t fs = (kOwn ? chk : ldt / 2) * 8;  // row stride of the exchange, bytes
  for (int cc = 0; cc < p.bs; cc += chk) {
    const uint32_t fc = kOwn ? m.fbuf : m.base + cc * 8;
    // first stage: rows j + n1 t of channel cc + c
    {
      const int tid = opq((int)threadIdx.x), j = (tid * p.chk_inv) >> 20, c = tid - j * chk;
      const uint32_t voff = 2 * (cc + c) * es + j * rsb, soff = n1 * rsb;
      Walk f{fc + c * 8 + j * fs, n1 * fs}, w{m.tw, (uint32_t)j * 8};
      dft_n2<false, SIZES>(n2, j < n1, [&](int t) { return cb.ld(voff, t * soff); }, [] {},
                           [&](int k, float2 v) {
                             const float2 r = ld_pair_at(w.next(), kF);
                             st_pair_at(f.next(), k == 0 ? v : c_mul(v, r), kF);
                           });
    }
    __syncthreads();
    // second stage: residue j of n2 -> spectrum rows j + n2 k
    {
      const int tid = opq((int)threadIdx.x), j = (tid * p.chk_inv) >> 20, c = tid - j * chk;
      Walk f{fc + c * 8 + j * n1 * fs, fs};
      Walk o{m.base + (j * ldt + 2 * (cc + c)) * es, n2 * ldt * es};
      dft_n1<false, SIZES>(n1, j < n2, [&](int) { return ld_pair_at(f.next(), kF); },
                           [] { __syncthreads(); },  // the exchange has been read
                           [&](int, float2 v) {
                             st_pair_at(o.next(), make_float2(v.x * scale, v.y * scale), (const T*)nullptr);
                           });
    }
  }
}

// the column at cb = inverse DFT along H of the tile's rows, scaled (the tile is used up)
template <typename T, int SIZES>
__device__ __forceinline__ void column_idft(const CBuf<T>& cb, uint32_t rsb, const ColMem<T>& m,
                                            const ColParams& p, float scale) {
  constexpr bool kOwn = sizeof(T) == 2;
  constexpr uint32_t es = sizeof(T);
  constexpr const float* kF = nullptr;
  const int n1 = p.n1, n2 = p.n2, chk = p.chk, ldt = p.ldt;
  const uint32_t fs = (kOwn ? chk : ldt / 2) * 8;
  for (int cc = 0; cc < p.bs; cc += chk) {
    const uint32_t fc = kOwn ? m.fbuf : m.base + cc * 8;
    {
      const int tid = opq((int)threadIdx.x), j = (tid * p.chk_inv) >> 20, c = tid - j * chk;
      Walk i{m.base + (j * ldt + 2 * (cc + c)) * es, n1 * ldt * es};
      Walk f{fc + c * 8 + j * fs, n1 * fs}, w{m.tw, (uint32_t)j * 8};
      dft_n2<true, SIZES>(n2, j < n1, [&](int) { return ld_pair_at(i.next(), (const T*)nullptr); },
                          [&] { if (!kOwn || p.overlay) __syncthreads(); },  // the tile has been read
                          [&](int k, float2 v) {
                            float2 r = ld_pair_at(w.next(), kF);
                            r.y = -r.y;
                            st_pair_at(f.next(), k == 0 ? v : c_mul(v, r), kF);
                          });
    }
    __syncthreads();
    {
      const int tid = opq((int)threadIdx.x), j = (tid * p.chk_inv) >> 20, c = tid - j * chk;
      const uint32_t voff = 2 * (cc + c) * es + j * rsb, soff = n2 * rsb;
      Walk f{fc + c * 8 + j * n1 * fs, fs};
      dft_n1<true, SIZES>(n1, j < n2, [&](int) { return ld_pair_at(f.next(), kF); }, [] {},
                          [&](int k, float2 v) {
                            cb.st(voff, k * soff, make_float2(v.x * scale, v.y * scale));
                          });
    }
    if (kOwn && cc + chk < p.bs) __syncthreads();  // the exchange is written again
  }
}

// ------------------------------------------------------------------ block products

// four consecutive entries (16-byte aligned in fp32, 8-byte in bf16)
__device__ __forceinline__ void st_quad(float* p, f32x4 v) {
  *reinterpret_cast<float4*>(p) = make_float4(v[0], v[1], v[2], v[3]);
}
__device__ __forceinline__ void st_quad(bf16* p, f32x4 v) {
  *reinterpret_cast<uint2*>(p) = make_uint2(cvt_pk(v[0], v[1]), cvt_pk(v[2], v[3]));
}
__device__ __forceinline__ f32x4 ld_quad(const float* p) {  // 4-byte aligned
  return f32x4{p[0], p[1], p[2], p[3]};
}
__device__ __forceinline__ f32x4 ld_quad(const bf16* p) {
  const uint32_t* q = reinterpret_cast<const uint32_t*>(p);
  const uint32_t a = q[0], b = q[1];
  return f32x4{__uint_as_float(a << 16), __uint_as_float(a & 0xffff0000u),
               __uint_as_float(b << 16), __uint_as_float(b & 0xffff0000u)};
}

// entries of a k-step of the products: one 16-byte word per lane and operand
template <typename T> __host__ __device__ constexpr int kstep() { return sizeof(T) == 2 ? 32 : 16; }

template <typename T>
__device__ __forceinline__ f32x4 mma_word(uint4 a, uint4 b, f32x4 c) {
  V16 x, y;
  x.u = a;
  y.u = b;
  if constexpr (sizeof(T) == 2) {
    union { uint4 u; bf16x8 f; } p, q;
    p.u = a;
    q.u = b;
    c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(p.f, q.f, c, 0, 0, 0);
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e) c = __builtin_amdgcn_mfma_f32_16x16x4f32(x.f[e], y.f[e], c, 0, 0, 0);
  }
  return c;
}

// the row tile (of 16 rows) at position i of the wave grid's list of live tiles
__device__ __forceinline__ int live_tile(const ColParams& p, int i) {
  return (int)(p.mlist >> (4 * i)) & 15;
}

// A product's weights: their prepared fragment words (at byte woff of wb), or (PLAIN) the
// layer's own array w [n_in][n_out][2], gathered entry by entry.
template <typename T>
struct Words {
  Buf wb;
  uint32_t woff;
  const T* w;
  int n_out;
};

// acc[m][n] = entry tile NW grp + n of W^T tile^T, row tile live_tile(MW wm + m): lane l16 is
// a row, its four values entries 4 g .. 4 g + 3; ks k-steps of nt entry tiles.
template <typename T, int MW, int NW, bool PLAIN = false>
__device__ __forceinline__ void column_product(const T* src, int ld, const Words<T>& ww, int ks,
                                               int nt, const ColParams& p, int wm, int grp,
                                               f32x4 (&acc)[MW][NW]) {
  const int lane = opq((int)threadIdx.x) & 63;
  const int l16 = lane & 15, g = lane >> 4;
  const T* row[MW];
#pragma unroll
  for (int m = 0; m < MW; ++m)
    row[m] = src + (16 * live_tile(p, min(MW * wm + m, p.mt - 1)) + l16) * ld + (kstep<T>() / 4) * g;
  const uint32_t voff = lane * 16u;
  uint32_t soff = ww.woff + NW * grp * 1024u;
  const uint32_t sstep = nt * 1024u;
  auto wload = [&](uint4 (&w)[NW], int s) {
    if constexpr (PLAIN) {
      constexpr int E = 16 / sizeof(T);
#pragma unroll
      for (int n = 0; n < NW; ++n) {
        union { uint4 u; T e[E]; } v;
#pragma unroll
        for (int e = 0; e < E; ++e)
          v.e[e] = real_entry(ww.w, ww.n_out, (4 * s + g) * E + e, 16 * (NW * grp + n) + l16);
        w[n] = v.u;
      }
    } else {
#pragma unroll
      for (int n = 0; n < NW; ++n) {
        const auto v = __builtin_amdgcn_raw_buffer_load_b128(ww.wb.r, voff, soff + n * 1024u, 0);
        w[n] = make_uint4(v[0], v[1], v[2], v[3]);
      }
    }
  };
#pragma unroll
  for (int m = 0; m < MW; ++m)
#pragma unroll
    for (int n = 0; n < NW; ++n) acc[m][n] = f32x4{0.f, 0.f, 0.f, 0.f};
  uint4 w[NW];
  wload(w, 0);
  for (int s = 0; s < ks; ++s) {
    uint4 wn[NW];
    if (s + 1 < ks) soff += sstep;
    wload(wn, min(s + 1, ks - 1));  // one k-step ahead (the last step's own words again)
#pragma unroll
    for (int m = 0; m < MW; ++m) {
      const uint4 y = *reinterpret_cast<const uint4*>(row[m] + s * kstep<T>());
#pragma unroll
      for (int n = 0; n < NW; ++n) acc[m][n] = mma_word<T>(w[n], y, acc[m][n]);
    }
#pragma unroll
    for (int n = 0; n < NW; ++n) w[n] = wn[n];
  }
}

// rows 16 t + l16 of the wave's live tiles: f(m, n, row, entry of its first value)
template <int MW, int NW, class F>
__device__ __forceinline__ void each_quad(const ColParams& p, int wm, int grp, F f) {
  const int lane = opq((int)threadIdx.x) & 63;
#pragma unroll
  for (int m = 0; m < MW; ++m) {
    const int i = MW * wm + m;
    if (i >= p.mt) continue;  // wave-uniform
    const int row = 16 * live_tile(p, i) + (lane & 15);
#pragma unroll
    for (int n = 0; n < NW; ++n) f(m, n, row, 16 * (NW * grp + n) + 4 * (lane >> 4));
  }
}

// S(v) with its 'else 0' taken to the letter: the middle of v - lam, 0 and v + lam, where a NaN
// gives 0 too (v_med3_f32 takes the least of its numbers then), as it does in the backward kernel's
// mask |o| > lam; v - clamp(v, -lam, lam) passes it on, with one instruction a value fewer.  That one
// costs 0.8 % of a call at 128 x 256 x 512 bf16 (147.1 us against 146.0), so where nothing is cut off
// the rows' keep is not taken either (144.0 against 143.9).
__device__ __forceinline__ float shrink_or_zero(float v, float lam) {
  return __builtin_amdgcn_fmed3f(v - lam, 0.f, v + lam);
}

// zeros in the tile's rows outside the live row tiles (cutoff)
template <typename T>
__device__ __forceinline__ void zero_dead_rows(T* tile, const ColParams& p) {
  const int mt = p.H16 / 16;
  if (p.mt == mt) return;
  uint32_t live = 0;
  for (int i = 0; i < p.mt; ++i) live |= 1u << live_tile(p, i);
  constexpr int V = Store<T>::kVec;
  const int vpr = 2 * p.bs / V;
  for (int t = 0; t < mt; ++t) {
    if ((live >> t) & 1u) continue;
    for (int it = threadIdx.x; it < 16 * vpr; it += blockDim.x) {
      const int r = it / vpr, v = it - r * vpr;
      *reinterpret_cast<uint4*>(tile + (16 * t + r) * p.ldt + v * V) = make_uint4(0, 0, 0, 0);
    }
  }
}

// padding rows H .. H16 - 1 = 0 (the transforms write rows h < H only)
template <typename T>
__device__ __forceinline__ void zero_pad_rows(T* tile, const ColParams& p) {
  constexpr int V = Store<T>::kVec;
  const int vpr = 2 * p.bs / V;
  for (int it = threadIdx.x; it < (p.H16 - p.H) * vpr; it += blockDim.x) {
    const int r = it / vpr, v = it - r * vpr;
    *reinterpret_cast<uint4*>(tile + (p.H + r) * p.ldt + v * V) = make_uint4(0, 0, 0, 0);
  }
}

// (mw, nw) of the wave grid -> compile-time sizes; f is a generic callable of two
// integral_constants.  The kernels with at most eight tiles a wave need 66 to 74 registers (six
// waves a SIMD); the wide ones, for the sizes that would take more than 12 waves so, 92.
#define AFNO_COL_GRID(X) X(1, 2) X(2, 2) X(3, 2) X(4, 2) X(1, 4) X(2, 4)
#define AFNO_COL_GRID_WIDE(X) X(6, 2) X(3, 4) X(4, 4)
template <bool WIDE, class F>
__device__ __forceinline__ void with_grid(const ColParams& p, F f) {
#define AFNO_CASE(MW, NW) \
    case MW * 8 + NW: f(std::integral_constant<int, MW>(), std::integral_constant<int, NW>()); break;
  if constexpr (WIDE) {
    switch (p.mw * 8 + p.nw) { AFNO_COL_GRID_WIDE(AFNO_CASE) AFNO_COL_GRID(AFNO_CASE) }
  } else {
    switch (p.mw * 8 + p.nw) { AFNO_COL_GRID(AFNO_CASE) }
  }
#undef AFNO_CASE
}

// ------------------------------------------------------------------ forward

// grid B * KW * nb (block index fastest), block p.threads, dynamic LDS pl.col_lds.  S updated in place.  stage: 0 full, 1 stop after the forward transform, 2 stop
// after the MLP.
// PLAIN: no prepared words (a fixed workspace without room for them), the weights gathered from w1
// and w2: 1 x 144 x 450 x 1024 bf16 (8 blocks of 128) 618 us a call against 334 with words, and 1,218
// with the radix passes that this replaced; 1 x 100 x 320 x 1024 fp32 672, 555 and 1,474.
template <typename T, int SIZES, bool WIDE, bool PLAIN>
__global__ void __launch_bounds__(1024)
column_general(T* __restrict__ S, const uint4* __restrict__ wfrag, const T* __restrict__ w1,
               const T* __restrict__ w2, const T* __restrict__ b1, const T* __restrict__ b2,
               ColParams p, int stage) {
  extern __shared__ float4 smem_raw[];
  const ColMem<T> mem(smem_raw, p);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int bs = p.bs, hs = p.hs, ldt = p.ldt, ldh = p.htile_bytes ? p.ldh : ldt;

  const int blk = blockIdx.x % p.nb;  // consecutive workgroups -> different XCDs -> blocks
  const int rest = blockIdx.x / p.nb;
  const int kw = rest % p.KW;
  const int64_t b = rest / p.KW;
  const uint32_t rsb = (uint32_t)p.KW * (uint32_t)p.C * 2 * (uint32_t)sizeof(T);
  T* col = S + ((b * p.H) * p.KW + kw) * (int64_t)p.C * 2 + (int64_t)blk * bs * 2;
  const CBuf<T> cb(col, buf_bytes((uint64_t)p.H * rsb));

  make_twiddles(mem.roots(smem_raw), p.H);
  column_dft<T, SIZES>(cb, rsb, mem, p, p.inv_sqrt_h);
  __syncthreads();  // (the padding rows H .. H16 - 1 hold anything: no row depends on another)

  if (stage != 1) {
    const int wm = wave / p.wn, wn = wave % p.wn;
    const bool wave_in = wm < p.wm;
    const uint32_t lbytes = (uint32_t)(bs * hs / 4) * 16u * (uint32_t)sizeof(T);  // one layer's words
    const Buf wb(reinterpret_cast<const char*>(wfrag) + (int64_t)blk * 2 * lbytes, PLAIN ? 0 : 2 * lbytes);
    const Words<T> l1{wb, 0, w1 + (int64_t)blk * bs * hs * 2, hs}, l2{wb, lbytes, w2 + (int64_t)blk * bs * hs * 2, bs};
    const int ks1 = 2 * bs / kstep<T>(), ks2 = 2 * hs / kstep<T>();
    with_grid<WIDE>(p, [&](auto MWc, auto NWc) {
      constexpr int MW = decltype(MWc)::value, NW = decltype(NWc)::value;
      f32x4 acc[MW][NW];
      // layer 1: entry groups wn, wn + p.wn, ...; in place (hs = bs) one group per wave, every
      // wave's reads before any write
      const int ng1 = 2 * hs / (16 * NW);
      for (int g0 = 0; g0 < ng1; g0 += p.wn) {
        const int grp = g0 + wn;
        const bool act = wave_in && grp < ng1;
        if (act) column_product<T, MW, NW, PLAIN>(mem.tile, ldt, l1, ks1, 2 * hs / 16, p, wm, grp, acc);
        if (!p.htile_bytes) __syncthreads();
        if (act) {
          f32x4 bias[NW];
#pragma unroll
          for (int n = 0; n < NW; ++n)
            bias[n] = ld_quad(b1 + (int64_t)blk * hs * 2 + 16 * (NW * grp + n) + 4 * (lane >> 4));
          each_quad<MW, NW>(p, wm, grp, [&](int m, int n, int row, int e0) {
            f32x4 v;
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = fmaxf(acc[m][n][r] + bias[n][r], 0.f);
            st_quad(mem.htile + row * ldh + e0, v);
          });
        }
      }
      __syncthreads();  // hidden layer complete
      const bool act = wave_in && wn < 2 * bs / (16 * NW);
      if (act) column_product<T, MW, NW, PLAIN>(mem.htile, ldh, l2, ks2, 2 * bs / 16, p, wm, wn, acc);
      __syncthreads();  // every wave has read the hidden rows
      if (act) {
        f32x4 bias[NW];
#pragma unroll
        for (int n = 0; n < NW; ++n)
          bias[n] = ld_quad(b2 + (int64_t)blk * bs * 2 + 16 * (NW * wn + n) + 4 * (lane >> 4));
        auto shrink = [&](auto all_rows) {  // nothing cut off: the padding rows may hold anything
          each_quad<MW, NW>(p, wm, wn, [&](int m, int n, int row, int e0) {
            const bool keep = all_rows || row_kept(row, p.H, p.kept_h);
            f32x4 v;
#pragma unroll
            for (int r = 0; r < 4; ++r) v[r] = keep ? shrink_or_zero(acc[m][n][r] + bias[n][r], p.lam) : 0.f;
            st_quad(mem.tile + row * ldt + e0, v);
          });
        };
        if (p.kept_h > p.H / 2)
          shrink(std::true_type());
        else
          shrink(std::false_type());
      }
    });
    zero_dead_rows(mem.tile, p);
    __syncthreads();
  }

  if (stage != 0) {  // diagnostic stop: the tile goes back to S as it is
    constexpr int V = Store<T>::kVec;
    const int vpr = 2 * bs / V;
    for (int it = tid; it < p.H * vpr; it += blockDim.x) {
      const int h = it / vpr, cv = it - h * vpr;
      *reinterpret_cast<uint4*>(reinterpret_cast<char*>(col) + (int64_t)h * rsb + cv * 16) =
          *reinterpret_cast<const uint4*>(mem.tile + h * ldt + cv * V);
    }
    return;
  }
  column_idft<T, SIZES>(cb, rsb, mem, p, p.inv_sqrt_h);
}

// ------------------------------------------------------------------ backward

// Per-mode factors: four tensors (X, h, do, dv), each [nb][mpad / 8][2 bs][8] in T: modes in
// groups of eight, the group's 2 bs entries consecutive, eight modes per entry contiguous (one
// 16-byte matrix-core operand for bf16).  The column (b, kw) holds modes (b KW + kw) HC ..
// + HC - 1, HC = H16 rounded up to 32 (rows past H hold X = 0, do = dv = 0, so they add
// nothing to the sums); mpad = B KW HC, a multiple of 32 (the slab product reads a chunk's
// ragged last 64-mode step as zeros past its end).
enum { kModeX = 0, kModeH = 1, kModeDo = 2, kModeDv = 3 };
__host__ __device__ inline int col_bwd_hc(int H16) { return (H16 + 31) / 32 * 32; }

// 16 bytes written once and read once by a later pass: non-temporal, so that they do not
// displace the spectra and the weights in the caches
template <typename T>
__device__ __forceinline__ void st_stream(T* p, uint4 v) {
  typedef uint32_t u4 __attribute__((ext_vector_type(4)));
  __builtin_nontemporal_store(u4{v.x, v.y, v.z, v.w}, reinterpret_cast<u4*>(p));
}

// tile rows 0 .. HC - 1 of the block's 2 bs entries -> dst groups m0 / 8 .., 8 rows per task
// (rows past H16 are zero)
__device__ __forceinline__ void write_modes(const float* tile, const ColParams& p, int HC,
                                            float* dst, int64_t m0) {
  const int nb2 = 2 * p.bs, tasks = p.bs * (HC / 8);
  for (int t = opq((int)threadIdx.x); t < tasks; t += blockDim.x) {
    const int r8 = (int)(((uint32_t)t * (uint32_t)p.bs_inv) >> 20), c = t - r8 * p.bs, r0 = 8 * r8;
    V16 re[2], im[2];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float2 z = r0 < p.H16 ? ld_c(tile + (r0 + i) * p.ldt + 2 * c) : make_float2(0.f, 0.f);
      re[i / 4].f[i % 4] = z.x;
      im[i / 4].f[i % 4] = z.y;
    }
    float* pr = dst + (((m0 + r0) / 8) * nb2 + 2 * c) * 8;
    st_stream(pr, re[0].u);
    st_stream(pr + 4, re[1].u);
    st_stream(pr + 8, im[0].u);
    st_stream(pr + 12, im[1].u);
  }
}
__device__ __forceinline__ void write_modes(const bf16* tile, const ColParams& p, int HC, bf16* dst,
                                            int64_t m0) {
  const int nb2 = 2 * p.bs, tasks = p.bs * (HC / 8);
  for (int t = opq((int)threadIdx.x); t < tasks; t += blockDim.x) {
    const int r8 = (int)(((uint32_t)t * (uint32_t)p.bs_inv) >> 20), c = t - r8 * p.bs, r0 = 8 * r8;
    uint32_t z[8];
#pragma unroll
    for (int i = 0; i < 8; ++i)
      z[i] = r0 < p.H16 ? *reinterpret_cast<const uint32_t*>(tile + (r0 + i) * p.ldt + 2 * c) : 0u;
    uint32_t re[4], im[4];  // the low halves and the high halves of two rows each
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      re[i] = __builtin_amdgcn_perm(z[2 * i + 1], z[2 * i], 0x05040100u);
      im[i] = __builtin_amdgcn_perm(z[2 * i + 1], z[2 * i], 0x07060302u);
    }
    bf16* pr = dst + (((m0 + r0) / 8) * nb2 + 2 * c) * 8;
    st_stream(pr, make_uint4(re[0], re[1], re[2], re[3]));
    st_stream(pr + 8, make_uint4(im[0], im[1], im[2], im[3]));
  }
}

// grid B * KW * nb (block index fastest), block p.threads, dynamic LDS pl.col_lds (hs = bs).
// Sx: the forward spectrum of x; Sg: that of g, replaced by the inverse side's gradient
// dX' = IDFT_H(dX) / c_kw (so that the C2R kernel's c_kw weights give the unit-weight
// transpose); modes: the four per-mode factor tensors, which the weight-product pass sums.
// wfrag: per block the words of W1x, W2x, W2x^T, W1x^T.  The two masks (relu, softshrink) stay
// in registers: every product of the kernel leaves the same four values with the same lane.
template <typename T, int SIZES, bool WIDE>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(WIDE ? 4 : 5)))
column_bwd_general(const T* __restrict__ Sx, T* __restrict__ Sg, const uint4* __restrict__ wfrag,
                   const T* __restrict__ b1, const T* __restrict__ b2, ColParams p,
                   T* __restrict__ modes, int64_t mpad, int W) {
  extern __shared__ float4 smem_raw[];
  const ColMem<T> mem(smem_raw, p);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int bs = p.bs, ldt = p.ldt, nb2 = 2 * bs;
  const int HC = col_bwd_hc(p.H16);
  T* tile = mem.tile;

  const int blk = blockIdx.x % p.nb;
  const int rest = blockIdx.x / p.nb;
  const int kw = rest % p.KW;
  const int64_t b = rest / p.KW;
  const uint32_t rsb = (uint32_t)p.KW * (uint32_t)p.C * 2 * (uint32_t)sizeof(T);
  const int64_t coff = ((b * p.H) * p.KW + kw) * (int64_t)p.C * 2 + (int64_t)blk * bs * 2;
  const CBuf<T> cx(Sx + coff, buf_bytes((uint64_t)p.H * rsb));
  const CBuf<T> cg(Sg + coff, buf_bytes((uint64_t)p.H * rsb));
  const int64_t m0 = (b * p.KW + kw) * (int64_t)HC;
  auto mode_tensor = [&](int t) { return modes + ((int64_t)t * p.nb + blk) * nb2 * mpad; };
  const float ckw = (kw == 0 || 2 * kw == W) ? 1.f : 2.f;

  const int wm = wave / p.wn, wn = wave % p.wn;
  const bool act = wm < p.wm;
  const uint32_t lbytes = (uint32_t)(bs * bs / 4) * 16u * (uint32_t)sizeof(T);  // one matrix's words
  const Buf wb(reinterpret_cast<const char*>(wfrag) + (int64_t)blk * 4 * lbytes, 4 * lbytes);
  auto mat = [&](int i) { return Words<T>{wb, i * lbytes, nullptr, 0}; };
  const int ks = nb2 / kstep<T>(), nt = nb2 / 16;
  constexpr int kMaxMW = 6;
  uint32_t mask[kMaxMW];  // per row tile: bit 4 n + r relu, bit 16 + 4 n + r softshrink

  make_twiddles(mem.roots(smem_raw), p.H);

  // X = F(x) column, then dz = c_kw F(g) column, by the same code
#pragma unroll 1
  for (int pass = 0; pass < 2; ++pass) {
    column_dft<T, SIZES>(pass ? cg : cx, rsb, mem, p, pass ? p.inv_sqrt_h * ckw : p.inv_sqrt_h);
    zero_pad_rows(tile, p);  // their factors meet zeros in the weight products' sums
    __syncthreads();
    if (pass == 0) {
      write_modes(tile, p, HC, mode_tensor(kModeX), m0);
      // h = relu(X W1 + b1) -> tile, mask v > 0
      with_grid<WIDE>(p, [&](auto MWc, auto NWc) {
        constexpr int MW = decltype(MWc)::value, NW = decltype(NWc)::value;
        f32x4 acc[MW][NW];
        if (act) column_product<T, MW, NW>(tile, ldt, mat(0), ks, nt, p, wm, wn, acc);
        __syncthreads();  // the tile's X rows are read (products and the X write)
        if (act) {
          f32x4 bias[NW];
#pragma unroll
          for (int n = 0; n < NW; ++n)
            bias[n] = ld_quad(b1 + (int64_t)blk * nb2 + 16 * (NW * wn + n) + 4 * (lane >> 4));
#pragma unroll
          for (int m = 0; m < MW; ++m) mask[m] = 0;
          each_quad<MW, NW>(p, wm, wn, [&](int m, int n, int row, int e0) {
            f32x4 v;
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              v[r] = acc[m][n][r] + bias[n][r];
              mask[m] |= (v[r] > 0.f ? 1u : 0u) << (4 * n + r);
              v[r] = fmaxf(v[r], 0.f);
            }
            st_quad(tile + row * ldt + e0, v);
          });
        }
      });
      __syncthreads();
      write_modes(tile, p, HC, mode_tensor(kModeH), m0);
      // layer 2: only its mask |o| > lam (and the cutoff) is needed
      with_grid<WIDE>(p, [&](auto MWc, auto NWc) {
        constexpr int MW = decltype(MWc)::value, NW = decltype(NWc)::value;
        if (!act) return;
        f32x4 acc[MW][NW];
        column_product<T, MW, NW>(tile, ldt, mat(1), ks, nt, p, wm, wn, acc);
        f32x4 bias[NW];
#pragma unroll
        for (int n = 0; n < NW; ++n)
          bias[n] = ld_quad(b2 + (int64_t)blk * nb2 + 16 * (NW * wn + n) + 4 * (lane >> 4));
        each_quad<MW, NW>(p, wm, wn, [&](int m, int n, int row, int) {
          const bool keep = row_kept(row, p.H, p.kept_h);
#pragma unroll
          for (int r = 0; r < 4; ++r)
            mask[m] |= (keep && fabsf(acc[m][n][r] + bias[n][r]) > p.lam ? 1u : 0u) << (16 + 4 * n + r);
        });
      });
      __syncthreads();  // the h rows are read (products and the h write)
    }
  }

  // do = dz masked; write do
  with_grid<WIDE>(p, [&](auto MWc, auto NWc) {
    constexpr int MW = decltype(MWc)::value, NW = decltype(NWc)::value;
    if (!act) return;
    each_quad<MW, NW>(p, wm, wn, [&](int m, int n, int row, int e0) {
      T* q = tile + row * ldt + e0;
      const float4 z = ld_c2(q);
      const uint32_t w = mask[m] >> (16 + 4 * n);
      st_quad(q, f32x4{w & 1 ? z.x : 0.f, w & 2 ? z.y : 0.f, w & 4 ? z.z : 0.f, w & 8 ? z.w : 0.f});
    });
  });
  zero_dead_rows(tile, p);
  __syncthreads();
  write_modes(tile, p, HC, mode_tensor(kModeDo), m0);

  // dv = (do W2^H) masked by v > 0, written; then dX = dv W1^H
#pragma unroll 1
  for (int pass = 0; pass < 2; ++pass) {
    with_grid<WIDE>(p, [&](auto MWc, auto NWc) {
      constexpr int MW = decltype(MWc)::value, NW = decltype(NWc)::value;
      f32x4 acc[MW][NW];
      if (act) column_product<T, MW, NW>(tile, ldt, mat(2 + pass), ks, nt, p, wm, wn, acc);
      __syncthreads();
      if (!act) return;
      each_quad<MW, NW>(p, wm, wn, [&](int m, int n, int row, int e0) {
        const uint32_t w = pass ? 15u : mask[m] >> (4 * n);
        st_quad(tile + row * ldt + e0, f32x4{w & 1 ? acc[m][n][0] : 0.f, w & 2 ? acc[m][n][1] : 0.f,
                                             w & 4 ? acc[m][n][2] : 0.f, w & 8 ? acc[m][n][3] : 0.f});
      });
    });
    __syncthreads();
    if (pass == 0) write_modes(tile, p, HC, mode_tensor(kModeDv), m0);
  }
  // -> inverse H-DFT -> Sg column / c_kw
  column_idft<T, SIZES>(cg, rsb, mem, p, p.inv_sqrt_h / ckw);
}

}  // namespace afno
