// afno_rows.hip -- the size-specialised W-axis passes (row_r2c_fast, row_c2r_fast) for every
// even 5-smooth width from 12 to 576: how each width is split, and the launches.
//
// This is the library's largest set of kernels, so a parallel build compiles it in four parts
// (AFNO_ROWS_PART 0 to 3: direction and storage type; the launchers of the other parts are then
// external).  Without AFNO_ROWS_PART all four are compiled, included by afno_kernels.hip.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "afno_internal.h"
#include "kernels_fast.h"

namespace afno {

// W = n1 n2: n2 strided samples per thread in the first stage, n1 in the second, np signals
// (2 np channels) per workgroup of np n1 threads.  Measured on 32 Mi elements with C = 512,
// every split of every third width or so in both storage types (us per pass, bf16; a copy of
// the same bytes takes 27 forward and 41 inverse):
//  * forward: np = 32 fills a 128-byte line per position in bf16 and is 3 to 5 us faster than
//    16 wherever the workgroup stays small: at most 8 n1 (9 up to W = 144; W = 162 as 9 x 18
//    takes 39.6, 160 as 8 x 20 30.6).  Without such a divisor np = 16 and n1 <= n2, the second
//    stage holding 2 n1 values: 12 x 15 33.9 against 15 x 12 41.0, 15 x 24 36.3 against 18 x 20
//    49.7; the few widths that need n1 > 16 take np = 32 (18 x 32: 44.9 against 50.8).
//  * inverse: one value set per thread and stage, so the longer factor goes on the threads:
//    up to W = 300 np = 32 with the largest n1 <= 16 (16 x 4 36.9 against 8 x 8 41.0), unless
//    that leaves n2 > 16 beside a short n1 (216: 18 x 12 at np 16 46.7, 12 x 18 at 32 55.1);
//    up to 400 the same at np = 16 (360 as 15 x 24: 85 us on 66 Mi elements, 24 x 15 90);
//    above, np = 16 and n2 <= 16 where it divides (32 x 16 46.3 against 16 x 32 49.6).
struct RowSplit { int n1, n2, np; };

constexpr RowSplit row_split_fwd(int W) {
  for (int n1 = W <= 144 ? 9 : 8; n1 >= 3; --n1)
    if (W % n1 == 0 && W / n1 >= 4 && W / n1 <= (n1 == 8 ? 32 : 25)) return {n1, W / n1, 32};
  for (int n1 = 16; n1 >= 9; --n1)
    if (W % n1 == 0 && W / n1 >= n1 && W / n1 <= 32) return {n1, W / n1, 16};
  for (int n1 = 17; n1 <= 24; ++n1)
    if (W % n1 == 0 && W / n1 <= 32) return {n1, W / n1, 32};
  return {0, 0, 0};
}
constexpr RowSplit row_split_inv(int W) {
  for (int n1 = 16; n1 >= 3 && W <= 400; --n1)
    if (W % n1 == 0 && W / n1 >= 4) {
      if (W / n1 > 16 && n1 <= 12) return {W / n1, n1, 16};
      return {n1, W / n1, W <= 300 ? 32 : 16};
    }
  for (int n2 = 16; n2 >= 10; --n2)
    if (W % n2 == 0 && W / n2 <= 32) return {W / n2, n2, 16};
  for (int n2 = 17; n2 <= 24; ++n2)
    if (W % n2 == 0 && W / n2 <= 32) return {W / n2, n2, 16};
  return {0, 0, 0};
}

#define AFNO_ROW_WIDTHS(X)                                                                       \
  X(12) X(16) X(18) X(20) X(24) X(30) X(32) X(36) X(40) X(48) X(50) X(54) X(60) X(64) X(72)      \
  X(80) X(90) X(96) X(100) X(108) X(120) X(128) X(144) X(150) X(160) X(162) X(180) X(192) X(200) \
  X(216) X(240) X(250) X(256) X(270) X(288) X(300) X(320) X(324) X(360) X(384) X(400) X(432)     \
  X(450) X(480) X(486) X(500) X(512) X(540) X(576)

// pj.tout / pj.wout null: no preparation job; else its ntask tasks go to extra workgroups
template <typename T>
void launch_row_fwd_fast(const Plan& pl, const T* x, T* S, PrepJob<T> pj, int64_t ntask,
                         hipStream_t st) {
  const int64_t rows = pl.B * pl.H;
  const float sc = 0.5f * pl.row.inv_sqrt_w;
  switch (pl.W) {
#define AFNO_CASE(w)                                                                             \
  case w: {                                                                                      \
    constexpr RowSplit sp = row_split_fwd(w);                                                    \
    constexpr int nt = sp.np * sp.n1;                                                            \
    static_assert(sp.n1 * sp.n2 == w, "no split for this width");                                \
    const unsigned nmain = (unsigned)row_grid<sp.np, (int)sizeof(T)>(rows, pl.C);                \
    pj.nprep = pj.wout ? (int)((std::min<int64_t>((ntask + nt - 1) / nt, 1024) + 7) / 8 * 8) : 0; \
    hipLaunchKernelGGL((row_r2c_fast<T, w, sp.n1, sp.n2, sp.np>), dim3(pj.nprep + nmain),        \
                       dim3(nt), 0, st, x, S, (int)pl.C, (int)pl.KW, sc, rows, pj);              \
    return;                                                                                      \
  }
    AFNO_ROW_WIDTHS(AFNO_CASE)
#undef AFNO_CASE
  }
}

template <typename T>
void launch_row_inv_fast(const Plan& pl, const T* S, const T* x, T* out, float* dst, int mode,
                         hipStream_t st) {
  const int64_t rows = pl.B * pl.H;
  const float sc = pl.row.inv_sqrt_w;
  switch (pl.W) {
#define AFNO_CASE(w)                                                                             \
  case w: {                                                                                      \
    constexpr RowSplit sp = row_split_inv(w);                                                    \
    static_assert(sp.n1 * sp.n2 == w, "no split for this width");                                \
    const unsigned ng = (unsigned)row_grid<sp.np, (int)sizeof(T)>(rows, pl.C);                   \
    hipLaunchKernelGGL((row_c2r_fast<T, w, sp.n1, sp.n2, sp.np>), dim3(ng), dim3(sp.np * sp.n1), \
                       0, st, S, x, out, dst, (int)pl.C, (int)pl.KW, sc, mode, rows);            \
    return;                                                                                      \
  }
    AFNO_ROW_WIDTHS(AFNO_CASE)
#undef AFNO_CASE
  }
}

#ifndef AFNO_ROWS_PART
#define AFNO_ROWS_PART -1
#endif
#define AFNO_INST_FWD(T)                                                                        \
  template void launch_row_fwd_fast<T>(const Plan&, const T*, T*, PrepJob<T>, int64_t, hipStream_t);
#define AFNO_INST_INV(T)                                                                        \
  template void launch_row_inv_fast<T>(const Plan&, const T*, const T*, T*, float*, int, hipStream_t);
#if AFNO_ROWS_PART < 0 || AFNO_ROWS_PART == 0
AFNO_INST_FWD(bf16)
// A width with a split whose byte offsets from a slice's first row stay in 32 bits.  A row alone
// always does (a grid row and a spectrum column span at most 4 GiB), and a slice stays in one row
// where C is a multiple of 2 np in both directions.  A slice that runs on covers two rows if C is
// at least 2 np, at most 2 (W / 2 + 1) C 8 = (W + 2) 8 C bytes of the spectrum, below 2^32 for
// W C < 2^28; with fewer channels it covers up to four rows of at most 576 x 48 values.
bool fast_row_available(int64_t W, int64_t C) {
  int np = 0;
#define AFNO_CASE(w) if (W == w) np = std::max(row_split_fwd(w).np, row_split_inv(w).np);
  AFNO_ROW_WIDTHS(AFNO_CASE)
#undef AFNO_CASE
  return np > 0 && (C % (2 * np) == 0 || W * C < ((int64_t)1 << 28));
}
#endif
#if AFNO_ROWS_PART < 0 || AFNO_ROWS_PART == 1
AFNO_INST_FWD(float)
#endif
#if AFNO_ROWS_PART < 0 || AFNO_ROWS_PART == 2
AFNO_INST_INV(bf16)
#endif
#if AFNO_ROWS_PART < 0 || AFNO_ROWS_PART == 3
AFNO_INST_INV(float)
#endif
#undef AFNO_INST_FWD
#undef AFNO_INST_INV

}  // namespace afno
