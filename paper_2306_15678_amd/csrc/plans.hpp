// plans.hpp -- compiled FFT tile variants of the row and column passes.
//
// Rows: X(N, variant, T, LINES, OPT, radices...); columns: X(N, variant,
// T, W, A, B, OPT, radices...).  OPT: 1 = late twiddles, 2 =
// the middle stage's in LDS (complex64, see MidTable), plus 0x100 times
// the wavefronts per SIMD the compiler must leave room for, 0x8000 = column
// exchanges through half the tile (see Plan).  T threads per line, LINES
// lines per workgroup (rows: LINES consecutive rows; columns: W adjacent
// columns, read as W * sizeof(complex) contiguous bytes per row), radix plan
// in stage order.  Column tiles keep point p of column c at LDS slot
// p W + c + (p / A) B: the padding (A, B) is chosen per plan to spread the
// stage exchanges over the LDS banks (64 banks of 4 bytes; a wave64 64-bit
// access served 32 lanes at a time).
//
// E = N/T points per thread.  Up to 1024^2 a pass is one generation of
// workgroups and its time is the chain load, transforms, store of one of
// them: 4 or 8 points a thread keep that chain short (128^2, us per step:
// E = 4 4.4, E = 8 5.0, E = 16 6.7; 256^2: E = 4 5.5, E = 8 6.0, E = 16 7.3;
// 1024^2 rows: E = 8 11.2, E = 16 12.1).  From 2048^2 on the vector units
// decide and the larger radices of 16 points a thread, fewest instructions,
// win (4096^2 rows: 16 points 84 us, 8 points 105 us).
#pragma once

#include "fft_core.hpp"

namespace ssfm {

#define SSFM_ROW_PLANS(X) \
  X(128, 0, 32, 2, 0x0, 4, 4, 4, 2) \
  X(128, 1, 16, 4, 0x0, 8, 4, 4) \
  X(256, 0, 64, 1, 0x0, 4, 4, 4, 4) \
  X(256, 1, 32, 2, 0x0, 8, 8, 4) \
  X(256, 2, 16, 4, 0x1, 16, 16) \
  X(512, 0, 64, 1, 0x0, 8, 8, 8) \
  X(512, 1, 128, 1, 0x0, 4, 4, 4, 4, 2) \
  X(768, 0, 64, 1, 0x0, 12, 4, 4, 4) \
  X(768, 1, 64, 1, 0x1, 12, 4, 4, 4) \
  X(768, 2, 64, 1, 0x0, 4, 4, 4, 4, 3) \
  X(1024, 0, 128, 1, 0x0, 8, 8, 4, 4) \
  X(1024, 1, 256, 1, 0x0, 4, 4, 4, 4, 4) \
  X(1024, 2, 128, 1, 0x1, 8, 8, 4, 4) \
  X(1024, 3, 64, 1, 0x3, 16, 8, 8) \
  X(2048, 0, 256, 1, 0x0, 8, 8, 8, 4) \
  X(2048, 1, 256, 1, 0x1, 8, 8, 8, 4) \
  X(2048, 2, 128, 1, 0x403, 16, 16, 8) \
  X(2048, 3, 128, 1, 0x3, 16, 16, 8) \
  X(4096, 0, 256, 1, 0x403, 16, 16, 16) \
  X(4096, 1, 256, 1, 0x3, 16, 16, 16) \
  X(4096, 2, 256, 1, 0x303, 16, 16, 16) \
  X(4096, 3, 256, 1, 0x203, 16, 16, 16) \
  X(4096, 4, 512, 1, 0x0, 8, 8, 8, 8) \
  X(4096, 5, 512, 1, 0x1, 8, 8, 8, 8) \
  X(4096, 6, 512, 1, 0x401, 8, 8, 8, 8) \
  X(4096, 7, 512, 1, 0x300, 8, 8, 8, 8) \
  X(4096, 8, 256, 1, 0x503, 16, 16, 16)

#define SSFM_COL_PLANS(X) \
  X(128, 0, 32, 2, 16, 6, 0x0, 4, 4, 4, 2) \
  X(128, 1, 32, 4, 8, 4, 0x0, 4, 4, 4, 2) \
  X(128, 2, 16, 4, 8, 4, 0x0, 8, 4, 4) \
  X(256, 0, 64, 2, 16, 6, 0x0, 4, 4, 4, 4) \
  X(256, 1, 64, 4, 8, 4, 0x0, 4, 4, 4, 4) \
  X(256, 2, 32, 2, 16, 2, 0x0, 8, 8, 4) \
  X(256, 3, 16, 4, 8, 4, 0x1, 16, 16) \
  X(256, 4, 16, 8, 4, 2, 0x1, 16, 16) \
  X(512, 0, 128, 2, 16, 6, 0x0, 4, 4, 4, 4, 2) \
  X(512, 1, 64, 2, 16, 2, 0x0, 8, 8, 8) \
  X(512, 2, 64, 4, 8, 4, 0x0, 8, 8, 8) \
  X(512, 3, 64, 1, 32, 3, 0x0, 8, 8, 8) \
  X(768, 0, 64, 4, 32, 4, 0x0, 12, 4, 4, 4) \
  X(768, 1, 64, 2, 32, 1, 0x0, 12, 4, 4, 4) \
  X(768, 2, 64, 4, 32, 4, 0x1, 12, 4, 4, 4) \
  X(768, 3, 64, 2, 16, 6, 0x0, 4, 4, 4, 4, 3) \
  X(1024, 0, 128, 4, 8, 4, 0x0, 8, 8, 4, 4) \
  X(1024, 1, 128, 2, 16, 2, 0x0, 8, 8, 4, 4) \
  X(1024, 2, 256, 2, 16, 6, 0x0, 4, 4, 4, 4, 4) \
  X(1024, 3, 64, 4, 8, 2, 0x0, 16, 8, 8) \
  X(1024, 4, 64, 4, 8, 2, 0x3, 16, 8, 8) \
  X(1024, 5, 128, 4, 8, 4, 0x1, 8, 8, 4, 4) \
  X(2048, 0, 128, 4, 8, 2, 0x403, 16, 16, 8) \
  X(2048, 1, 256, 2, 16, 2, 0x0, 8, 8, 8, 4) \
  X(2048, 2, 128, 8, 4, 2, 0x403, 16, 16, 8) \
  X(2048, 3, 128, 2, 16, 2, 0x403, 16, 16, 8) \
  X(2048, 4, 256, 4, 8, 4, 0x401, 8, 8, 8, 4) \
  X(4096, 0, 256, 2, 16, 2, 0x403, 16, 16, 16) \
  X(4096, 1, 256, 4, 8, 2, 0x403, 16, 16, 16) \
  X(4096, 2, 256, 2, 16, 2, 0x303, 16, 16, 16) \
  X(4096, 3, 256, 2, 16, 2, 0x3, 16, 16, 16) \
  X(4096, 4, 128, 4, 16, 2, 0x8402, 16, 16, 16) \
  X(4096, 5, 128, 4, 8, 2, 0x8402, 16, 16, 16) \
  X(4096, 6, 512, 2, 16, 2, 0x0, 8, 8, 8, 8) \
  X(4096, 7, 512, 2, 16, 2, 0x401, 8, 8, 8, 8) \
  X(4096, 8, 128, 4, 8, 2, 0x8202, 16, 16, 16) \
  X(4096, 9, 128, 2, 16, 2, 0x8402, 16, 16, 16) \
  X(4096, 10, 256, 4, 8, 4, 0x8400, 8, 8, 8, 8)

// LDS of a pass workgroup against the 160 KiB a gfx950 workgroup may
// allocate; half-exchange plans are built for complex64 columns only.
constexpr size_t kMaxLdsBytes = 160 * 1024;
template <typename R, class P>
constexpr size_t plan_lds_bytes(bool column) {
  const size_t tile =
      column ? size_t(LdsPointMajor<R, P::LINES, P::PA, P::PB>::size(P::HX ? P::N / 2 : P::N))
             : size_t(P::LINES) * LdsLineMajor<R, P::N>::LINE;
  return ((tile + 1) / 2 * 2 + mid_table_size<R, P>()) * sizeof(cx<R>);
}
template <typename R, class P>
constexpr bool plan_fits(bool column) {
  return plan_lds_bytes<R, P>(column) <= kMaxLdsBytes &&
         !(P::HX && (sizeof(R) != 4 || !column));
}

template <int N, int V>
struct RowPlanSel;
template <int N, int V>
struct ColPlanSel;

#define SSFM_DEF_ROW(NN, VV, TT, LL, OO, ...) \
  template <> struct RowPlanSel<NN, VV> { using P = Plan<NN, TT, LL, Radices<__VA_ARGS__>, 32, 0, OO>; };
#define SSFM_DEF_COL(NN, VV, TT, LL, AA, BB, OO, ...) \
  template <> struct ColPlanSel<NN, VV> { using P = Plan<NN, TT, LL, Radices<__VA_ARGS__>, AA, BB, OO>; };
SSFM_ROW_PLANS(SSFM_DEF_ROW)
SSFM_COL_PLANS(SSFM_DEF_COL)
#undef SSFM_DEF_ROW
#undef SSFM_DEF_COL

}  // namespace ssfm
