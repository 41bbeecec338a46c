// fft_core.hpp -- register/LDS Stockham FFT building blocks for gfx950.
//
// A "line" is one row or one column of the transverse grid (the split-step
// diffraction operator of Eq. (1) factorises exactly into a row operator and
// a column operator, each diagonal in its own 1-D Fourier basis).  T threads
// cooperate on a line of N points; thread t holds the E = N/T points
// t + T*e (e = 0..E-1) in registers.  Each radix stage of the
// self-sorting (Stockham, decimation-in-time) FFT computes N/R butterflies
// of radix R; thread t owns butterflies j = t + T*b (b < E/R).
//
//   stage with span Ns (1, R0, R0*R1, ...):
//     inputs    x[j + r*N/R]                       r = 0..R-1
//     twiddle   w^(r * (j mod Ns) * N/(Ns*R)),     w = exp(dir 2 pi i / N)
//     DFT_R
//     outputs   y[(j div Ns)*Ns*R + (j mod Ns) + r*Ns]
//
// The inputs of the first stage and the outputs of the last stage are
// exactly the thread's own register points, so an FFT needs LDS only
// between stages, and FFT -> pointwise multiply -> inverse FFT needs no LDS
// traffic at the junction.  Twiddles come from a table in stage order
// computed in FP64 on the host and rounded once; a thread with few points
// loads the ones it needs once and keeps them in registers, one with many
// loads them stage by stage or takes part of them from LDS.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

namespace ssfm {

template <typename R>
struct cx {
  R re, im;
};

// A stretch of memory read and written through a buffer descriptor: element
// i + c, i per thread, c the same for all.  A thread's elements lie at
// compile-time distances; the instruction takes those as a scalar offset, so
// they cost no vector instruction (flat addresses took one or two an access,
// 8 to 10 % of a pass).
template <typename T>
struct Buf {
  typedef uint32_t U2 __attribute__((ext_vector_type(2)));
  typedef uint32_t U4 __attribute__((ext_vector_type(4)));
  static constexpr int S = int(sizeof(T));
  static_assert(S == 4 || S == 8 || S == 16, "dword, two or four dwords");
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ explicit Buf(const T* p)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p), 0, -1, 0x00020000)) {}
  __device__ __forceinline__ T get(uint32_t i, uint32_t c) const {
    const uint32_t v = i * uint32_t(S), k = c * uint32_t(S);
    if constexpr (S == 4)
      return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, int(v), int(k), 0));
    else if constexpr (S == 8)
      return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, int(v), int(k), 0));
    else
      return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b128(r, int(v), int(k), 0));
  }
  __device__ __forceinline__ void put(uint32_t i, uint32_t c, T x) const {
    const uint32_t v = i * uint32_t(S), k = c * uint32_t(S);
    if constexpr (S == 4)
      __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(uint32_t, x), r, int(v), int(k), 0);
    else if constexpr (S == 8)
      __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U2, x), r, int(v), int(k), 0);
    else
      __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(U4, x), r, int(v), int(k), 0);
  }
};

template <typename R>
__device__ __forceinline__ cx<R> operator+(cx<R> a, cx<R> b) {
  return {a.re + b.re, a.im + b.im};
}
template <typename R>
__device__ __forceinline__ cx<R> operator-(cx<R> a, cx<R> b) {
  return {a.re - b.re, a.im - b.im};
}
__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }
// Products with the fused operation spelled out: the compiler is left no
// choice of which product to round, so every kernel forms the same bits.
template <typename R>
__device__ __forceinline__ cx<R> cmul(cx<R> a, cx<R> b) {
  return {fma_(a.re, b.re, -(a.im * b.im)), fma_(a.re, b.im, a.im * b.re)};
}
// a * conj(b)
template <typename R>
__device__ __forceinline__ cx<R> cmulc(cx<R> a, cx<R> b) {
  return {fma_(a.re, b.re, a.im * b.im), fma_(a.im, b.re, -(a.re * b.im))};
}
template <typename R>
__device__ __forceinline__ cx<R> conjg(cx<R> a) {
  return {a.re, -a.im};
}
// multiply by (dir * i): dir = -1 gives -i, dir = +1 gives +i
template <int DIR, typename R>
__device__ __forceinline__ cx<R> rot_q(cx<R> a) {
  if constexpr (DIR < 0) {
    return {a.im, -a.re};
  } else {
    return {-a.im, a.re};
  }
}
// a + s b
template <typename R>
__device__ __forceinline__ cx<R> axpy(cx<R> a, R s, cx<R> b) {
  return {fma_(s, b.re, a.re), fma_(s, b.im, a.im)};
}
// a + b w (DIR < 0) or a + b conj(w): 4 fused operations
template <int DIR, typename R>
__device__ __forceinline__ cx<R> cfma(cx<R> a, cx<R> b, cx<R> w) {
  if constexpr (DIR < 0)
    return {fma_(-b.im, w.im, fma_(b.re, w.re, a.re)), fma_(b.re, w.im, fma_(b.im, w.re, a.im))};
  else
    return {fma_(b.im, w.im, fma_(b.re, w.re, a.re)), fma_(-b.re, w.im, fma_(b.im, w.re, a.im))};
}
// b w or b conj(w)
template <int DIR, typename R>
__device__ __forceinline__ cx<R> twist(cx<R> b, cx<R> w) {
  return (DIR > 0) ? cmulc(b, w) : cmul(b, w);
}
// 2 a - b
template <typename R>
__device__ __forceinline__ cx<R> other(cx<R> a, cx<R> b) {
  return {fma_(R(2), a.re, -b.re), fma_(R(2), a.im, -b.im)};
}
// sqrt(2) a exp(dir i pi/4) and sqrt(2) a exp(3 dir i pi/4): the scale
// 1/sqrt(2) is left to the fused operations that add the result
template <int DIR, typename R>
__device__ __forceinline__ cx<R> rot_8s(cx<R> a) {
  if constexpr (DIR < 0)
    return {a.re + a.im, a.im - a.re};
  else
    return {a.re - a.im, a.im + a.re};
}
template <int DIR, typename R>
__device__ __forceinline__ cx<R> rot_38s(cx<R> a) {
  if constexpr (DIR < 0)
    return {a.im - a.re, -(a.re + a.im)};
  else
    return {-(a.re + a.im), a.re - a.im};
}

// ---------------------------------------------------------------- DFTs
// In-place DFT of RAD points in natural order: y_k = sum_n x_n w^(nk),
// w = exp(dir 2 pi i / RAD).  The TW forms take x_n w_n instead of x_n, with
// the stage twiddles tw[n - 1] = w_n (n > 0; conjugated for DIR > 0).
//
// Operation counts decide the large grids (their passes keep the vector
// units 85-90 % busy), so everything is arranged for fused multiply-adds:
// a twiddled butterfly a + w b, a - w b is formed as t = a + w b (4 fused
// operations) and 2 a - t (2), instead of 4 for the product and 4 for the
// sums; a rotation by a constant leaves its scale to the fused operations
// that add it.  Per radix-16 stage 188 operations instead of 220, radix 8
// 72 instead of 84, radix 4 24 instead of 28, with no more roundings on the
// way to any output.

// s a, rounded by itself
template <typename R>
__device__ __forceinline__ cx<R> scaled(cx<R> a, R s) {
#pragma clang fp contract(off)
  return {a.re * s, a.im * s};
}
// Half of a radix-4 butterfly's rest: from t0, t1 = x0 +- x2 and s u, s w
// with u = x1 + x3, w = rot(x1 - x3) over the scale s.  complex128 rounds
// the products by themselves: the march against its oracle is closer so
// (100 steps of a 256^2 gradient: 4.8e-13, fused 5.7e-13).
template <typename R>
__device__ __forceinline__ void dft4_tail(cx<R> t0, cx<R> t1, cx<R> u, cx<R> w, R s, cx<R>& a0,
                                          cx<R>& a1, cx<R>& a2, cx<R>& a3) {
  if constexpr (sizeof(R) == 8) {
    u = scaled(u, s);
    w = scaled(w, s);
    a0 = t0 + u;
    a2 = t0 - u;
    a1 = t1 + w;
    a3 = t1 - w;
  } else {
    a0 = axpy(t0, s, u);
    a2 = axpy(t0, -s, u);
    a1 = axpy(t1, s, w);
    a3 = axpy(t1, -s, w);
  }
}

template <int DIR, typename R>
__device__ __forceinline__ void dft4_(cx<R>& a0, cx<R>& a1, cx<R>& a2,
                                      cx<R>& a3) {
  cx<R> t0 = a0 + a2, t1 = a0 - a2, t2 = a1 + a3;
  cx<R> t3 = rot_q<DIR>(a1 - a3);
  a0 = t0 + t2;
  a2 = t0 - t2;
  a1 = t1 + t3;
  a3 = t1 - t3;
}

// radix 4 of x0, a1 w1, a2 w2, a3 w3 (x0 twiddled by the caller)
template <int DIR, typename R>
__device__ __forceinline__ void dft4_tw_(cx<R>& a0, cx<R>& a1, cx<R>& a2, cx<R>& a3, cx<R> w1,
                                         cx<R> w2, cx<R> w3) {
  const cx<R> t0 = cfma<DIR>(a0, a2, w2), t1 = other(a0, t0);
  const cx<R> x1 = twist<DIR>(a1, w1);
  const cx<R> t2 = cfma<DIR>(x1, a3, w3), t3 = rot_q<DIR>(other(x1, t2));
  a0 = t0 + t2;
  a2 = t0 - t2;
  a1 = t1 + t3;
  a3 = t1 - t3;
}

template <int DIR, bool TW, typename R>
__device__ __forceinline__ void dft2(cx<R>* v, const cx<R>* w) {
  if constexpr (TW) {
    const cx<R> t = cfma<DIR>(v[0], v[1], w[0]);
    v[1] = other(v[0], t);
    v[0] = t;
  } else {
    const cx<R> a = v[0];
    v[0] = a + v[1];
    v[1] = a - v[1];
  }
}

template <int DIR, typename R>
__device__ __forceinline__ void dft3(cx<R>* v) {
  const R h = R(0.86602540378443864676);  // sqrt(3)/2
  const cx<R> t = v[1] + v[2];
  const cx<R> u = rot_q<DIR>(v[1] - v[2]);
  const cx<R> m = axpy(v[0], R(-0.5), t);
  v[0] = v[0] + t;
  v[1] = axpy(m, h, u);
  v[2] = axpy(m, -h, u);
}

template <int DIR, bool TW, typename R>
__device__ __forceinline__ void dft4(cx<R>* v, const cx<R>* w) {
  if constexpr (TW)
    dft4_tw_<DIR>(v[0], v[1], v[2], v[3], w[0], w[1], w[2]);
  else
    dft4_<DIR>(v[0], v[1], v[2], v[3]);
}

template <int DIR, bool TW, typename R>
__device__ __forceinline__ void dft8(cx<R>* v, const cx<R>* w) {
  const R h = R(0.70710678118654752440);
  cx<R> b[4], c[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if constexpr (TW) {
      const cx<R> x = (i == 0) ? v[0] : twist<DIR>(v[i], w[i == 0 ? 0 : i - 1]);
      b[i] = cfma<DIR>(x, v[i + 4], w[i + 3]);
      c[i] = other(x, b[i]);
    } else {
      b[i] = v[i] + v[i + 4];
      c[i] = v[i] - v[i + 4];
    }
  }
  dft4_<DIR>(b[0], b[1], b[2], b[3]);  // even outputs
  // odd outputs: radix 4 of c0, c1 w8, c2 w8^2, c3 w8^3
  const cx<R> c2 = rot_q<DIR>(c[2]);
  const cx<R> p = rot_8s<DIR>(c[1]), q = rot_38s<DIR>(c[3]);
  dft4_tail(c[0] + c2, c[0] - c2, p + q, rot_q<DIR>(p - q), h, v[1], v[3], v[5], v[7]);
  v[0] = b[0];
  v[2] = b[1];
  v[4] = b[2];
  v[6] = b[3];
}

// 16 = 4 x 4: inner DFT4 over n2 (stride 4), twiddle w16^(n1 k2), outer
// DFT4 over n1; output index k2 + 4 k1.
template <int DIR, bool TW, typename R>
__device__ __forceinline__ void dft16(cx<R>* v, const cx<R>* w) {
  const R h = R(0.70710678118654752440);
  const R c1 = R(0.92387953251128675613);              // cos(pi/8)
  const R tau = R(DIR * 0.41421356237309504880);       // dir tan(pi/8)
  const R tq = R(0.41421356237309504880), d = R(DIR);
#pragma unroll
  for (int n1 = 0; n1 < 4; ++n1) {
    if constexpr (TW) {
      if (n1 > 0) v[n1] = twist<DIR>(v[n1], w[n1 > 0 ? n1 - 1 : 0]);
      dft4_tw_<DIR>(v[n1], v[n1 + 4], v[n1 + 8], v[n1 + 12], w[n1 + 3], w[n1 + 7], w[n1 + 11]);
    } else {
      dft4_<DIR>(v[n1], v[n1 + 4], v[n1 + 8], v[n1 + 12]);
    }
  }
  // v[n1 + 4 k2]; over the scale c1: a w16 and a w16^3 (2 operations each)
  auto w16 = [&](cx<R> a) { return cx<R>{fma_(-tau, a.im, a.re), fma_(tau, a.re, a.im)}; };
  auto w16_3 = [&](cx<R> a) { return cx<R>{fma_(tq, a.re, -d * a.im), fma_(tq, a.im, d * a.re)}; };
  cx<R> y[16];
  dft4_<DIR>(v[0], v[1], v[2], v[3]);
#pragma unroll
  for (int k1 = 0; k1 < 4; ++k1) y[4 * k1] = v[k1];
  {  // k2 = 1: w16^(0, 1, 2, 3)
    const cx<R> p = rot_8s<DIR>(v[6]);
    const cx<R> t0 = axpy(v[4], h, p), t1 = axpy(v[4], -h, p);
    const cx<R> b = w16(v[5]), e = w16_3(v[7]);
    dft4_tail(t0, t1, b + e, rot_q<DIR>(b - e), c1, y[1], y[5], y[9], y[13]);
  }
  {  // k2 = 2: w16^(0, 2, 4, 6)
    const cx<R> r = rot_q<DIR>(v[10]);
    const cx<R> p = rot_8s<DIR>(v[9]), q = rot_38s<DIR>(v[11]);
    dft4_tail(v[8] + r, v[8] - r, p + q, rot_q<DIR>(p - q), h, y[2], y[6], y[10], y[14]);
  }
  {  // k2 = 3: w16^(0, 3, 6, 9), w16^9 = -w16
    const cx<R> q = rot_38s<DIR>(v[14]);
    const cx<R> t0 = axpy(v[12], h, q), t1 = axpy(v[12], -h, q);
    const cx<R> b = w16_3(v[13]), e = w16(v[15]);
    dft4_tail(t0, t1, b - e, rot_q<DIR>(b + e), c1, y[3], y[7], y[11], y[15]);
  }
#pragma unroll
  for (int k = 0; k < 16; ++k) v[k] = y[k];
}

// 12 = 4 x 3: inner DFT4 over n2 (points n1 + 3 n2), twiddle w12^(n1 k2),
// outer DFT3 over n1; output index k2 + 4 k1.
template <int DIR, bool TW, typename R>
__device__ __forceinline__ void dft12(cx<R>* v, const cx<R>* w) {
  constexpr double h = 0.86602540378443864676;  // cos(pi/6)
  cx<R> t[3][4];
#pragma unroll
  for (int n1 = 0; n1 < 3; ++n1) {
#pragma unroll
    for (int n2 = 0; n2 < 4; ++n2) t[n1][n2] = v[n1 + 3 * n2];
    if constexpr (TW) {
      if (n1 > 0) t[n1][0] = twist<DIR>(t[n1][0], w[n1 > 0 ? n1 - 1 : 0]);
      dft4_tw_<DIR>(t[n1][0], t[n1][1], t[n1][2], t[n1][3], w[n1 + 2], w[n1 + 5], w[n1 + 8]);
    } else {
      dft4_<DIR>(t[n1][0], t[n1][1], t[n1][2], t[n1][3]);
    }
  }
  // w12^1, w12^2, w12^3 = dir i; w12^2, w12^4, w12^6 = -1
  t[1][1] = cmul(t[1][1], cx<R>{R(h), R(DIR * 0.5)});
  t[1][2] = cmul(t[1][2], cx<R>{R(0.5), R(DIR * h)});
  t[1][3] = rot_q<DIR>(t[1][3]);
  t[2][1] = cmul(t[2][1], cx<R>{R(0.5), R(DIR * h)});
  t[2][2] = cmul(t[2][2], cx<R>{R(-0.5), R(DIR * h)});
  t[2][3] = cx<R>{-t[2][3].re, -t[2][3].im};
#pragma unroll
  for (int k2 = 0; k2 < 4; ++k2) {
    cx<R> g[3] = {t[0][k2], t[1][k2], t[2][k2]};
    dft3<DIR>(g);
#pragma unroll
    for (int k1 = 0; k1 < 3; ++k1) v[k2 + 4 * k1] = g[k1];
  }
}

// radix RAD with (TW) or without stage twiddles
template <int RAD, int DIR, bool TW, typename R>
__device__ __forceinline__ void dft(cx<R>* v, const cx<R>* w) {
  if constexpr (RAD == 2) dft2<DIR, TW>(v, w);
  else if constexpr (RAD == 3) {
    if constexpr (TW) {
      v[1] = twist<DIR>(v[1], w[0]);
      v[2] = twist<DIR>(v[2], w[1]);
    }
    dft3<DIR>(v);
  }
  else if constexpr (RAD == 4) dft4<DIR, TW>(v, w);
  else if constexpr (RAD == 8) dft8<DIR, TW>(v, w);
  else if constexpr (RAD == 12) dft12<DIR, TW>(v, w);
  else if constexpr (RAD == 16) dft16<DIR, TW>(v, w);
  else static_assert(RAD == 2, "unsupported radix");
}

// ------------------------------------------------------------ plans
template <int... Rs>
struct Radices {};

template <int R0, int... Rest>
constexpr int first_radix() {
  return R0;
}

// N points per line, T threads per line, LINES lines per workgroup; column
// tiles pad their LDS by B slots every A points (see LdsPointMajor).  OPT:
// bit 0 set loads each stage's twiddles just before that stage (fewer live
// registers) instead of all of them before the first; bit 1 has the middle
// stage's in LDS and the last stage's in registers (three stages, complex64;
// see MidTable); bits 8-11 give the
// wavefronts per SIMD the compiler must leave room for in the complex64
// kernels (0: no target), bits 12-14 the same for the complex128 ones; bit
// 15 makes a column pass exchange through half its tile (hx_stages),
// complex64 only.
template <int N_, int T_, int LINES_, class Rad, int PA_ = 32, int PB_ = 0, int OPT_ = 0>
struct Plan {
  static constexpr int N = N_;
  static constexpr int T = T_;
  static constexpr int LINES = LINES_;
  static constexpr int E = N_ / T_;
  static constexpr int THREADS = T_ * LINES_;
  static constexpr int WAVES = (THREADS + 63) / 64;
  static constexpr int PA = PA_;
  static constexpr int PB = PB_;
  static constexpr bool LATE_TW = (OPT_ & 1) != 0;
  static constexpr bool MID_TW = (OPT_ & 2) != 0;  // complex64 (see MidTable)
  static constexpr int WAVES_PER_EU = ((OPT_ >> 8) & 15) ? ((OPT_ >> 8) & 15) : 1;
  static constexpr int WAVES_PER_EU_F64 = ((OPT_ >> 12) & 7) ? ((OPT_ >> 12) & 7) : 1;
  static constexpr bool HX = (OPT_ & 0x8000) != 0;
  using radices = Rad;
  static_assert(N_ % T_ == 0, "T must divide N");
  static_assert(THREADS % 64 == 0, "whole wavefronts");
};

// --------------------------------------------------------- LDS layouts
// Row lines: line-major with 3 pad slots per 32 points (complex64; per 16,
// complex128), which a bank model (64 banks of 4 bytes, a wavefront's 8- and
// 16-byte accesses served 32 and 16 lanes at a time) gives 1.0-1.3 cycles
// per served group over all stages of the radix 4, 8 and 16 plans.
//
// Both layouts map point p to slot idx(p), a sum of floors of p by powers of
// two: for points p, q without a common bit idx(p + q) = idx(p) + idx(q).
// The stages use that: a thread's slots are one computed index plus
// compile-time offsets, which fold into the LDS instructions (one by one
// the indices took a quarter to a third of the column passes' instructions).
template <typename R, int N>
struct LdsLineMajor {
  static constexpr int A = sizeof(R) == 4 ? 32 : 16;
  static constexpr int LINE = N + N / A * 3;
  static constexpr __device__ __host__ unsigned idx(unsigned p) { return p + p / A * 3u; }
  cx<R>* base;
  __device__ __forceinline__ cx<R>& slot(unsigned i) const { return base[i]; }
};

// Column tiles: point-major, the W columns of a point adjacent, B padding
// slots after every A points (complex64; half of both for complex128, whose
// elements span twice the banks).
template <typename R, int W, int A_, int B_>
struct LdsPointMajor {
  static constexpr bool HALF = sizeof(R) == 8 && A_ % 2 == 0 && B_ % 2 == 0;
  static constexpr int A = HALF ? A_ / 2 : A_, B = HALF ? B_ / 2 : B_;
  static constexpr int size(int n) { return n * W + (n / A) * B; }
  static constexpr __device__ __host__ unsigned idx(unsigned p) {
    return p * unsigned(W) + p / unsigned(A) * unsigned(B);
  }
  cx<R>* base;  // already offset by the column index
  __device__ __forceinline__ cx<R>& slot(unsigned i) const { return base[i]; }
};

// First output point of butterfly j (span NS, radix RAD); output r is r NS
// further.  Slot of that output: with NS and NS RAD powers of two the bits
// of r NS are free in the first point, so the slots differ by constants.
constexpr bool pow2(int x) { return (x & (x - 1)) == 0; }
template <class Lds, int RAD, int NS>
struct OutSlots {
  unsigned first, at;
  __device__ __forceinline__ explicit OutSlots(unsigned j)
      : first((j / NS) * (NS * RAD) + j % NS), at(Lds::idx(first)) {}
  __device__ __forceinline__ unsigned operator()(unsigned r) const {
    if constexpr (pow2(NS) && pow2(RAD))
      return at + Lds::idx(r * NS);
    else
      return Lds::idx(first + r * NS);
  }
};

// ------------------------------------------------------------ twiddles
// The twiddles of a radix plan in the order its stages read them: stage of
// span NS > 1 and radix R has a block of (R - 1) NS entries, entry
// (r - 1) NS + k = exp(-2 pi i r k / (NS R)) for the butterflies with j mod
// NS = k.  Blocks follow each other: the block of span NS starts at NS - R0,
// N - R0 entries together (built on the host in FP64 and rounded once).  The
// lanes of a wave read consecutive k, so a twiddle costs one coalesced load
// (hits in L2 and mostly L1) and no index arithmetic; against a quarter table in LDS
// that saves 10 KB of LDS a workgroup and about 6 instructions a twiddle.
// Butterflies of one thread share their twiddles when NS divides T.
template <int N, int T, int NS, int RAD>
constexpr int stage_tw_sets() {
  return (T % NS == 0) ? 1 : N / T / RAD;
}
template <int N, int T, int... Rs>
constexpr int twiddle_count() {
  int ns = 1, c = 0;
  ((c += (ns > 1 ? ((T % ns == 0) ? 1 : N / T / Rs) * (Rs - 1) : 0), ns *= Rs), ...);
  return c;
}

// registers for the twiddles of the stage that follows (1 if there are none
// to request)
template <int N, int T, bool LATE, int NS>
constexpr int next_tw_regs() {
  return 1;
}
template <int N, int T, bool LATE, int NS, int RAD, int... Rest>
constexpr int next_tw_regs() {
  return LATE ? stage_tw_sets<N, T, NS, RAD>() * (RAD - 1) : 1;
}

template <class P>
struct TwCount;
template <int N, int T, int L, int... Rs, int A, int B, int O>
struct TwCount<Plan<N, T, L, Radices<Rs...>, A, B, O>> {
  // late twiddles are loaded stage by stage: nothing held up front
  static constexpr int value = (O & 1) ? 0 : twiddle_count<N, T, Rs...>();
};

template <typename R, int N, int T, int NS, int RAD, int R0>
__device__ __forceinline__ void load_stage_twiddles(cx<R>* w, int t,
                                                    const Buf<cx<R>>& tw) {
  if constexpr (NS > 1) {
#pragma unroll
    for (int b = 0; b < stage_tw_sets<N, T, NS, RAD>(); ++b) {
      // unsigned (t >= 0): masks
      const uint32_t k = uint32_t(t + T * b) % uint32_t(NS);
#pragma unroll
      for (int r = 1; r < RAD; ++r)
        w[b * (RAD - 1) + r - 1] = tw.get(k, uint32_t(NS - R0 + (r - 1) * NS));
    }
  }
}

template <typename R, int N, int T, int NS, int R0, int RA, int... Rest>
__device__ __forceinline__ void load_twiddles_rec(cx<R>* w, int t,
                                                  const Buf<cx<R>>& tw) {
  load_stage_twiddles<R, N, T, NS, RA, R0>(w, t, tw);
  if constexpr (sizeof...(Rest) > 0) {
    constexpr int used = (NS > 1) ? stage_tw_sets<N, T, NS, RA>() * (RA - 1) : 0;
    load_twiddles_rec<R, N, T, NS * RA, R0, Rest...>(w + used, t, tw);
  }
}

template <typename R, int N, int T, int R0, int... Rs>
__device__ __forceinline__ void load_twiddles_impl(cx<R>* w, int t,
                                                   const Buf<cx<R>>& tw,
                                                   Radices<R0, Rs...>) {
  load_twiddles_rec<R, N, T, 1, R0, R0, Rs...>(w, t, tw);
}

template <typename R, class P>
__device__ __forceinline__ void load_twiddles(cx<R>* w, int t, const Buf<cx<R>>& tw) {
  if constexpr (!P::LATE_TW) load_twiddles_impl<R, P::N, P::T>(w, t, tw, typename P::radices{});
}

// Twiddles of late-twiddle plans with three stages, complex64: the middle
// stage's come from a table in LDS, R0 rows of R1 - 1 entries read in pairs
// of 16 bytes (the rows' pitch spreads them over all banks), and the last
// stage's stay in registers from a factor's first transform to its second
// (a half exchange has no room for them and reads them as it goes).  Read
// from the plan's table in every stage, twiddles were 120 of a thread's 168
// loads in a 4096-point pass and kept the compute unit's address unit busier
// than the strided columns did (us, before and now: 4096^2 rows 100, 84.5,
// adjoint 124, 107; columns 157, 134, adjoint 225, 215; 2048^2 columns 36,
// 31).  complex128 tiles leave no LDS for the table (two workgroups of
// 4096^2 rows fill it: 215 us, with the table 345).
template <typename R, class Rad>
struct MidTable {
  static constexpr int PITCH = 0, SIZE = 0;
};
template <typename R, int R0, int R1, int R2>
struct MidTable<R, Radices<R0, R1, R2>> {
  static constexpr int PITCH = R1 + 2;
  static constexpr int SIZE = R0 * PITCH;
  const cx<R>* base;
  static __device__ __forceinline__ void fill(cx<R>* mem, int threads, const Buf<cx<R>>& tw) {
    // entry i: twiddle i / R0 + 1 of row i mod R0
    for (uint32_t i = threadIdx.x; i < uint32_t(R0 * (R1 - 1)); i += uint32_t(threads))
      mem[(i % R0) * PITCH + i / R0] = tw.get(i, 0);
  }
  __device__ __forceinline__ void read(cx<R>* w, int t) const {
    const cx<R>* p = base + (unsigned(t) % unsigned(R0)) * PITCH;
    static_assert(sizeof(R) == 4 && R1 % 2 == 0, "pairs of 16 bytes");
#pragma unroll
    for (int i = 0; i < R1; i += 2) {
      const float4 q = *reinterpret_cast<const float4*>(p + i);
      w[i] = {q.x, q.y};
      if (i + 1 < R1 - 1) w[i + 1] = {q.z, q.w};
    }
  }
};

template <typename R, class P>
constexpr bool mid_tw() {
  return sizeof(R) == 4 && P::MID_TW;
}
template <typename R, class P>
constexpr bool keep_tw() {
  return mid_tw<R, P>() && !P::HX;
}
template <typename R, class P>
constexpr int mid_table_size() {
  return mid_tw<R, P>() ? MidTable<R, typename P::radices>::SIZE : 0;
}

// The last stage's twiddles.
template <typename R, int N, int T, int R0, int R1, int R2>
__device__ __forceinline__ void load_last_impl(cx<R>* w, int t, const Buf<cx<R>>& tw,
                                               Radices<R0, R1, R2>) {
  load_stage_twiddles<R, N, T, R0 * R1, R2, R0>(w, t, tw);
}
template <int N, int T, int R0, int R1, int R2>
constexpr int last_count_impl(Radices<R0, R1, R2>) {
  return stage_tw_sets<N, T, R0 * R1, R2>() * (R2 - 1);
}

// The twiddles of a pass as its transforms see them: all preloaded, the
// middle table and the last stage's, or the plan's table.  keep() before a
// factor's first transform.
template <typename R, class P>
struct Twiddles {
  static constexpr int regs() {
    if constexpr (keep_tw<R, P>())
      return last_count_impl<P::N, P::T>(typename P::radices{});
    else if constexpr (P::LATE_TW || P::HX)
      return 1;
    else
      return TwCount<P>::value > 0 ? TwCount<P>::value : 1;
  }
  Buf<cx<R>> tw;
  cx<R>* mid;  // the LDS table, after the tile
  cx<R> w[regs()];
  __device__ __forceinline__ Twiddles(const cx<R>* table, cx<R>* lds_table, int t)
      : tw(table), mid(lds_table) {
    if constexpr (mid_tw<R, P>())
      MidTable<R, typename P::radices>::fill(mid, P::THREADS, tw);
    else if constexpr (!P::LATE_TW && !P::HX)
      load_twiddles<R, P>(w, t, tw);
  }
  __device__ __forceinline__ void keep(int t) {
    if constexpr (keep_tw<R, P>()) {
      asm volatile("" : "+v"(t));  // loaded here, not held from the first factor
      load_last_impl<R, P::N, P::T>(w, t, tw, typename P::radices{});
    }
  }
};

// ------------------------------------------------------------- stages
// w: the twiddles of the stage at hand, from registers (preloaded) or, with
// LATE, requested one stage ahead, so that their latency passes behind a
// whole butterfly and exchange (requested where they are used, the waits for
// them were a fifth of a 4096-point pass); of a plan that keeps them, the
// last stage's, the middle stage reading its own from mid.  tail() is called
// where the last stage would request the next one's: it requests what
// follows the transform.
template <typename R, int N, int T, int DIR, int NS, int R0, bool LATE, class Mid, class Lds,
          class Tail, int RAD, int... Rest>
__device__ __forceinline__ void fft_stages(cx<R>* v, int t, const Lds& lds, const cx<R>* w,
                                           const Buf<cx<R>>& tw, const Mid& mid, Tail&& tail) {
  // with late twiddles the thread index is made opaque per stage, so the
  // stage's LDS and twiddle addresses are computed where they are used
  // instead of held in registers from the kernel's start
  if constexpr (LATE) asm volatile("" : "+v"(t));
  constexpr bool FIRST = NS == 1, LAST = sizeof...(Rest) == 0;
  constexpr int E = N / T;
  constexpr int NB = E / RAD;
  constexpr int STRIDE = N / RAD;
  constexpr int SETS = stage_tw_sets<N, T, NS, RAD>();
  static_assert(E % RAD == 0, "radix must divide points per thread");
  static_assert(pow2(T), "the input slots of a thread differ by constants");
  constexpr bool KEEP = !std::is_same_v<Mid, int>;
  constexpr bool MIDDLE = KEEP && !FIRST && !LAST;
  cx<R> wn[KEEP ? 1 : next_tw_regs<N, T, LATE, NS * RAD, Rest...>()];
  if constexpr (LATE) {
    if constexpr (LAST)
      tail();
    else if constexpr (!KEEP)
      load_stage_twiddles<R, N, T, NS * RAD, first_radix<Rest...>(), R0>(wn, t, tw);
  }
  cx<R> a[NB][RAD];
  cx<R> wm[MIDDLE ? RAD : 1];
  if constexpr (MIDDLE) mid.read(wm, t);
  const unsigned in0 = Lds::idx(unsigned(t));
#pragma unroll
  for (int b = 0; b < NB; ++b) {
#pragma unroll
    for (int r = 0; r < RAD; ++r) {
      if constexpr (FIRST) {
        a[b][r] = v[b + r * NB];
      } else {
        a[b][r] = lds.slot(in0 + Lds::idx(T * b + r * STRIDE));
      }
    }
  }
  if constexpr (!FIRST) {
    __syncthreads();
  }
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    dft<RAD, DIR, (NS > 1)>(a[b], MIDDLE ? wm : w + (SETS == 1 ? 0 : b * (RAD - 1)));
    if constexpr (!LAST) {
      const OutSlots<Lds, RAD, NS> out(unsigned(t + T * b));  // >= 0: shifts and masks
#pragma unroll
      for (int r = 0; r < RAD; ++r) lds.slot(out(r)) = a[b][r];
    } else {
#pragma unroll
      for (int r = 0; r < RAD; ++r) v[b + r * NB] = a[b][r];
    }
  }
  if constexpr (!LAST) {
    __syncthreads();
    constexpr int used = NS > 1 ? SETS * (RAD - 1) : 0;
    fft_stages<R, N, T, DIR, NS * RAD, R0, LATE, Mid, Lds, Tail, Rest...>(
        v, t, lds, KEEP ? w : LATE ? wn : w + used, tw, mid, static_cast<Tail&&>(tail));
  }
}

// ------------------------------------ exchanges through half an LDS tile
// A tile that would fill the LDS can exchange through half of it, so that
// two workgroups fit one compute unit.  In a stage of radix R and span NS
// (not the last), butterfly j writes its outputs below N/2 exactly when
// j < N/(2R) (given N/(NS R) even), i.e. for b < NB/2 of every thread; the
// next stage (radix R') reads point t + T b' + r' N/R', below N/2 exactly
// when r' < R'/2.  So each exchange runs in two rounds over the same N/2
// slots: the lower outputs are written and the lower inputs read, then the
// upper ones, with a barrier between every write and read (four per
// exchange, the first guarding the previous exchange's last reads).  The
// butterflies, their twiddles (always loaded late) and their order are those
// of the full exchange.
template <typename R, int N, int T, int RAD, int NS, int RB, class Lds>
__device__ __forceinline__ void hx_exchange(cx<R> (&a)[N / T / RAD][RAD],
                                            cx<R> (&nx)[N / T / RB][RB], int t, const Lds& lds) {
  constexpr int NB = N / T / RAD, NB2 = N / T / RB, H = N / 2;
  static_assert(NB % 2 == 0 && RB % 2 == 0 && (N / (NS * RAD)) % 2 == 0,
                "half exchange: even butterfly count, next radix and remaining span");
  asm volatile("" : "+v"(t));
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    __syncthreads();
#pragma unroll
    for (int b = h * NB / 2; b < (h + 1) * NB / 2; ++b) {
      // butterfly t + T (b - h NB / 2) of the half's own N/2 points
      const OutSlots<Lds, RAD, NS> out(unsigned(t + T * (b - h * NB / 2)));
#pragma unroll
      for (int r = 0; r < RAD; ++r) lds.slot(out(r)) = a[b][r];
    }
    __syncthreads();
    const unsigned in0 = Lds::idx(unsigned(t));
#pragma unroll
    for (int b = 0; b < NB2; ++b) {
#pragma unroll
      for (int r = h * RB / 2; r < (h + 1) * RB / 2; ++r)
        nx[b][r] = lds.slot(in0 + Lds::idx(T * b + r * (N / RB) - h * H));
    }
  }
}

template <typename R, int N, int T, int DIR, int NS, int R0, class Mid, class Lds, class Tail,
          int RA, int... Rest>
__device__ __forceinline__ void hx_stages(cx<R>* v, cx<R> (&a)[N / T / RA][RA], int t,
                                          const Lds& lds, const Buf<cx<R>>& tw, const Mid& mid,
                                          Tail&& tail) {
  constexpr bool LAST = sizeof...(Rest) == 0;
  constexpr int NB = N / T / RA;
  constexpr int SETS = stage_tw_sets<N, T, NS, RA>();
  // the thread index made opaque per stage (addresses computed in the stage)
  asm volatile("" : "+v"(t));
  // one butterfly at a time, each with its own twiddles: all of a thread's
  // points are live here, and twiddles of two butterflies beside them would
  // not fit the registers of two workgroups per compute unit
  constexpr bool MIDDLE = !std::is_same_v<Mid, int> && NS > 1 && !LAST;
  cx<R> w[NS > 1 ? RA : 1];
  if constexpr (MIDDLE) {
    static_assert(SETS == 1);
    mid.read(w, t);
  }
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    if constexpr (NS > 1 && !MIDDLE) {
      if (b < SETS) {
        const uint32_t k = uint32_t(t + T * b) % uint32_t(NS);
#pragma unroll
        for (int r = 1; r < RA; ++r) w[r - 1] = tw.get(k, uint32_t(NS - R0 + (r - 1) * NS));
      }
    }
    dft<RA, DIR, (NS > 1)>(a[b], w);
#pragma unroll
    for (int r = 0; r < RA; ++r) asm volatile("" : "+v"(a[b][r].re), "+v"(a[b][r].im));
    __builtin_amdgcn_sched_barrier(0);
  }
  if constexpr (LAST) tail();
  if constexpr (LAST) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < RA; ++r) v[b + r * NB] = a[b][r];
  } else {
    constexpr int RB = first_radix<Rest...>();
    cx<R> nx[N / T / RB][RB];
    hx_exchange<R, N, T, RA, NS, RB>(a, nx, t, lds);
    hx_stages<R, N, T, DIR, NS * RA, R0, Mid, Lds, Tail, Rest...>(v, nx, t, lds, tw, mid,
                                                                  static_cast<Tail&&>(tail));
  }
}

template <typename R, class P, int DIR, class Lds, class Tail, int R0, int... Rest>
__device__ __forceinline__ void fft_line_impl(cx<R>* v, int t, const Lds& lds,
                                              const Twiddles<R, P>& tws, Tail&& tail,
                                              Radices<R0, Rest...>) {
  if constexpr (P::HX) {
    constexpr int NB = P::E / R0;
    cx<R> a[NB][R0];
#pragma unroll
    for (int b = 0; b < NB; ++b) {
#pragma unroll
      for (int r = 0; r < R0; ++r) a[b][r] = v[b + r * NB];
    }
    if constexpr (mid_tw<R, P>()) {
      using Mid = MidTable<R, typename P::radices>;
      hx_stages<R, P::N, P::T, DIR, 1, R0, Mid, Lds, Tail, R0, Rest...>(
          v, a, t, lds, tws.tw, Mid{tws.mid}, static_cast<Tail&&>(tail));
    } else {
      hx_stages<R, P::N, P::T, DIR, 1, R0, int, Lds, Tail, R0, Rest...>(
          v, a, t, lds, tws.tw, 0, static_cast<Tail&&>(tail));
    }
  } else if constexpr (keep_tw<R, P>()) {
    using Mid = MidTable<R, typename P::radices>;
    fft_stages<R, P::N, P::T, DIR, 1, R0, true, Mid, Lds, Tail, R0, Rest...>(
        v, t, lds, tws.w, tws.tw, Mid{tws.mid}, static_cast<Tail&&>(tail));
  } else {
    fft_stages<R, P::N, P::T, DIR, 1, R0, P::LATE_TW, int, Lds, Tail, R0, Rest...>(
        v, t, lds, tws.w, tws.tw, 0, static_cast<Tail&&>(tail));
  }
}

// In-register FFT of one line (DIR = -1 forward, +1 inverse, unscaled),
// with the thread's twiddles in tws; tail() is called with the last stage (a
// plan whose twiddles come late).  On entry and
// exit v[e] holds point t + T*e.  A full exchange leaves the LDS free (its
// last barrier follows the last reads); a half exchange opens with the
// barrier that guards the last reads.
template <typename R, class P, int DIR, class Lds, class Tail>
__device__ __forceinline__ void fft_line(cx<R>* v, int t, const Lds& lds,
                                         const Twiddles<R, P>& tws, Tail&& tail) {
  fft_line_impl<R, P, DIR>(v, t, lds, tws, static_cast<Tail&&>(tail), typename P::radices{});
}
template <typename R, class P, int DIR, class Lds>
__device__ __forceinline__ void fft_line(cx<R>* v, int t, const Lds& lds,
                                         const Twiddles<R, P>& tws) {
  fft_line<R, P, DIR>(v, t, lds, tws, [] {});
}

// Host side: the radix list of a plan.
template <int... Rs>
inline void radix_list(Radices<Rs...>, int* out) {
  int i = 0;
  ((out[i++] = Rs), ...);
  out[i] = 0;
}

}  // namespace ssfm
