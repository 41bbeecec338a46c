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
// loads them stage by stage.
#pragma once

#include <hip/hip_runtime.h>

#include <utility>

namespace ssfm {

template <typename R>
struct cx {
  R re, im;
};

template <typename R>
__device__ __forceinline__ cx<R> operator+(cx<R> a, cx<R> b) {
  return {a.re + b.re, a.im + b.im};
}
template <typename R>
__device__ __forceinline__ cx<R> operator-(cx<R> a, cx<R> b) {
  return {a.re - b.re, a.im - b.im};
}
template <typename R>
__device__ __forceinline__ cx<R> cmul(cx<R> a, cx<R> b) {
  return {a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re};
}
// a * conj(b)
template <typename R>
__device__ __forceinline__ cx<R> cmulc(cx<R> a, cx<R> b) {
  return {a.re * b.re + a.im * b.im, a.im * b.re - a.re * b.im};
}
template <typename R>
__device__ __forceinline__ cx<R> conjg(cx<R> a) {
  return {a.re, -a.im};
}
template <typename R>
__device__ __forceinline__ cx<R> scale(cx<R> a, R s) {
  return {a.re * s, a.im * s};
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
// multiply by exp(dir i pi/4) = (1 + dir i)/sqrt(2)
template <int DIR, typename R>
__device__ __forceinline__ cx<R> rot_8(cx<R> a) {
  const R h = R(0.70710678118654752440);
  if constexpr (DIR < 0) {
    return {(a.re + a.im) * h, (a.im - a.re) * h};
  } else {
    return {(a.re - a.im) * h, (a.im + a.re) * h};
  }
}
// multiply by exp(dir 3 i pi/4) = (-1 + dir i)/sqrt(2)
template <int DIR, typename R>
__device__ __forceinline__ cx<R> rot_38(cx<R> a) {
  const R h = R(0.70710678118654752440);
  if constexpr (DIR < 0) {
    return {(a.im - a.re) * h, -(a.re + a.im) * h};
  } else {
    return {-(a.re + a.im) * h, (a.re - a.im) * h};
  }
}
// multiply by exp(dir 2 pi i e / 16) for e = 1, 3, 9
template <int DIR, int EXP, typename R>
__device__ __forceinline__ cx<R> rot_16(cx<R> a) {
  constexpr double c1 = 0.92387953251128675613;  // cos(pi/8)
  constexpr double s1 = 0.38268343236508977173;  // sin(pi/8)
  double cr, ci;
  if constexpr (EXP == 1) {
    cr = c1;
    ci = DIR * s1;
  } else if constexpr (EXP == 3) {
    cr = s1;
    ci = DIR * c1;
  } else {  // EXP == 9
    cr = -c1;
    ci = -DIR * s1;
  }
  return cmul(a, cx<R>{R(cr), R(ci)});
}

// ---------------------------------------------------------------- DFTs
// In-place DFT of R points in natural order: y_k = sum_n x_n w^(nk),
// w = exp(dir 2 pi i / R).

template <int DIR, typename R>
__device__ __forceinline__ void dft2(cx<R>* v) {
  cx<R> a = v[0];
  v[0] = a + v[1];
  v[1] = a - v[1];
}

template <int DIR, typename R>
__device__ __forceinline__ void dft3(cx<R>* v) {
  const R h = R(0.86602540378443864676);  // sqrt(3)/2
  cx<R> t = v[1] + v[2];
  cx<R> u = v[1] - v[2];
  cx<R> m = {v[0].re - R(0.5) * t.re, v[0].im - R(0.5) * t.im};
  cx<R> w = scale(rot_q<DIR>(u), h);
  v[0] = v[0] + t;
  v[1] = m + w;
  v[2] = m - w;
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

template <int DIR, typename R>
__device__ __forceinline__ void dft4(cx<R>* v) {
  dft4_<DIR>(v[0], v[1], v[2], v[3]);
}

template <int DIR, typename R>
__device__ __forceinline__ void dft8(cx<R>* v) {
  cx<R> b0 = v[0] + v[4], c0 = v[0] - v[4];
  cx<R> b1 = v[1] + v[5], c1 = v[1] - v[5];
  cx<R> b2 = v[2] + v[6], c2 = v[2] - v[6];
  cx<R> b3 = v[3] + v[7], c3 = v[3] - v[7];
  c1 = rot_8<DIR>(c1);
  c2 = rot_q<DIR>(c2);
  c3 = rot_38<DIR>(c3);
  dft4_<DIR>(b0, b1, b2, b3);  // even outputs
  dft4_<DIR>(c0, c1, c2, c3);  // odd outputs
  v[0] = b0; v[2] = b1; v[4] = b2; v[6] = b3;
  v[1] = c0; v[3] = c1; v[5] = c2; v[7] = c3;
}

// 16 = 4 x 4: inner DFT4 over n2 (stride 4), twiddle w16^(n1 k2), outer
// DFT4 over n1; output index k2 + 4 k1.
template <int DIR, typename R>
__device__ __forceinline__ void dft16(cx<R>* v) {
  dft4_<DIR>(v[0], v[4], v[8], v[12]);
  dft4_<DIR>(v[1], v[5], v[9], v[13]);
  dft4_<DIR>(v[2], v[6], v[10], v[14]);
  dft4_<DIR>(v[3], v[7], v[11], v[15]);
  // v[n1 + 4 k2] *= w16^(n1 k2)
  v[5] = rot_16<DIR, 1>(v[5]);
  v[9] = rot_8<DIR>(v[9]);
  v[13] = rot_16<DIR, 3>(v[13]);
  v[6] = rot_8<DIR>(v[6]);
  v[10] = rot_q<DIR>(v[10]);
  v[14] = rot_38<DIR>(v[14]);
  v[7] = rot_16<DIR, 3>(v[7]);
  v[11] = rot_38<DIR>(v[11]);
  v[15] = rot_16<DIR, 9>(v[15]);
  dft4_<DIR>(v[0], v[1], v[2], v[3]);
  dft4_<DIR>(v[4], v[5], v[6], v[7]);
  dft4_<DIR>(v[8], v[9], v[10], v[11]);
  dft4_<DIR>(v[12], v[13], v[14], v[15]);
  // now v[4 k2 + k1] holds y[k2 + 4 k1]: transpose the 4x4 index
  cx<R> t;
#define SSFM_SWAP(a, b) t = v[a]; v[a] = v[b]; v[b] = t;
  SSFM_SWAP(1, 4) SSFM_SWAP(2, 8) SSFM_SWAP(3, 12)
  SSFM_SWAP(6, 9) SSFM_SWAP(7, 13) SSFM_SWAP(11, 14)
#undef SSFM_SWAP
}

// 12 = 4 x 3: inner DFT4 over n2 (points n1 + 3 n2), twiddle w12^(n1 k2),
// outer DFT3 over n1; output index k2 + 4 k1.
template <int DIR, typename R>
__device__ __forceinline__ void dft12(cx<R>* v) {
  constexpr double h = 0.86602540378443864676;  // cos(pi/6)
  cx<R> t[3][4];
#pragma unroll
  for (int n1 = 0; n1 < 3; ++n1) {
#pragma unroll
    for (int n2 = 0; n2 < 4; ++n2) t[n1][n2] = v[n1 + 3 * n2];
    dft4_<DIR>(t[n1][0], t[n1][1], t[n1][2], t[n1][3]);
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

// cos(e pi / 16) and sin(e pi / 16) for integer e (exact table of the
// first octant, extended by symmetry).
constexpr double kCos16[9] = {1.0,
                              0.98078528040323044913,
                              0.92387953251128675613,
                              0.83146961230254523708,
                              0.70710678118654752440,
                              0.55557023301960222474,
                              0.38268343236508977173,
                              0.19509032201612826785,
                              0.0};
constexpr double cos16(int e) {
  e = ((e % 32) + 32) % 32;
  if (e <= 8) return kCos16[e];
  if (e <= 16) return -kCos16[16 - e];
  if (e <= 24) return -kCos16[e - 16];
  return kCos16[32 - e];
}
constexpr double sin16(int e) { return cos16(8 - e); }

// multiply by exp(dir 2 pi i e / 32)
template <int DIR, int EXP, typename R>
__device__ __forceinline__ cx<R> rot_32(cx<R> a) {
  constexpr int e = ((EXP % 32) + 32) % 32;
  if constexpr (e == 0) return a;
  else if constexpr (e == 8) return rot_q<DIR>(a);
  else if constexpr (e == 16) return cx<R>{-a.re, -a.im};
  else if constexpr (e == 24) return rot_q<-DIR>(a);
  else if constexpr (e == 4) return rot_8<DIR>(a);
  else if constexpr (e == 12) return rot_38<DIR>(a);
  else return cmul(a, cx<R>{R(cos16(e)), R(DIR * sin16(e))});
}

// 32 = 4 x 8: inner DFT8 over n2 (points n1 + 4 n2), twiddle w32^(n1 k2),
// outer DFT4 over n1; output index k2 + 8 k1.
template <int DIR, int N1, int K2, typename R>
__device__ __forceinline__ void dft32_tw(cx<R>* v) {
  v[N1 + 4 * K2] = rot_32<DIR, N1 * K2>(v[N1 + 4 * K2]);
}

template <int DIR, typename R>
__device__ __forceinline__ void dft32(cx<R>* v) {
  cx<R> t[32];
#pragma unroll
  for (int n1 = 0; n1 < 4; ++n1) {
    cx<R> g[8];
#pragma unroll
    for (int n2 = 0; n2 < 8; ++n2) g[n2] = v[n1 + 4 * n2];
    dft8<DIR>(g);
#pragma unroll
    for (int k2 = 0; k2 < 8; ++k2) t[n1 + 4 * k2] = g[k2];
  }
  [&]<int... I>(std::integer_sequence<int, I...>) {
    ((dft32_tw<DIR, I / 8, I % 8>(t)), ...);
  }(std::make_integer_sequence<int, 32>{});
#pragma unroll
  for (int k2 = 0; k2 < 8; ++k2) {
    dft4_<DIR>(t[4 * k2], t[4 * k2 + 1], t[4 * k2 + 2], t[4 * k2 + 3]);
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1) v[k2 + 8 * k1] = t[4 * k2 + k1];
  }
}

template <int RAD, int DIR, typename R>
__device__ __forceinline__ void dft(cx<R>* v) {
  if constexpr (RAD == 2) dft2<DIR>(v);
  else if constexpr (RAD == 3) dft3<DIR>(v);
  else if constexpr (RAD == 4) dft4<DIR>(v);
  else if constexpr (RAD == 8) dft8<DIR>(v);
  else if constexpr (RAD == 12) dft12<DIR>(v);
  else if constexpr (RAD == 16) dft16<DIR>(v);
  else if constexpr (RAD == 32) dft32<DIR>(v);
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
// registers) instead of all of them before the first; bits 8-11 give the
// wavefronts per SIMD the compiler must leave room for in the complex64
// kernels (0: no target), bits 12-14 the same for the complex128 ones; bit
// 15 makes a column pass exchange through half its tile (fft_line_hx),
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
template <typename R, int N>
struct LdsLineMajor {
  static constexpr unsigned A = sizeof(R) == 4 ? 32 : 16;
  static constexpr int LINE = N + N / int(A) * 3;
  cx<R>* base;
  // unsigned (p >= 0): constant offsets of p that are multiples of A fold
  // into the instruction's offset
  __device__ __forceinline__ cx<R>& at(int p) const {
    return base[unsigned(p) + (unsigned(p) / A) * 3u];
  }
  __device__ __forceinline__ cx<R> get(int p) const { return at(p); }
  __device__ __forceinline__ void put(int p, cx<R> v) const { at(p) = v; }
};

// Column tiles: point-major, the W columns of a point adjacent, B padding
// slots after every A points (complex64; half of both for complex128, whose
// elements span twice the banks).
template <typename R, int W, int A_, int B_>
struct LdsPointMajor {
  static constexpr bool HALF = sizeof(R) == 8 && A_ % 2 == 0 && B_ % 2 == 0;
  static constexpr int A = HALF ? A_ / 2 : A_, B = HALF ? B_ / 2 : B_;
  static constexpr int size(int n) { return n * W + (n / A) * B; }
  cx<R>* base;  // already offset by the column index
  // unsigned (p >= 0): the division is a shift, and constant offsets of p
  // that are multiples of A fold into the instruction's offset
  __device__ __forceinline__ int idx(int p) const {
    const unsigned u = unsigned(p);
    return int(u * W + (u / A) * B);
  }
  __device__ __forceinline__ cx<R> get(int p) const { return base[idx(p)]; }
  __device__ __forceinline__ void put(int p, cx<R> v) const { base[idx(p)] = v; }
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

template <class P>
struct TwCount;
template <int N, int T, int L, int... Rs, int A, int B, int O>
struct TwCount<Plan<N, T, L, Radices<Rs...>, A, B, O>> {
  // late twiddles are loaded stage by stage: nothing held up front
  static constexpr int value = (O & 1) ? 0 : twiddle_count<N, T, Rs...>();
};

template <typename R, int N, int T, int NS, int RAD, int R0>
__device__ __forceinline__ void load_stage_twiddles(cx<R>* w, int t,
                                                    const cx<R>* __restrict__ tw) {
  if constexpr (NS > 1) {
#pragma unroll
    for (int b = 0; b < stage_tw_sets<N, T, NS, RAD>(); ++b) {
      // unsigned (t >= 0): masks; 32-bit offsets from a uniform base
      const uint32_t k = uint32_t(t + T * b) % uint32_t(NS);
#pragma unroll
      for (int r = 1; r < RAD; ++r)
        w[b * (RAD - 1) + r - 1] = tw[k + uint32_t(NS - R0 + (r - 1) * NS)];
    }
  }
}

template <typename R, int N, int T, int NS, int R0, int RA, int... Rest>
__device__ __forceinline__ void load_twiddles_rec(cx<R>* w, int t,
                                                  const cx<R>* __restrict__ tw) {
  load_stage_twiddles<R, N, T, NS, RA, R0>(w, t, tw);
  if constexpr (sizeof...(Rest) > 0) {
    constexpr int used = (NS > 1) ? stage_tw_sets<N, T, NS, RA>() * (RA - 1) : 0;
    load_twiddles_rec<R, N, T, NS * RA, R0, Rest...>(w + used, t, tw);
  }
}

template <typename R, int N, int T, int R0, int... Rs>
__device__ __forceinline__ void load_twiddles_impl(cx<R>* w, int t,
                                                   const cx<R>* __restrict__ tw,
                                                   Radices<R0, Rs...>) {
  load_twiddles_rec<R, N, T, 1, R0, R0, Rs...>(w, t, tw);
}

template <typename R, class P>
__device__ __forceinline__ void load_twiddles(cx<R>* w, int t, const cx<R>* __restrict__ tw) {
  if constexpr (!P::LATE_TW) load_twiddles_impl<R, P::N, P::T>(w, t, tw, typename P::radices{});
}

// ---------------------------------------------------------- one stage
// w: this stage's twiddles in registers (preloaded), or, with LATE, loaded
// here from the table before the stage's LDS reads so that their latency
// overlaps the exchange.
template <typename R, int N, int T, int RAD, int NS, int R0, int DIR, bool FIRST,
          bool LAST, bool LATE, class Lds>
__device__ __forceinline__ void fft_stage(cx<R>* v, int t, const Lds& lds,
                                          const cx<R>* wpre, const cx<R>* __restrict__ tw) {
  // with late twiddles the thread index is made opaque per stage, so the
  // stage's LDS and twiddle addresses are computed where they are used
  // instead of held in registers from the kernel's start
  if constexpr (LATE) asm volatile("" : "+v"(t));
  constexpr int E = N / T;
  constexpr int NB = E / RAD;
  constexpr int STRIDE = N / RAD;
  constexpr int SETS = stage_tw_sets<N, T, NS, RAD>();
  static_assert(E % RAD == 0, "radix must divide points per thread");
  cx<R> wl[(LATE && NS > 1) ? SETS * (RAD - 1) : 1];
  if constexpr (LATE && NS > 1) load_stage_twiddles<R, N, T, NS, RAD, R0>(wl, t, tw);
  const cx<R>* w = LATE ? wl : wpre;
  cx<R> a[NB][RAD];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
#pragma unroll
    for (int r = 0; r < RAD; ++r) {
      if constexpr (FIRST) {
        a[b][r] = v[b + r * NB];
      } else {
        a[b][r] = lds.get(t + T * b + r * STRIDE);
      }
    }
  }
  if constexpr (!FIRST) {
    __syncthreads();
  }
#pragma unroll
  for (int b = 0; b < NB; ++b) {
    const unsigned j = unsigned(t + T * b);  // j >= 0: shifts and masks
    if constexpr (NS > 1) {
#pragma unroll
      for (int r = 1; r < RAD; ++r) {
        const cx<R> ww = w[(SETS == 1 ? 0 : b * (RAD - 1)) + r - 1];
        a[b][r] = (DIR > 0) ? cmulc(a[b][r], ww) : cmul(a[b][r], ww);
      }
    }
    dft<RAD, DIR>(a[b]);
    if constexpr (!LAST) {
      const int base = int((j / NS) * NS * RAD + j % NS);
#pragma unroll
      for (int r = 0; r < RAD; ++r) lds.put(base + r * NS, a[b][r]);
    } else {
#pragma unroll
      for (int r = 0; r < RAD; ++r) v[b + r * NB] = a[b][r];
    }
  }
  if constexpr (!LAST) {
    __syncthreads();
  }
}

template <typename R, int N, int T, int DIR, int NS, int R0, bool FIRST, bool LATE,
          class Lds, int RA, int... Rest>
__device__ __forceinline__ void fft_stages(cx<R>* v, int t, const Lds& lds,
                                           const cx<R>* w, const cx<R>* __restrict__ tw) {
  constexpr bool LAST = sizeof...(Rest) == 0;
  fft_stage<R, N, T, RA, NS, R0, DIR, FIRST, LAST, LATE>(v, t, lds, w, tw);
  if constexpr (!LAST) {
    constexpr int used = (!LATE && NS > 1) ? stage_tw_sets<N, T, NS, RA>() * (RA - 1) : 0;
    fft_stages<R, N, T, DIR, NS * RA, R0, false, LATE, Lds, Rest...>(v, t, lds, w + used, tw);
  }
}

template <typename R, int N, int T, int DIR, bool LATE, class Lds, int R0, int... Rs>
__device__ __forceinline__ void fft_line_impl(cx<R>* v, int t, const Lds& lds,
                                              const cx<R>* w, const cx<R>* __restrict__ tw,
                                              Radices<R0, Rs...>) {
  fft_stages<R, N, T, DIR, 1, R0, true, LATE, Lds, R0, Rs...>(v, t, lds, w, tw);
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
      const unsigned j = unsigned(t + T * b);
      const int base = int((j / NS) * NS * RAD + j % NS) - h * H;
#pragma unroll
      for (int r = 0; r < RAD; ++r) lds.put(base + r * NS, a[b][r]);
    }
    __syncthreads();
#pragma unroll
    for (int b = 0; b < NB2; ++b) {
#pragma unroll
      for (int r = h * RB / 2; r < (h + 1) * RB / 2; ++r)
        nx[b][r] = lds.get(t + T * b + r * (N / RB) - h * H);
    }
  }
}

template <typename R, int N, int T, int DIR, int NS, int R0, class Lds, int RA, int... Rest>
__device__ __forceinline__ void hx_stages(cx<R>* v, cx<R> (&a)[N / T / RA][RA], int t,
                                          const Lds& lds, const cx<R>* __restrict__ tw) {
  constexpr int NB = N / T / RA;
  constexpr int SETS = stage_tw_sets<N, T, NS, RA>();
  // the thread index made opaque per stage (addresses computed in the stage)
  asm volatile("" : "+v"(t));
  if constexpr (NS > 1) {
    cx<R> w[SETS * (RA - 1)];
    load_stage_twiddles<R, N, T, NS, RA, R0>(w, t, tw);
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 1; r < RA; ++r) {
        const cx<R> ww = w[(SETS == 1 ? 0 : b * (RA - 1)) + r - 1];
        a[b][r] = (DIR > 0) ? cmulc(a[b][r], ww) : cmul(a[b][r], ww);
      }
  }
#pragma unroll
  for (int b = 0; b < NB; ++b) dft<RA, DIR>(a[b]);
  if constexpr (sizeof...(Rest) == 0) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < RA; ++r) v[b + r * NB] = a[b][r];
  } else {
    constexpr int RB = first_radix<Rest...>();
    cx<R> nx[N / T / RB][RB];
    hx_exchange<R, N, T, RA, NS, RB>(a, nx, t, lds);
    hx_stages<R, N, T, DIR, NS * RA, R0, Lds, Rest...>(v, nx, t, lds, tw);
  }
}

template <typename R, int N, int T, int DIR, class Lds, int R0, int... Rest>
__device__ __forceinline__ void fft_line_hx_impl(cx<R>* v, int t, const Lds& lds,
                                                 const cx<R>* __restrict__ tw,
                                                 Radices<R0, Rest...>) {
  constexpr int NB = N / T / R0;
  cx<R> a[NB][R0];
#pragma unroll
  for (int b = 0; b < NB; ++b) {
#pragma unroll
    for (int r = 0; r < R0; ++r) a[b][r] = v[b + r * NB];
  }
  hx_stages<R, N, T, DIR, 1, R0, Lds, R0, Rest...>(v, a, t, lds, tw);
}

// In-register FFT of one line (DIR = -1 forward, +1 inverse, unscaled),
// with the thread's twiddles preloaded by load_twiddles<R, P> (w), or, for
// a late-twiddle or half-exchange plan, read stage by stage from the plan's
// stage-ordered table tw.  On entry and exit v[e] holds point t + T*e.  A
// full exchange leaves the LDS free (its last barrier follows the last
// reads); a half exchange opens with the barrier that guards the last reads.
template <typename R, class P, int DIR, class Lds>
__device__ __forceinline__ void fft_line(cx<R>* v, int t, const Lds& lds, const cx<R>* w,
                                         const cx<R>* __restrict__ tw) {
  if constexpr (P::HX)
    fft_line_hx_impl<R, P::N, P::T, DIR>(v, t, lds, tw, typename P::radices{});
  else
    fft_line_impl<R, P::N, P::T, DIR, P::LATE_TW>(v, t, lds, w, tw, typename P::radices{});
}

// Host side: the radix list of a plan.
template <int... Rs>
inline void radix_list(Radices<Rs...>, int* out) {
  int i = 0;
  ((out[i++] = Rs), ...);
  out[i] = 0;
}

}  // namespace ssfm
