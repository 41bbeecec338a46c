// pass_kernels.hpp -- the row and column pass kernels of the march.
//
// One z step of the march (Math and Equations, Eq. (1)-(3), (9)) is
//   V = F_y^-1 P_y F_y  F_x^-1 P_x F_x  S(U-)      (S: the previous screen)
// where P_x P_y = exp(-i (kx^2 + ky^2) dz / 2k0) is the separable
// diffraction factor and the 1/N of each inverse DFT is folded into P.  The
// two factors commute, so the order may alternate: even steps diffract
// along x first, odd ones along y.  Then the second factor of one step, its
// screen and the first factor of the next step all act along the same axis,
// and one pass over the field does the three:
//   ROW_FWD, COL_FWD   u -> V = F^-1 P F u (kept for the adjoint, its power
//                      summed) -> S(V) -> F^-1 P F S(V)
// A march of n steps is n + 1 passes instead of 2 n, each reading and
// writing every point once: half the launches and half the traffic of two
// passes a step.  The first pass of a march has no factor to end a step
// with, the last one neither screen nor next factor (PASS_* flags; one body
// serves all, so a march cut anywhere gives the same bits).  Between
// marches the field is the pre-screen field V_n, its screen pending; within
// one it is the half-diffracted field, and V exists in registers only,
// stored from there when the adjoint needs it.
//
// Each workgroup owns whole lines: a row workgroup reads and writes LINES
// contiguous rows; a column workgroup reads W = LINES adjacent columns row
// by row.  FFT -> multiply -> inverse FFT run in registers with LDS
// exchanges between radix stages only.
#pragma once

#include <algorithm>
#include <type_traits>

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include "fft_core.hpp"
#include "kernels.hpp"
#include "noise.hpp"
#include "plans.hpp"
#include "screen.hpp"

namespace ssfm {

template <typename R>
__device__ __forceinline__ ScreenConst<R> screen_const(const InstDev& in) {
  ScreenConst<R> s;
  if constexpr (sizeof(R) == 4) {
    s.cK = in.cK_f;
    s.cM = in.cM_f;
    s.inv2k1 = in.inv2k1_f;
    s.x_weak = in.x_weak_f;
#pragma unroll
    for (int p = 0; p < 8; ++p) s.th[p] = in.theta_f[p];
  } else {
    s.cK = in.cK;
    s.cM = in.cM;
    s.inv2k1 = in.inv2k1;
    s.x_weak = in.x_weak;
#pragma unroll
    for (int p = 0; p < 8; ++p) s.th[p] = in.theta[p];
  }
  s.K = in.K;
  s.terms = in.terms;
  return s;
}

// Uniform reads of the beam table, the screen step lists and the spectra
// through the constant address space: scalar loads, counted apart from the
// vector loads, so waiting for them never waits for the field loads in
// flight.  No kernel that may run at the same time writes these tables: the
// launches that do (k_put, k_load_field) are on the context's stream, and
// the chains of the size groups fork from it after them and join it again.
template <typename T>
using const_as4 = const __attribute__((address_space(4))) T;
template <typename T>
__device__ __forceinline__ T load_uniform(const T* p) {
  static_assert(sizeof(T) % 4 == 0, "whole dwords");
  T out;
  const_as4<uint32_t>* src =
      reinterpret_cast<const_as4<uint32_t>*>(reinterpret_cast<uintptr_t>(p));
  uint32_t* dst = reinterpret_cast<uint32_t*>(&out);
#pragma unroll
  for (int i = 0; i < int(sizeof(T) / 4); ++i) dst[i] = src[i];
  return out;
}

// Turbulence plane applied after context step `step` (nullptr if none): the
// screen whose step equals the beam's own step index (the context step
// minus the step at which the beam's field was set), by lower-bound search
// of the beam's increasing step list (a workgroup-uniform chain of
// log2(n_screens) scalar loads).
template <typename R>
__device__ __forceinline__ const R* find_plane(const R* screens, const int64_t* steps,
                                               const InstDev& in, int64_t step) {
  if (step < 0 || !(in.terms & T_TURB) || in.n_screens <= 0 || screens == nullptr)
    return nullptr;
  step -= in.step_base;
  const int64_t* st = steps + in.steps_off;
  int lo = 0, hi = in.n_screens - 1;
  if (step < load_uniform(st + lo) || step > load_uniform(st + hi)) return nullptr;
  while (lo < hi) {
    const int mid = (lo + hi) >> 1;
    if (load_uniform(st + mid) < step)
      lo = mid + 1;
    else
      hi = mid;
  }
  if (load_uniform(st + lo) != step) return nullptr;
  return screens + in.screen_off + int64_t(lo) * in.n * in.n;
}

// Deterministic workgroup reduction of NV doubles (sum or max); the result
// is valid in thread 0.  red: shared [THREADS/64][NV].
template <int NV, int THREADS, bool MAX>
__device__ __forceinline__ void block_reduce(double (&v)[NV], double* red) {
#pragma unroll
  for (int off = 32; off >= 1; off >>= 1) {
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      const double o = __shfl_xor(v[k], off, 64);
      v[k] = MAX ? fmax(v[k], o) : v[k] + o;
    }
  }
  constexpr int NW = (THREADS + 63) / 64;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0) {
#pragma unroll
    for (int k = 0; k < NV; ++k) red[wave * NV + k] = v[k];
  }
  __syncthreads();
  if (threadIdx.x == 0) {
#pragma unroll
    for (int k = 0; k < NV; ++k) {
      double s = red[k];
      for (int w = 1; w < NW; ++w) s = MAX ? fmax(s, red[w * NV + k]) : s + red[w * NV + k];
      v[k] = s;
    }
  }
}

// Sum of s and maximum of m over a wavefront, valid in every lane, in a
// fixed order.  Each wavefront of a pass stores its own partial: no barrier
// and no LDS between the last wavefront's points and the rest of its pass.
template <int CTRL>
__device__ __forceinline__ double dpp_f64(double x) {
  union {
    double d;
    int i[2];
  } a, b;
  a.d = x;
  b.i[0] = __builtin_amdgcn_update_dpp(0, a.i[0], CTRL, 0xf, 0xf, true);
  b.i[1] = __builtin_amdgcn_update_dpp(0, a.i[1], CTRL, 0xf, 0xf, true);
  return b.d;
}
__device__ __forceinline__ void wave_sum_max(double& s, double& m) {
  // within rows of 16 lanes: exchange pairs, pairs of pairs, then mirror
  // images of 8 and of 16 (equal values on each side by then)
  s += dpp_f64<0xB1>(s);
  m = fmax(m, dpp_f64<0xB1>(m));
  s += dpp_f64<0x4E>(s);
  m = fmax(m, dpp_f64<0x4E>(m));
  s += dpp_f64<0x141>(s);
  m = fmax(m, dpp_f64<0x141>(m));
  s += dpp_f64<0x140>(s);
  m = fmax(m, dpp_f64<0x140>(m));
  s += __shfl_xor(s, 16, 64);
  m = fmax(m, __shfl_xor(m, 16, 64));
  s += __shfl_xor(s, 32, 64);
  m = fmax(m, __shfl_xor(m, 32, 64));
}

// Sums of 8 values over a wavefront in a fixed order: lanes that differ in
// bits 5, 4, 3 exchange the halves they do not keep, so lane l ends with
// the sum of value l >> 3 (10 exchanges instead of 48).
__device__ __forceinline__ double wave_sum8(const double (&g)[8]) {
  const int l = int(threadIdx.x) & 63;
  double h[4], q[2];
  const bool b5 = (l & 32) != 0, b4 = (l & 16) != 0, b3 = (l & 8) != 0;
#pragma unroll
  for (int k = 0; k < 4; ++k)
    h[k] = (b5 ? g[4 + k] : g[k]) + __shfl_xor(b5 ? g[k] : g[4 + k], 32, 64);
#pragma unroll
  for (int k = 0; k < 2; ++k)
    q[k] = (b4 ? h[2 + k] : h[k]) + __shfl_xor(b4 ? h[k] : h[2 + k], 16, 64);
  double s = (b3 ? q[1] : q[0]) + __shfl_xor(b3 ? q[0] : q[1], 8, 64);
  s += dpp_f64<0x141>(s);  // mirror of 8: lanes l and 7 - l
  s += dpp_f64<0xB1>(s);   // neighbours
  s += dpp_f64<0x4E>(s);   // pairs of neighbours
  return s;
}

// dz G(x) of the finite-difference scheme, x = |u|^2 / I_a: the generators
// of the Kerr, plasma and multiphoton terms (each split-step screen term is
// the exact solution of du/dz = G u over one step).
template <typename R>
__device__ __forceinline__ void fd_generator(const ScreenConst<R>& s, R x, R& gr, R& gi) {
  const unsigned tm = s.terms;
  R xk1 = R(0);
  if (tm & (T_MPA | T_PLASMA)) xk1 = ipow(x, s.K - 1);
  gr = R(0);
  gi = R(0);
  if (tm & T_KERR) gi += s.cK * x;
  if (tm & T_PLASMA) gi -= s.cK * x * (R(1) - rcp(R(1) + xk1));
  if (tm & T_MPA) gr -= s.cM * s.inv2k1 * xk1;
}

// A workgroup's tile of a launch and its threads' points: thread t of a
// line holds points t + T e, at element offset toff + STRIDE e from the
// tile's base.
template <class P, bool COL>
struct Tile {
  static constexpr int N = P::N, T = P::T, E = P::E, W = P::LINES;
  static constexpr int PER = N / W;
  static constexpr uint32_t STRIDE = COL ? uint32_t(T) * N : uint32_t(T);
  int tile;       // index in the launch (>= the launch's tiles: none)
  int beam, l0;   // beam of the launch, its first line
  int line, t;    // line within the tile, thread within the line
  uint32_t toff;
  // XCD-aware order: workgroups are dispatched round-robin over the 8 XCDs
  // (blockIdx mod 8); each XCD takes a contiguous run of tiles, so
  // neighbouring lines (which share cache lines in a column pass) meet in
  // one XCD's L2.  The grid is a multiple of 8.
  __device__ __forceinline__ Tile() {
    tile = int((blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3));
    beam = int(unsigned(tile) / unsigned(PER));
    l0 = (tile - beam * PER) * W;
    if constexpr (COL) {
      line = int(threadIdx.x % W);
      t = int(threadIdx.x / W);
      toff = uint32_t(t) * N + uint32_t(line);
    } else {
      line = int(threadIdx.x / T);
      t = int(threadIdx.x) - line * T;
      toff = uint32_t(line) * N + uint32_t(t);
    }
  }
  // element offset of the tile in a field buffer (or, with the beam's own
  // start in off0, in that beam's array)
  __device__ __forceinline__ int64_t in_beam() const {
    return COL ? int64_t(l0) : int64_t(l0) * N;
  }
  __device__ __forceinline__ int64_t base(int64_t off0) const {
    return off0 + int64_t(beam) * N * N + in_beam();
  }
  // recorded fields: line by line along the pass's axis, whichever it is (a
  // field is recorded, marched on from and differentiated by passes of one
  // axis).  Thread point e at kept_off() + T e from kept_base().
  __device__ __forceinline__ int64_t kept_base(int64_t off0) const {
    return off0 + int64_t(beam) * N * N + int64_t(l0) * N;
  }
  __device__ __forceinline__ uint32_t kept_off() const {
    uint32_t o = uint32_t(line) * N + uint32_t(t);
    asm volatile("" : "+v"(o));  // formed where it is used
    return o;
  }
};

template <typename R, class P, bool COL>
struct TileLds {
  using L = std::conditional_t<COL, LdsPointMajor<R, P::LINES, P::PA, P::PB>,
                               LdsLineMajor<R, P::N>>;
  static constexpr int tile() {
    if constexpr (COL)
      return L::size(P::HX ? P::N / 2 : P::N);
    else
      return P::LINES * L::LINE;
  }
  // the twiddle table of a plan that keeps them, at a 16-byte boundary
  static constexpr int table() { return (tile() + 1) / 2 * 2; }
  static constexpr int size() { return table() + mid_table_size<R, P>(); }
  static __device__ __forceinline__ L make(cx<R>* mem, int line) {
    if constexpr (COL)
      return L{mem + line};
    else
      return L{mem + line * L::LINE};
  }
};

template <typename R, class P>
constexpr int waves_target() {
  return sizeof(R) == 4 ? P::WAVES_PER_EU : P::WAVES_PER_EU_F64;
}

// ---------------------------------------------------------- march pass
// PRECISE: the screens call the device library's sincosf (FP32 only).  Its
// argument reduction needs tens of registers, so the kernels that use the
// hardware sine are compiled without it.
template <typename R, class P, bool COL, bool ADJ, bool PRECISE>
__global__ void __launch_bounds__(P::THREADS)
    __attribute__((amdgpu_waves_per_eu(waves_target<R, P>()))) k_march(PassArgs<R> a) {
  constexpr int N = P::N, T = P::T, E = P::E;
  using TL = Tile<P, COL>;
  constexpr uint32_t STRIDE = TL::STRIDE;
  using LD = TileLds<R, P, COL>;
  __shared__ __align__(16) cx<R> lds_mem[LD::size()];
  const TL tl;
  if (tl.tile >= a.n_tiles) return;
  const int64_t base = tl.base(a.off0);
  const Buf<cx<R>> src(static_cast<const cx<R>*>(a.src) + base);
  const int32_t flags = a.flags;
  cx<R> v[E];
  if (COL && !ADJ && (flags & PASS_SRC_KEPT)) {
    const Buf<cx<R>> kept(static_cast<const cx<R>*>(a.src) + tl.kept_base(a.off0));
    const uint32_t ko = tl.kept_off();
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = kept.get(ko, uint32_t(T * e));
  } else {
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = src.get(tl.toff, STRIDE * uint32_t(e));
  }
  const cx<R>* tables = static_cast<const cx<R>*>(a.tables);
  const Buf<cx<R>> prop(tables + a.prop0 + int64_t(tl.beam) * a.prop_stride);
  // plans with few points a thread keep twiddles and propagator in
  // registers for both factors; the others read them as they go
  constexpr bool LATE = P::LATE_TW || P::HX;
  cx<R> pr[P::HX ? 1 : E];
  if constexpr (!LATE) {
#pragma unroll
    for (int e = 0; e < E; ++e) pr[e] = prop.get(uint32_t(tl.t), uint32_t(T * e));
  }
  Twiddles<R, P> tws(tables + a.tw, lds_mem + LD::table(), tl.t);
  const auto lds = LD::make(lds_mem, tl.line);
  const InstDev* ip = a.inst + (a.beam0 + tl.beam);
  const int64_t part_at = int64_t(a.part0) + int64_t(tl.tile) * P::WAVES + (threadIdx.x >> 6);

  bool second = !(flags & PASS_OP1);
#pragma unroll 1
  for (;;) {
    if (second) {
      // thread offset laundered: addresses are formed here, not held from
      // the loads
      uint32_t to = tl.toff;
      asm volatile("" : "+v"(to));
      if constexpr (!ADJ) {
        if (a.rec != nullptr) {
          const Buf<cx<R>> rec(static_cast<const cx<R>*>(a.rec) + tl.kept_base(a.off0));
          const uint32_t ko = tl.kept_off();
#pragma unroll
          for (int e = 0; e < E; ++e) rec.put(ko, uint32_t(T * e), v[e]);
        }
        if ((flags & PASS_SCREEN) || a.part != nullptr) {
          const InstDev in = load_uniform(ip);
          const ScreenConst<R> sc = screen_const<R>(in);
          const R* plane = (flags & PASS_PLANE)
                               ? find_plane(a.screens, a.screen_steps, in, a.step)
                               : nullptr;
          if (plane) plane += tl.in_beam();
          constexpr int SB = 4;  // points per batch
          static_assert(E % SB == 0, "whole batches");
          double s = 0.0, m = 0.0;
#pragma unroll
          for (int c = 0; c < E; c += SB) {
            R x[SB], ph[SB];
#pragma unroll
            for (int e = 0; e < SB; ++e) ph[e] = R(0);
            if (plane) {
#pragma unroll
              for (int e = 0; e < SB; ++e) ph[e] = plane[to + STRIDE * uint32_t(c + e)];
            }
#pragma unroll
            for (int e = 0; e < SB; ++e) x[e] = v[c + e].re * v[c + e].re + v[c + e].im * v[c + e].im;
            const ScreenTerms<R, SB> st(sc, x);
            if (a.part != nullptr) {
              // x A^2 with the A^2 of its own exponential whether or not the
              // screen is applied here: the trace of a march cut anywhere is
              // the same (the square of the screen's A rounds differently)
              R a2[SB];
#pragma unroll
              for (int e = 0; e < SB; ++e) a2[e] = R(1);
              if (!(flags & PASS_RAW)) st.amp2(sc, a2);
#pragma unroll
              for (int e = 0; e < SB; ++e) {
                const double xa = double(x[e]) * double(a2[e]);
                s += xa;
                m = fmax(m, xa);
              }
            }
            if (flags & PASS_SCREEN) st.template apply<PRECISE>(sc, v + c, ph);
          }
          if (a.part != nullptr) {
            wave_sum_max(s, m);
            if ((threadIdx.x & 63) == 0) {
              a.part[part_at * 2 + 0] = s;
              a.part[part_at * 2 + 1] = m;
            }
          }
        }
      } else {
        if (flags & PASS_SCREEN) {
          const InstDev in = load_uniform(ip);
          const ScreenConst<R> sc = screen_const<R>(in);
          const R* plane = (flags & PASS_PLANE)
                               ? find_plane(a.screens, a.screen_steps, in, a.step)
                               : nullptr;
          if (plane) plane += tl.in_beam();
          const Buf<cx<R>> svp(static_cast<const cx<R>*>(a.aux) + tl.kept_base(a.off0));
          const uint32_t ko = tl.kept_off();
          constexpr int AC = 2;  // points per batch
          static_assert(E % AC == 0, "whole batches");
          // each batch's stored field and phases are requested one batch
          // ahead, so their latency overlaps the previous batch's screen
          cx<R> sv[2][AC];
          R ph[2][AC];
          auto load_inputs = [&](int c, int k) {
#pragma unroll
            for (int e = 0; e < AC; ++e) sv[k][e] = svp.get(ko, uint32_t(T * (c + e)));
#pragma unroll
            for (int e = 0; e < AC; ++e) ph[k][e] = R(0);
            if (plane) {
#pragma unroll
              for (int e = 0; e < AC; ++e) ph[k][e] = plane[to + STRIDE * uint32_t(c + e)];
            }
          };
          double g[8] = {0, 0, 0, 0, 0, 0, 0, 0};
          load_inputs(0, 0);
#pragma unroll
          for (int c = 0; c < E; c += AC) {
            const int k = (c / AC) & 1;
            if (c + AC < E) load_inputs(c + AC, k ^ 1);
            screen_adjoint_n<R, AC, PRECISE>(sc, sv[k], v + c, ph[k], plane != nullptr, g);
            // the batch is finished here: left to itself the compiler sinks
            // the last products below the later batches and holds their
            // factors (70 to 100 more registers)
#pragma unroll
            for (int e = c; e < c + AC; ++e) asm volatile("" : "+v"(v[e].re), "+v"(v[e].im));
            __builtin_amdgcn_sched_barrier(0);
          }
          if (in.terms & T_ANSATZ) {
            const double gs = wave_sum8(g);
            const int l = int(threadIdx.x) & 63;
            if ((l & 7) == 0) a.part[part_at * 8 + (l >> 3)] -= in.cK * gs;
          }
        }
      }
      if (!(flags & PASS_OP2)) break;
    }
    tws.keep(tl.t);
    fft_line<R, P, -1>(v, tl.t, lds, tws, [&] {
      if constexpr (LATE && !P::HX) {
        int tp = tl.t;
        asm volatile("" : "+v"(tp));
#pragma unroll
        for (int e = 0; e < E; ++e) pr[e] = prop.get(uint32_t(tp), uint32_t(T * e));
      }
    });
    if constexpr (P::HX) {
      // the points fill the registers: the propagator comes in batches
      constexpr int PB = 4;
      int tp = tl.t;
      asm volatile("" : "+v"(tp));
#pragma unroll
      for (int c = 0; c < E; c += PB) {
        cx<R> q[PB];
#pragma unroll
        for (int e = 0; e < PB; ++e) q[e] = prop.get(uint32_t(tp), uint32_t(T * (c + e)));
#pragma unroll
        for (int e = 0; e < PB; ++e) v[c + e] = ADJ ? cmulc(v[c + e], q[e]) : cmul(v[c + e], q[e]);
        if (c % (4 * PB) == 3 * PB) __builtin_amdgcn_sched_barrier(0);
      }
    } else {
#pragma unroll
      for (int e = 0; e < E; ++e) v[e] = ADJ ? cmulc(v[e], pr[e]) : cmul(v[e], pr[e]);
    }
    fft_line<R, P, +1>(v, tl.t, lds, tws);
    if (second) break;
    second = true;
  }
  if (a.dst == nullptr) return;
  const Buf<cx<R>> dst(static_cast<const cx<R>*>(a.dst) + base);
  uint32_t to = tl.toff;
  asm volatile("" : "+v"(to));
#pragma unroll
  for (int e = 0; e < E; ++e) dst.put(to, STRIDE * uint32_t(e), v[e]);
}

// ------------------------------------------------ screen synthesis pass
// A pair of screens is two launches.  The row pass draws its spectrum as it
// needs it (the work buffer is never loaded) and the column pass adds the
// subharmonic modes to what it has in registers, factored by axis: per
// level and column the three cells of each table exponent of the rows are
// summed first, which leaves four FP64 multiply-adds per point.  Bound by
// the arithmetic of the draws (Philox, FP64 log and sincospi), two in
// flight per thread.
template <typename R, class P, bool COL>
__global__ void __launch_bounds__(P::THREADS) k_inverse(PassArgs<R> a) {
  constexpr int N = P::N, T = P::T, E = P::E;
  using TL = Tile<P, COL>;
  using LD = TileLds<R, P, COL>;
  __shared__ __align__(16) cx<R> lds_mem[LD::size()];
  const TL tl;
  if (tl.tile >= a.n_tiles) return;
  const InstDev in = load_uniform(a.inst + (a.beam0 + tl.beam));
  if (2 * a.pair >= in.n_screens || !(in.terms & T_TURB)) return;
  const int64_t base = tl.base(a.off0);
  const SubBeam sb = load_uniform(static_cast<const SubBeam*>(a.aux) + (a.beam0 + tl.beam));
  cx<R> v[E];
  if constexpr (COL) {
    const cx<R>* __restrict__ src = static_cast<const cx<R>*>(a.src) + base;
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = src[tl.toff + TL::STRIDE * uint32_t(e)];
  } else {
    // through the thread's own LDS slots, so that the draws can loop
    const int row = tl.l0 + tl.line;
#pragma unroll 2
    for (int e = 0; e < E; ++e) {
      double re, im;
      noise_sample(sb, N, row, tl.t + T * e, a.pair, &re, &im);
      lds_mem[e * P::THREADS + int(threadIdx.x)] = {R(re), R(im)};
    }
#pragma unroll
    for (int e = 0; e < E; ++e) v[e] = lds_mem[e * P::THREADS + int(threadIdx.x)];
    __syncthreads();  // the transform's slots are other threads'
  }
  Twiddles<R, P> tws(static_cast<const cx<R>*>(a.tables) + a.tw, lds_mem + LD::table(), tl.t);
  tws.keep(tl.t);
  fft_line<R, P, +1>(v, tl.t, LD::make(lds_mem, tl.line), tws);
  if constexpr (COL) {
    // screen pair: real part -> plane 2p, imaginary part -> plane 2p+1
    R* pre = a.planes_out + in.screen_off + int64_t(2 * a.pair) * N * N + tl.l0;
    R* pim = pre + int64_t(N) * N;
    const bool has_im = 2 * a.pair + 1 < in.n_screens;
    if (sb.sp.levels > 0) {
      const double* region = static_cast<const double*>(a.state);
      const double* blk = region + sb.coef_off + int64_t(kSubPair) * a.pair;
      const double* tab = region + sb.tab_off;
      const int col = tl.l0 + tl.line;
      double sre[E], sim[E];
#pragma unroll
      for (int e = 0; e < E; ++e) {
        sre[e] = -blk[128];
        sim[e] = -blk[129];
      }
#pragma unroll 1
      for (int p = 0; p < sb.sp.levels; ++p) {
        const double xr = tab[2 * (p * N + col)], xi = tab[2 * (p * N + col) + 1];
        const double* w = blk + 16 * p;
        // b[iy]: the cells q = 3 iy + ix (without q = 4) over ix, with
        // e^{i a ix} = conj(x), 1, x
        double br[3], bi[3];
#pragma unroll
        for (int iy = 0; iy < 3; ++iy) {
          const int j0 = (iy < 2) ? 3 * iy : 5;         // cell (0, iy)
          const int j2 = (iy == 0) ? 2 : j0 + (iy == 1 ? 1 : 2);  // cell (2, iy)
          const double lr = w[2 * j0], li = w[2 * j0 + 1];
          const double hr = w[2 * j2], hi = w[2 * j2 + 1];
          br[iy] = (lr + hr) * xr + (li - hi) * xi;
          bi[iy] = (li + hi) * xr + (hr - lr) * xi;
          if (iy != 1) {
            br[iy] += w[2 * (j0 + 1)];
            bi[iy] += w[2 * (j0 + 1) + 1];
          }
        }
        const double sr = br[0] + br[2], si = bi[0] + bi[2];
        const double dr = br[2] - br[0], di = bi[0] - bi[2];
#pragma unroll
        for (int e = 0; e < E; ++e) {
          const int row = tl.t + T * e;
          const double yr = tab[2 * (p * N + row)], yi = tab[2 * (p * N + row) + 1];
          sre[e] += br[1] + sr * yr + di * yi;
          sim[e] += bi[1] + si * yr + dr * yi;
        }
      }
#pragma unroll
      for (int e = 0; e < E; ++e) v[e] = {R(double(v[e].re) + sre[e]), R(double(v[e].im) + sim[e])};
    }
#pragma unroll
    for (int e = 0; e < E; ++e) {
      pre[tl.toff + TL::STRIDE * uint32_t(e)] = v[e].re;
      if (has_im) pim[tl.toff + TL::STRIDE * uint32_t(e)] = v[e].im;
    }
  } else {
    cx<R>* __restrict__ dst = static_cast<cx<R>*>(a.dst) + base;
#pragma unroll
    for (int e = 0; e < E; ++e) dst[tl.toff + TL::STRIDE * uint32_t(e)] = v[e];
  }
}

// ------------------------------------------- finite-difference row pass
template <typename R, class P>
__global__ void __launch_bounds__(P::THREADS) k_fd_row(PassArgs<R> a) {
  constexpr int T = P::T, E = P::E;
  using TL = Tile<P, false>;
  using LD = TileLds<R, P, false>;
  __shared__ __align__(16) cx<R> lds_mem[LD::size()];
  const TL tl;
  if (tl.tile >= a.n_tiles) return;
  const int64_t base = tl.base(a.off0);
  const cx<R>* __restrict__ src = static_cast<const cx<R>*>(a.src) + base;
  cx<R>* __restrict__ st = static_cast<cx<R>*>(a.state) + base;
  cx<R>* __restrict__ dst = static_cast<cx<R>*>(a.dst) + base;
  // v is Ubar row-transformed (the column pass applied the solve and both
  // 1/N), or U itself when the step starts
  cx<R> v[E], un[E];
#pragma unroll
  for (int e = 0; e < E; ++e) v[e] = src[tl.toff + uint32_t(T * e)];
#pragma unroll
  for (int e = 0; e < E; ++e) un[e] = st[tl.toff + uint32_t(T * e)];
  Twiddles<R, P> tws(static_cast<const cx<R>*>(a.tables) + a.tw, lds_mem + LD::table(), tl.t);
  tws.keep(tl.t);
  const auto lds = LD::make(lds_mem, tl.line);
  const InstDev in = load_uniform(a.inst + (a.beam0 + tl.beam));
  const ScreenConst<R> sc = screen_const<R>(in);
  if (a.flags & FD_SPECTRAL) fft_line<R, P, +1>(v, tl.t, lds, tws);
  if (a.flags & FD_FINISH) {
    // U+ = 2 Ubar - U, its power partials; it is the next step's U and
    // its first Ubar
    double s = 0.0, m = 0.0;
#pragma unroll
    for (int e = 0; e < E; ++e) {
      v[e] = {R(2) * v[e].re - un[e].re, R(2) * v[e].im - un[e].im};
      st[tl.toff + uint32_t(T * e)] = v[e];
      const double x = double(v[e].re) * double(v[e].re) + double(v[e].im) * double(v[e].im);
      s += x;
      m = fmax(m, x);
      un[e] = v[e];
    }
    if (a.part != nullptr) {
      wave_sum_max(s, m);
      if ((threadIdx.x & 63) == 0) {
        const int64_t at = int64_t(a.part0) + int64_t(tl.tile) * P::WAVES + (threadIdx.x >> 6);
        a.part[at * 2 + 0] = s;
        a.part[at * 2 + 1] = m;
      }
    }
    if (a.flags & FD_LAST) return;
  }
  // right-hand side U + (dz/2) G(J) Ubar, J = (|2 Ubar - U|^2 + |U|^2) / 2
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const R dr = R(2) * v[e].re - un[e].re, di = R(2) * v[e].im - un[e].im;
    const R j = R(0.5) * (dr * dr + di * di + un[e].re * un[e].re + un[e].im * un[e].im);
    R gr, gi;
    fd_generator<R>(sc, j, gr, gi);
    gr *= R(0.5);
    gi *= R(0.5);
    v[e] = {un[e].re + (gr * v[e].re - gi * v[e].im), un[e].im + (gr * v[e].im + gi * v[e].re)};
  }
  fft_line<R, P, -1>(v, tl.t, lds, tws);
#pragma unroll
  for (int e = 0; e < E; ++e) dst[tl.toff + uint32_t(T * e)] = v[e];
}

// ---------------------------------------- finite-difference column pass
// (1 - (i dz/4k0) Lap_h)^-1 = 1 / (1 + i (d[kx] + d[ky])) with the 1/N^2 of
// both inverse DFTs; the table holds d[m] = (dz/4k0)(4/dx^2) sin^2(pi m / N)
// in its real parts.
template <typename R, class P>
__global__ void __launch_bounds__(P::THREADS) k_fd_col(PassArgs<R> a) {
  constexpr int N = P::N, T = P::T, E = P::E;
  using TL = Tile<P, true>;
  using LD = TileLds<R, P, true>;
  __shared__ __align__(16) cx<R> lds_mem[LD::size()];
  const TL tl;
  if (tl.tile >= a.n_tiles) return;
  const int64_t base = tl.base(a.off0);
  const cx<R>* __restrict__ src = static_cast<const cx<R>*>(a.src) + base;
  cx<R>* __restrict__ dst = static_cast<cx<R>*>(a.dst) + base;
  const cx<R>* tables = static_cast<const cx<R>*>(a.tables);
  const cx<R>* __restrict__ prop = tables + a.prop0 + int64_t(tl.beam) * a.prop_stride;
  cx<R> v[E];
#pragma unroll
  for (int e = 0; e < E; ++e) v[e] = src[tl.toff + TL::STRIDE * uint32_t(e)];
  const R dkx = prop[tl.l0 + tl.line].re;
  Twiddles<R, P> tws(tables + a.tw, lds_mem + LD::table(), tl.t);
  tws.keep(tl.t);
  const auto lds = LD::make(lds_mem, tl.line);
  fft_line<R, P, -1>(v, tl.t, lds, tws);
  int tp = tl.t;
  asm volatile("" : "+v"(tp));
  const R inv_n2 = R(1) / (R(N) * R(N));
#pragma unroll
  for (int e = 0; e < E; ++e) {
    const R sm = dkx + prop[uint32_t(tp + T * e)].re;
    const R den = inv_n2 / (R(1) + sm * sm);
    v[e] = cmul(v[e], cx<R>{den, -sm * den});
  }
  fft_line<R, P, +1>(v, tl.t, lds, tws);
  uint32_t to = tl.toff;
  asm volatile("" : "+v"(to));
#pragma unroll
  for (int e = 0; e < E; ++e) dst[to + TL::STRIDE * uint32_t(e)] = v[e];
}

// -------------------------------------------------------------- launch
// With ev, the launch carries start/stop events on its own dispatch (timing
// of the kernel alone, no separate marker packets).
template <typename R, class P>
hipError_t launch_kernel(void (*k)(PassArgs<R>), const PassArgs<R>& a, hipStream_t s,
                         const LaunchEv* ev) {
  const dim3 grid(unsigned((a.n_tiles + 7) / 8 * 8));
  if (ev)
    hipExtLaunchKernelGGL(k, grid, dim3(P::THREADS), 0, s, ev->start, ev->stop, 0, a);
  else
    hipLaunchKernelGGL(k, grid, dim3(P::THREADS), 0, s, a);
  return hipGetLastError();
}

// Column passes of half-exchange plans (their kernels are compiled in a
// unit of their own, pass_col_hx_f32.hip).
template <typename R, class P, int KIND>
hipError_t launch_hx(const PassArgs<R>& a, hipStream_t s, const LaunchEv* ev);

template <typename R, class P, int KIND>
hipError_t launch_built(const PassArgs<R>& a, hipStream_t s, const LaunchEv* ev) {
  if constexpr (KIND == ROW_FWD || KIND == ROW_ADJ || KIND == COL_FWD || KIND == COL_ADJ) {
    constexpr bool COL = is_col_kind(KIND), ADJ = KIND == ROW_ADJ || KIND == COL_ADJ;
    if constexpr (sizeof(R) == 4)
      if (a.precise) return launch_kernel<R, P>(k_march<R, P, COL, ADJ, true>, a, s, ev);
    return launch_kernel<R, P>(k_march<R, P, COL, ADJ, false>, a, s, ev);
  }
  else if constexpr (KIND == ROW_INV || KIND == COL_INV)
    return launch_kernel<R, P>(k_inverse<R, P, KIND == COL_INV>, a, s, ev);
  else if constexpr (KIND == ROW_FD)
    return launch_kernel<R, P>(k_fd_row<R, P>, a, s, ev);
  else
    return launch_kernel<R, P>(k_fd_col<R, P>, a, s, ev);
}

// A plan whose LDS tile does not fit a workgroup at this precision is not
// built for it.
template <typename R, class P, int KIND>
hipError_t launch_one(const PassArgs<R>& a, hipStream_t s, const LaunchEv* ev) {
  if constexpr (!plan_fits<R, P>(is_col_kind(KIND)))
    return hipErrorInvalidValue;
  else if constexpr (P::HX)
    return launch_hx<R, P, KIND>(a, s, ev);
  else
    return launch_built<R, P, KIND>(a, s, ev);
}

template <typename R, int KIND>
hipError_t launch_row_kind(int n, int v, const PassArgs<R>& a, hipStream_t s,
                           const LaunchEv* ev) {
#define SSFM_RCASE(NN, VV, ...) \
  if (n == NN && v == VV)       \
    return launch_one<R, typename RowPlanSel<NN, VV>::P, KIND>(a, s, ev);
  SSFM_ROW_PLANS(SSFM_RCASE)
#undef SSFM_RCASE
  return hipErrorInvalidValue;
}

template <typename R, int KIND>
hipError_t launch_col_kind(int n, int v, const PassArgs<R>& a, hipStream_t s,
                           const LaunchEv* ev) {
#define SSFM_CCASE(NN, VV, ...) \
  if (n == NN && v == VV)       \
    return launch_one<R, typename ColPlanSel<NN, VV>::P, KIND>(a, s, ev);
  SSFM_COL_PLANS(SSFM_CCASE)
#undef SSFM_CCASE
  return hipErrorInvalidValue;
}

// Per-unit entry points (defined in pass_{row,col}_{f32,f64}.hip).
template <typename R>
hipError_t launch_row(int kind, int n, int v, const PassArgs<R>& a, hipStream_t s,
                      const LaunchEv* ev);
template <typename R>
hipError_t launch_col(int kind, int n, int v, const PassArgs<R>& a, hipStream_t s,
                      const LaunchEv* ev);

}  // namespace ssfm
