// kernels.hpp -- host-visible interface of the HIP kernels (launch wrappers).
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "internal.hpp"

namespace ssfm {

template <typename R>
struct cx;

// Pass kinds.  The diffraction factor is a product of a row and a column
// factor, which commute, so the march takes them in alternating order: an
// even step diffracts along the rows first, an odd one along the columns.
// The second factor of a step, its screen and the first factor of the next
// step then act along one axis, and one ROW_FWD or COL_FWD pass does all
// three on lines it reads and writes once.  ROW_ADJ / COL_ADJ are the same
// for the adjoint.  ROW_INV / COL_INV are plain inverse DFTs for screen
// synthesis.  ROW_FD / COL_FD are the finite-difference reference scheme's
// passes: COL_FD applies the inverse of 1 - (i dz/4k0) Lap_h between a
// forward and an inverse column DFT (Lap_h diagonal in the 2-D DFT basis),
// ROW_FD inverts the row DFT, forms the next right-hand side pointwise (or
// finishes the step) and transforms the rows again.
enum PassKind {
  ROW_FWD = 0, ROW_ADJ = 1, ROW_INV = 2, COL_FWD = 3, COL_ADJ = 4, COL_INV = 5,
  ROW_FD = 6, COL_FD = 7
};
constexpr bool is_col_kind(int k) {
  return k == COL_FWD || k == COL_ADJ || k == COL_INV || k == COL_FD;
}

// Parts of a march pass (ROW_FWD, COL_FWD, ROW_ADJ, COL_ADJ), in the order
// they act: the diffraction factor of the step that ends, the screen (its
// adjoint), the factor of the step that begins.  PASS_RAW: the power
// partials are those of |V|^2 without the screen's A^2; PASS_PLANE: some
// beam of the launch may have a turbulence plane at this step (else none is
// looked for); PASS_SRC_KEPT: src is a recorded field (*_FWD).
enum : int32_t {
  PASS_OP1 = 1, PASS_SCREEN = 2, PASS_OP2 = 4, PASS_RAW = 8, PASS_PLANE = 16, PASS_SRC_KEPT = 32
};
// ROW_FD flags: the input is row-transformed (else it is U itself), the pass
// finishes the step (U+ = 2 Ubar - U into the state, power partials), the
// finished step is the last one of the launch sequence (no next RHS).
enum : int32_t { FD_SPECTRAL = 2, FD_FINISH = 4, FD_LAST = 8 };

// Start/stop events carried by one pass launch (sampled timing).
struct LaunchEv {
  hipEvent_t start, stop;
};

// One launch covers the beams of one grid size, which are consecutive in
// the beam table and in every field buffer: tile t of the launch holds
// lines (t mod per) LINES .. of beam beam0 + t / per, per = n / LINES.
template <typename R>
struct PassArgs {
  const void* src;            // cx<R> field buffer read
  void* dst;                  // cx<R> field buffer written (*_FWD: or null)
  const void* aux;            // *_ADJ: recorded pre-screen field V of the screen (cx<R>);
                              // *_INV: the screens' spectra (SubBeam per beam)
  void* rec;                  // *_FWD: pre-screen field V recorded here too (or null)
  void* state;                // ROW_FD: U of the step (read; U+ written when finishing);
                              // COL_INV: the subharmonic region (read)
  const InstDev* inst;        // beam table
  const void* tables;         // cx<R> twiddle and propagator tables
  const R* screens;           // turbulence planes (read)
  R* planes_out;              // COL_INV: screen planes (write)
  const int64_t* screen_steps;  // per-beam sorted step lists
  double* part;               // *_FWD, ROW_FD: per wavefront {sum x A^2, max x A^2};
                              // *_ADJ: per wavefront 8 theta accumulators
  int64_t step;               // step whose screen the pass applies
  int64_t off0;               // element offset of the launch's first beam in a field buffer
  int64_t prop0;              // element offset of its propagator (filter, solve) table
  int64_t tw;                 // element offset of the plan's stage-ordered twiddles
  int32_t prop_stride;        // elements from one beam's table to the next one's
  int32_t beam0;              // beam table index of the first beam
  int32_t part0;              // partials of the beams before it
  int32_t n_tiles;            // tiles of the launch
  int32_t pair;               // *_INV: screen pair index
  int32_t flags;              // march passes: PASS_*; ROW_FD: FD_*
  int32_t precise;            // library sine and cosine in the screens (FP32)
};

struct PlanInfo {
  int threads;   // workgroup size
  int lines;     // lines per workgroup
  int waves;     // wavefronts per workgroup (each writes its own partials)
  int t;         // threads per line
  size_t lds;    // static LDS bytes
  int radices[8];  // radix plan in stage order, ended by 0
};

// Number of variants, the default one, and their shape for (kind is column?,
// n, precision).
int plan_default(bool column, int n, bool fp64);
int plan_count(bool column, int n);
bool plan_info(bool column, int n, int variant, bool fp64, PlanInfo* out);

template <typename R>
hipError_t launch_pass(int kind, int n, int variant, const PassArgs<R>& a, hipStream_t s,
                       const LaunchEv* ev = nullptr);

// Pointwise helpers -------------------------------------------------------

// dst (cx<R> device state, beam b at off) = src (complex128 SI) * scale; the
// beam's entry goes to its slot of the beam table with it (a launch of its
// own for each: 12 beams of 256^2 took 703 us an evaluation, so 678)
template <typename R>
hipError_t launch_load_field(const double* src, void* dst, int64_t n_elem, double scale,
                             const InstDev& entry, InstDev* slot, hipStream_t s);

// dst (complex128 SI) = sqrt(I_a) * [pending screen](state); optionally
// intensity only (float64 I = I_a |u|^2).
template <typename R>
hipError_t launch_store_field(const void* state, const InstDev* inst, int b,
                              int n, const R* screens,
                              const int64_t* screen_steps, int64_t pending_step,
                              double out_scale, double* dst, bool intensity,
                              hipStream_t s);

// Loss / cotangent seed.  For each point of beam b: u_N = screen(s_N);
// mode 0 (g_scale = I_a): I = I_a |u|^2, partial sums of (I - w)^2 and
// G_u = 4 (I - w) I_a u / sum w^2 (w_part: launch_sumsq's sums of w^2, SI;
// part_loss[n] gets their sum);
// mode 1 (g_scale = sqrt(I_a)): G_u = sqrt(I_a) G_ext (G_ext in SI).
// Then the adjoint of the pending screen writes mu_N = S^*(G_u) into lam and
// the ansatz terms of that screen go to part_theta[row][8].
template <typename R>
hipError_t launch_seed(int mode, const void* state, const InstDev* inst, int b,
                       int n, const R* screens, const int64_t* screen_steps,
                       int64_t pending_step, const double* target,
                       const double* w_part, const double* g_ext,
                       double g_scale, void* lam, double* part_loss,
                       double* part_theta, int n_blocks, hipStream_t s);

template <typename R>
hipError_t launch_copy(const void* src, void* dst, int64_t n_elem, hipStream_t s);

// For beams [b0, b0 + n_beams): reduce the diag partials of `steps`
// consecutive steps, stride entries each: part[step][stride][2] ->
// diag[b][(ring0 + step) % cap][2].  Beam b's partials of a step are entries
// [begin[b], begin[b + 1]); begin is begin_even for even steps (ring0 +
// step) and begin_odd for odd ones.
hipError_t launch_diag_finalize(const double* part, int64_t stride, const int32_t* begin_even,
                                const int32_t* begin_odd, int b0, int n_beams, int steps,
                                double* diag, int64_t ring0, int64_t cap, hipStream_t s);

// Per beam the fixed-order sum of its entries of two [entries][8] FP64
// arrays (row-pass and column-pass accumulators).
hipError_t launch_reduce_theta(const double* rows, const int32_t* row_begin, const double* cols,
                               const int32_t* col_begin, int n_beams, double* out,
                               hipStream_t s);

// kSumParts partial sums of the squares of a float64 array.
constexpr int kSumParts = 256;
hipError_t launch_sumsq(const double* x, int64_t n, double* partial, hipStream_t s);

// Copies `count` records (beam table entries, screen spectra) from host
// memory to dst, by value.
template <typename T>
hipError_t launch_put(const T* src, int count, T* dst, hipStream_t s);

// The screen of step `pending` on every beam's state, in place.
template <typename R>
hipError_t launch_flush(void* state, const InstDev* inst, int n_beams, int max_n, const R* screens,
                        const int64_t* steps, int64_t pending, hipStream_t s);

// Beam b's fluence mismatch (pending: as in launch_store_field): part[row] =
// sum (I - w)^2 over a row, then launch_sumsq's partials of sum w^2.
template <typename R>
hipError_t launch_mismatch(const void* state, const InstDev* inst, int b, int n, const R* screens,
                           const int64_t* steps, int64_t pending, const double* target,
                           double i_ref, double* part, hipStream_t s);

template <typename R>
hipError_t launch_screen_to_f64(const R* plane, int64_t n_elem, double* dst,
                                hipStream_t s);

hipError_t launch_fill_f64(double* p, int64_t n, double v, hipStream_t s);

// Effective lens: FP64 parameters of one application (SI; segments
// {r_end, amplitude, frequency, phase}).
struct LensDev {
  double i_ref, w_l, c1, c2;
  int32_t n_re, n_im;
  double re[8][4];
  double im[8][4];
};
// wk[i] = (|s[i]|^2, 0) over all n_elem points (device units).
template <typename R>
hipError_t launch_lens_prep(const void* s, void* wk, int64_t n_elem, hipStream_t st);
// u[i] *= exp(i f(w_dif[i])) over one beam's n2 points where w_dif >= w_l.
template <typename R>
hipError_t launch_lens_apply(void* u, const void* wdif, int64_t n2, const LensDev& p,
                             hipStream_t st);

// Hot-area count of an n x n FP64 array (labels: n^2 ints of scratch):
// regions, and whether a union exceeded its retry cap.
struct HotResult {
  int64_t regions;
  int32_t overflow;
  int32_t pad;
};
hipError_t launch_hot_areas(const double* w, int n, double threshold, int periodic, int* labels,
                            HotResult* res, hipStream_t s);
// Spatial moment partial sums (n_part blocks).
hipError_t launch_moment(const double* w, int n, double dx, double p, int m, double* part,
                         int n_part, hipStream_t s);
// Measure-vector partials: n_part blocks x [sum w, sum w r^2, sum w^2,
// sum w^2 r^2, max w].
hipError_t launch_measure(const double* w, int n, double dx, double* part, int n_part,
                          hipStream_t s);

hipError_t launch_block_mean(const double* src, int n, int b, double* dst,
                             hipStream_t s);

// Allocation-free hot-area count: a file-scope device array (one per GPU)
// holds the labels of grids up to kStaticMaxN^2 and the result at
// kStaticResultOff.
constexpr int kStaticMaxN = 2048;
constexpr size_t kStaticResultOff = size_t(kStaticMaxN) * kStaticMaxN * sizeof(int);
constexpr size_t kStaticScratchBytes = kStaticResultOff + 4096;
// Device address of the current device's copy (looked up once per device).
hipError_t static_scratch(void** out);

}  // namespace ssfm
