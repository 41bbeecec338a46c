// ssfm.cpp -- host plan, workspace layout and the C ABI of libssfm.
//
// The host side turns beam descriptions into device tables (twiddles and
// diffraction factors computed in FP64 and rounded once, per-beam screen
// constants) and drives the march:
//
//   forward  one pass per step: the diffraction factor that ends step n, its
//            screen, the factor that begins step n+1, along one axis; the
//            axis alternates from step to step (see pass_kernels.hpp)
//   adjoint  the same passes in reverse
//
// All beams of a context march by the same number of steps; beams of equal
// grid size are neighbours in every table and buffer and share one launch
// per pass, so a batch of uneven beams costs one launch per distinct size
// per pass.  The sizes march as independent chains, forked and joined once
// per call (captured once into a HIP graph and replayed).
#include "../../include/ssfm.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <array>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <map>
#include <memory>
#include <string>
#include <tuple>
#include <vector>

#include "internal.hpp"
#include "kernels.hpp"
#include "lens_vjp.hpp"
#include "subharmonics.hpp"

using namespace ssfm;

namespace {

thread_local std::string g_last_error;

int fail(int status, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  g_last_error = buf;
  return status;
}

#define HIP_TRY(expr)                                                              \
  do {                                                                             \
    hipError_t e_ = (expr);                                                        \
    if (e_ != hipSuccess)                                                          \
      return fail(SSFM_EHIP, "%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_), \
                  __FILE__, __LINE__);                                             \
  } while (0)

constexpr int kDiagChunk = 64;
constexpr size_t kAlign = 256;

size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

bool supported_n(int n) {
  return n == 128 || n == 256 || n == 512 || n == 768 || n == 1024 || n == 2048 || n == 4096;
}

int validate_desc(const ssfm_instance_desc* d, int32_t n_inst, int32_t precision) {
  if (!d) return fail(SSFM_EINVAL, "desc is NULL");
  if (n_inst < 1 || n_inst > 65536) return fail(SSFM_EINVAL, "n_inst %d out of range", n_inst);
  if (precision != SSFM_FP32 && precision != SSFM_FP64)
    return fail(SSFM_EINVAL, "precision must be 32 or 64, got %d", precision);
  for (int i = 0; i < n_inst; ++i) {
    const ssfm_instance_desc& x = d[i];
    if (!supported_n(x.n))
      return fail(SSFM_EUNSUPPORTED, "instance %d: grid size %d not supported", i, x.n);
    if (!(x.length > 0) || !(x.dz > 0) || !(x.wavelength > 0) || !(x.i_ref > 0))
      return fail(SSFM_EINVAL, "instance %d: length, dz, wavelength, i_ref must be > 0", i);
    if (x.terms & ~31u) return fail(SSFM_EINVAL, "instance %d: unknown term bits", i);
    if ((x.terms & (SSFM_MPA | SSFM_PLASMA)) && x.mpa_order < 2)
      return fail(SSFM_EINVAL, "instance %d: mpa_order must be >= 2", i);
    if (x.mpa_order > 32) return fail(SSFM_EINVAL, "instance %d: mpa_order > 32", i);
    if (x.n_screens < 0 || x.n_screens > 4096)
      return fail(SSFM_EINVAL, "instance %d: n_screens out of range", i);
    if ((x.terms & SSFM_TURB) && x.n_screens > 0 && (!(x.screen_dz > 0) || !(x.cn2 >= 0)))
      return fail(SSFM_EINVAL, "instance %d: turbulence needs screen_dz > 0, cn2 >= 0", i);
    // closer screens could fall on one step (or before the first one)
    if ((x.terms & SSFM_TURB) && x.n_screens > 0 && !(x.screen_dz >= x.dz))
      return fail(SSFM_EINVAL, "instance %d: screen_dz %g below dz %g", i, x.screen_dz, x.dz);
  }
  return SSFM_OK;
}

// Device-side layout of everything a context keeps in the workspace.
struct Layout {
  size_t inst, steps, begins, tables;
  // theta_rows, theta_cols: theta accumulators of the adjoint passes; the
  // region at theta_rows also takes the power partials of finite-difference
  // marches (fd_chunk steps of them) and of timed passes.  Those of the other
  // marches, which leave the work buffer alone, go there.  One for each
  // wavefront, sized for any variant, the partials would be up to a fifth of
  // a batch's workspace in regions of their own.
  size_t S, Wk, Lam, ckpt, stack, screens, stage, diag, theta_rows, theta_cols, theta_out,
      seed_loss, seed_theta, sumsq_part, subh, subh_beams;
  size_t total;
  int64_t field_elems;  // sum n^2
  int64_t table_elems;
  int64_t part_stride;  // power partials of one step (room for any variant, either axis)
  int64_t theta_row_parts, theta_col_parts;  // theta accumulators of the adjoint passes
  int fd_chunk;
  int64_t n_ckpt, n_stack, diag_cap, screen_elems, n_steps_total;
  // regions of n_stack segment slots: recompute banks (0, 1 or 2) and
  // segments kept whole by the forward record
  int64_t n_banks, n_kept;
  int max_n;
};

// The passes a beam size runs through: variants of the forward and adjoint
// row and column pass.
enum PassSlot { P_ROW = 0, P_COL = 1, P_ROW_ADJ = 2, P_COL_ADJ = 3, P_SLOTS = 4 };
// Tables of n entries each beam keeps: propagator, lens filter, half steps
// forward and back, finite-difference solve.
enum BeamTable { T_PROP = 0, T_LENS = 1, T_HALF = 2, T_BACK = 3, T_FD = 4, T_COUNT = 5 };

// Beams of one grid size: consecutive in the beam table and every buffer.
struct Group {
  int n;
  int beam0 = 0, count = 0;
  // variants of the adjoint passes may be -1: the forward ones
  int var[P_SLOTS] = {0, 0, -1, -1};
  int64_t tw = 0;     // element offset of P_SLOTS stage-ordered twiddle tables, n entries each
  int64_t prop = 0;   // element offset of beam0's tables (T_COUNT n entries per beam)
  int32_t part0[P_SLOTS] = {0, 0, 0, 0};  // first partial of beam0 in each pass
  int lines[P_SLOTS] = {0, 0, 0, 0};      // lines per workgroup of each pass
  int variant(int slot) const {
    return (slot >= P_ROW_ADJ && var[slot] < 0) ? var[slot - P_ROW_ADJ] : var[slot];
  }
};

}  // namespace

struct ssfm_ctx {
  int precision = SSFM_FP32;
  size_t el = 8;  // bytes per complex element
  // beams in the order of the groups (equal sizes together); slot[i] is the
  // position of the caller's instance i, caller[b] the instance at position b
  std::vector<ssfm_instance_desc> desc;
  std::vector<int32_t> slot, caller;
  std::vector<InstDev> inst;
  std::vector<int64_t> screen_steps;
  // Strang splitting: the state holds V = L(dz/2) U and every step applies
  // its own screen on load
  bool strang = false;
  // finite-difference reference scheme (Crank-Nicolson, fixed-point
  // iterations per step)
  bool fd = false;
  int fd_iters = 4;
  bool precise = false;  // library sine and cosine in the FP32 screens
  // radix plans whose twiddles the device holds, per size group and pass
  std::vector<std::array<std::vector<int>, P_SLOTS>> tw_radices;
  struct Spectrum {
    int kind = SSFM_SPECTRUM_KOLMOGOROV;
    double tau = 0.0, kappa_h = 0.0;
    int subharmonics = 0;  // subharmonic levels added to each screen
  };
  std::vector<Spectrum> spectrum;  // per beam, for gen_screens
  std::vector<Group> groups;
  std::vector<int32_t> begins;  // P_SLOTS lists of n_inst + 1 first partials per beam
  Layout L{};
  char* ws = nullptr;
  hipStream_t stream = nullptr;
  int64_t max_steps = 0;
  int32_t ckpt_every = 1;
  int32_t stored_segments = 0;  // last segments of a record kept whole
  // march state
  int64_t step = 0;        // steps taken since the last set_field
  bool pending = false;    // state holds V with its screen still to apply
  int64_t diag_valid = 0;  // steps of diag kept from the last call
  // adjoint record
  int64_t rec_steps = 0, rec_step0 = 0;
  bool rec_valid = false, seeded = false, grads_valid = false;
  // backward sweep: recompute of the next segment on the second stream
  // beside the adjoint of the current one (else after it, on the stream)
  bool overlap_recompute = false;
  std::vector<char> seeded_beam;  // per beam: cotangent set since the record
  bool use_graphs = true;
  // captured marches by (kind, a, b, i0, i1) and the steps at which the
  // turbulent beams' fields were set: the passes hold whether a turbulence
  // screen acts on them
  using GraphKey = std::tuple<int, int64_t, int64_t, int64_t, int64_t, std::vector<int64_t>>;
  std::map<GraphKey, hipGraphExec_t> graphs;
  // Sampled pass timing (0: off): with timing_every = m, the pass that ends
  // step s of a forward march, s % m == m / 2, runs outside the step
  // graphs, launched with start/stop events on its own dispatch, and so
  // does a neighbouring pass (along the other axis); samples holds those of
  // the most recent forward march.  ev[2 g + {0, 1}]: start/stop for size
  // group g.
  struct PassSample {
    std::vector<hipEvent_t> ev;
    bool col = false;
  };
  int32_t timing_every = 0;
  std::vector<PassSample> samples, free_samples;
  int32_t n_samples = 0;
  // samples of the most recent backward: adjoint steps s of its first
  // segment (which runs alone, not beside a recompute) with
  // s % timing_every == timing_every / 2, and the pass after each
  std::vector<PassSample> adj_samples;
  int32_t n_adj_samples = 0;
  // second stream (default priority) and events for the overlapped backward
  hipStream_t aux = nullptr;
  hipEvent_t ev_fork = nullptr, ev_join = nullptr;
  // streams and events for running the grid-size groups of one pass
  // concurrently on the main chain (group g > 0 on gstream[g - 1])
  std::vector<hipStream_t> gstream;
  std::vector<hipEvent_t> gjoin;
  hipEvent_t gfork = nullptr;

  template <typename T>
  T* at(size_t off) const {
    return reinterpret_cast<T*>(ws + off);
  }
  void* field(size_t off, int64_t k = 0) const {
    return ws + off + size_t(k) * size_t(L.field_elems) * el;
  }
  static void destroy(std::vector<PassSample>& v) {
    for (auto& e : v)
      for (auto x : e.ev) (void)hipEventDestroy(x);
    v.clear();
  }
  ~ssfm_ctx() {
    for (auto& kv : graphs) (void)hipGraphExecDestroy(kv.second);
    destroy(samples);
    destroy(free_samples);
    destroy(adj_samples);
    if (ev_fork) (void)hipEventDestroy(ev_fork);
    if (ev_join) (void)hipEventDestroy(ev_join);
    if (aux) (void)hipStreamDestroy(aux);
    for (auto s : gstream) (void)hipStreamDestroy(s);
    for (auto e : gjoin) (void)hipEventDestroy(e);
    if (gfork) (void)hipEventDestroy(gfork);
  }
};

namespace {

// Per-beam screen step list (turbulence): screen s (1-based) sits at
// z_s = (s - 1/2) dz_s and is applied after step floor(z_s / dz + 1/2) - 1
// (the step that reaches z_s; ties round up).
std::vector<int64_t> screen_step_list(const ssfm_instance_desc& d) {
  std::vector<int64_t> out;
  if (!(d.terms & SSFM_TURB)) return out;
  for (int s = 1; s <= d.n_screens; ++s) {
    const double zs = (s - 0.5) * d.screen_dz;
    out.push_back(int64_t(std::floor(zs / d.dz + 0.5)) - 1);
  }
  return out;
}

// Eq. (10) band in mode-index units: the Fourier mode m = (mx, my) of a
// window of side L has kappa = 2 pi |m| / L, so kappa <= kappa_h reads
// |m|^2 <= (kappa_h L / 2 pi)^2.  That bound is formed once here, with a
// relative slack of 2^-40 so that a kappa_h placed on a ring of modes keeps
// the ring whatever the rounding; the kernels then decide on the exact
// integer |m|^2.
double band_q2(double length, double kappa_h) {
#pragma clang fp contract(off)
  const double q = kappa_h * length / (2.0 * M_PI);
  return q * q * (1.0 + 0x1p-40);
}

// Beams in group order: by grid size in first-appearance order, beams of
// one size in the caller's order.  order[b]: the caller's index of beam b.
std::vector<int32_t> group_order(const ssfm_instance_desc* d, int n_inst) {
  std::vector<int32_t> order;
  std::vector<int> sizes;
  for (int i = 0; i < n_inst; ++i)
    if (std::find(sizes.begin(), sizes.end(), d[i].n) == sizes.end()) sizes.push_back(d[i].n);
  for (int n : sizes)
    for (int i = 0; i < n_inst; ++i)
      if (d[i].n == n) order.push_back(i);
  return order;
}

// Groups of beams of one grid size (d in group order).
std::vector<Group> make_groups(const ssfm_instance_desc* d, int n_inst) {
  std::vector<Group> g;
  for (int i = 0; i < n_inst; ++i) {
    if (g.empty() || g.back().n != d[i].n) {
      Group ng;
      ng.n = d[i].n;
      ng.beam0 = i;
      g.push_back(ng);
    }
    ++g.back().count;
  }
  return g;
}

using VariantMap = std::map<int, std::array<int, P_SLOTS>>;  // n -> variants

// Most partials any variant gives a beam of size n (one per wavefront).
int64_t max_parts(bool column, int n, bool fp64) {
  int64_t m = 0;
  for (int v = 0; v < plan_count(column, n); ++v) {
    PlanInfo pi;
    if (plan_info(column, n, v, fp64, &pi)) m = std::max<int64_t>(m, int64_t(n / pi.lines) * pi.waves);
  }
  return m;
}

// Builds groups, partial offsets and the layout (d in group order).  Pure
// host computation.
int plan_layout(const ssfm_instance_desc* d, int n_inst, int precision, int64_t max_steps,
                int32_t ckpt_every, int32_t stored_segments, const VariantMap* variants,
                std::vector<Group>* groups_out, std::vector<int32_t>* begins_out, Layout* L) {
  const bool fp64 = precision == SSFM_FP64;
  const size_t el = fp64 ? 16 : 8;
  const size_t rel = el / 2;
  std::vector<Group> groups = make_groups(d, n_inst);
  std::vector<int32_t> begins(size_t(P_SLOTS) * (n_inst + 1), 0);
  int64_t fill[P_SLOTS] = {0, 0, 0, 0};
  int64_t toff = 0, nr_max = 0, nc_max = 0;
  for (auto& g : groups) {
    g.var[P_ROW] = plan_default(false, g.n, fp64);
    g.var[P_COL] = plan_default(true, g.n, fp64);
    if (variants) {
      auto it = variants->find(g.n);
      if (it != variants->end()) std::copy(it->second.begin(), it->second.end(), g.var);
    }
    for (int s = 0; s < P_SLOTS; ++s) {
      PlanInfo pi;
      if (!plan_info(s & 1, g.n, g.variant(s), fp64, &pi))
        return fail(SSFM_EUNSUPPORTED, "no kernel plan for n=%d", g.n);
      g.lines[s] = pi.lines;
      g.part0[s] = int32_t(fill[s]);
      for (int b = g.beam0; b < g.beam0 + g.count; ++b) {
        begins[size_t(s) * (n_inst + 1) + b] = int32_t(fill[s]);
        fill[s] += int64_t(g.n / pi.lines) * pi.waves;
      }
    }
    g.tw = toff;
    toff += int64_t(P_SLOTS) * g.n;
    g.prop = toff;
    toff += int64_t(g.count) * T_COUNT * g.n;
    // partial-sum arrays are sized for the variant with the most of them
    nr_max += g.count * max_parts(false, g.n, fp64);
    nc_max += g.count * max_parts(true, g.n, fp64);
  }
  for (int s = 0; s < P_SLOTS; ++s)
    begins[size_t(s) * (n_inst + 1) + n_inst] = int32_t(fill[s]);
  Layout l{};
  int64_t fe = 0, se = 0, nsteps = 0, subh_doubles = 0;
  int max_n = 0;
  for (int b = 0; b < n_inst; ++b) {
    fe += int64_t(d[b].n) * d[b].n;
    max_n = std::max(max_n, d[b].n);
    if (d[b].terms & SSFM_TURB) {
      se += int64_t(d[b].n_screens) * d[b].n * d[b].n;
      nsteps += d[b].n_screens;
      subh_doubles += subharmonic_region_doubles(d[b].n, (d[b].n_screens + 1) / 2);
    }
  }
  l.field_elems = fe;
  l.table_elems = toff;
  l.screen_elems = se;
  l.n_steps_total = nsteps;
  l.max_n = max_n;
  l.part_stride = std::max(nr_max, nc_max);
  l.theta_row_parts = nr_max;
  l.theta_col_parts = nc_max;
  if (max_steps > 0) {
    const int64_t m = std::max<int64_t>(1, ckpt_every);
    const int64_t seg = std::min<int64_t>(m, max_steps);
    l.n_ckpt = (max_steps + seg - 1) / seg;
    l.n_stack = seg - 1;
    if (l.n_ckpt == 1) {
      l.n_banks = 0;  // a single segment is always kept whole
      l.n_kept = 1;
    } else {
      l.n_kept = std::min<int64_t>(stored_segments, l.n_ckpt);
      l.n_banks = std::min<int64_t>(2, l.n_ckpt - l.n_kept);
    }
  }
  l.diag_cap = std::max<int64_t>(max_steps, 4096);
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align_up(off + std::max<size_t>(bytes, 1));
    return o;
  };
  l.inst = take(sizeof(InstDev) * n_inst);
  l.steps = take(sizeof(int64_t) * std::max<int64_t>(nsteps, 1));
  l.begins = take(sizeof(int32_t) * P_SLOTS * (n_inst + 1));
  l.tables = take(el * toff);
  l.S = take(el * fe);
  l.Wk = take(el * fe);
  // (with more than one segment the recompute of the next segment runs
  // beside the adjoint of the current one, in its own bank of segment
  // slots; both work in place)
  l.Lam = take(max_steps > 0 ? el * fe : 0);
  l.ckpt = take(el * fe * l.n_ckpt);
  l.stack = take(el * fe * l.n_stack * (l.n_banks + l.n_kept));
  l.screens = take(rel * se);
  l.stage = take(16 * size_t(max_n) * max_n);
  l.diag = take(sizeof(double) * 2 * l.diag_cap * n_inst);
  // the accumulators live within one backward: in the staging area where they
  // fit it (all but large batches)
  const size_t theta_bytes = sizeof(double) * 8 * size_t(nr_max + nc_max);
  const size_t stage_bytes = 16 * size_t(max_n) * max_n;
  l.theta_rows = theta_bytes <= stage_bytes ? l.stage : take(theta_bytes);
  l.theta_cols = l.theta_rows + sizeof(double) * 8 * nr_max;
  const size_t step_bytes = sizeof(double) * 2 * size_t(l.part_stride);
  l.fd_chunk = int(std::min<size_t>(kDiagChunk, std::max(theta_bytes, stage_bytes) / step_bytes));
  // a line of n points is at most n / 256 wavefronts, so that kDiagChunk steps
  // of partials take no more than half of a complex64 field
  if (l.fd_chunk < 1 || kDiagChunk * step_bytes > el * size_t(fe))
    return fail(SSFM_EUNSUPPORTED, "the work buffer cannot hold the power partials");
  l.theta_out = take(sizeof(double) * 8 * n_inst);
  l.seed_loss = take(sizeof(double) * (max_n + 1));
  l.seed_theta = take(sizeof(double) * 8 * max_n * n_inst);
  // 256 partials of a sum of squares, moment or hot-area count, then 256 x 5
  // measure-vector partials
  l.sumsq_part = take(sizeof(double) * 256 * 6);
  // subharmonic tables and coefficients of every turbulent beam, its beam list
  l.subh = take(sizeof(double) * size_t(subh_doubles));
  l.subh_beams = take(sizeof(SubBeam) * n_inst);
  l.total = off;
  if (groups_out) *groups_out = groups;
  if (begins_out) *begins_out = begins;
  *L = l;
  return SSFM_OK;
}

// Twiddles of a radix plan in the order its stages read them (see
// fft_core.hpp): exp(-2 pi i r k / (NS R)) in FP64, rounded to the working
// precision; n entries, the last R0 unused.
void stage_twiddles(int n, const int* radices, std::vector<double>* out) {
  out->assign(2 * size_t(n), 0.0);
  const int r0 = radices[0];
  int ns = r0;
  for (int i = 1; radices[i] != 0; ++i) {
    const int rad = radices[i], step = n / (ns * rad);
    for (int r = 1; r < rad; ++r)
      for (int k = 0; k < ns; ++k) {
        const double a = 2.0 * M_PI * double(int64_t(r) * k * step) / double(n);
        const size_t at = size_t(ns - r0) + size_t(r - 1) * ns + k;
        (*out)[2 * at] = std::cos(a);
        (*out)[2 * at + 1] = -std::sin(a);
      }
    ns *= rad;
  }
}

// exp(-i k_m^2 dz / 2k0) / n, phase reduced modulo 2 pi in FP64.
void propagator(const ssfm_instance_desc& d, std::vector<double>* out) {
  const int n = d.n;
  const double k0 = 2.0 * M_PI / d.wavelength;
  out->resize(2 * size_t(n));
  for (int m = 0; m < n; ++m) {
    const int ms = (m <= n / 2) ? m : m - n;
    const double k = 2.0 * M_PI * double(ms) / d.length;
    double ph = std::fmod(k * k * d.dz / (2.0 * k0), 2.0 * M_PI);
    (*out)[2 * m] = std::cos(ph) / n;
    (*out)[2 * m + 1] = -std::sin(ph) / n;
  }
}

template <typename R>
void append_table(std::vector<unsigned char>* blob, const std::vector<double>& v) {
  const size_t n = v.size();
  const size_t o = blob->size();
  blob->resize(o + n * sizeof(R));
  R* p = reinterpret_cast<R*>(blob->data() + o);
  for (size_t i = 0; i < n; ++i) p[i] = R(v[i]);
}

int check_ctx(ssfm_ctx* c) {
  if (!c) return fail(SSFM_EINVAL, "ctx is NULL");
  return SSFM_OK;
}

// Maps the caller's instance to its position among the beams.
int check_inst(ssfm_ctx* c, int32_t& i) {
  if (int r = check_ctx(c)) return r;
  if (i < 0 || i >= int32_t(c->desc.size()))
    return fail(SSFM_EINVAL, "instance %d out of range [0, %zu)", i, c->desc.size());
  i = c->slot[i];
  return SSFM_OK;
}

// Forget a recorded march, its cotangents and gradients (the fields or
// parameters it was recorded with have changed).
void drop_record(ssfm_ctx* c) {
  c->rec_valid = false;
  c->seeded = false;
  c->grads_valid = false;
  c->seeded_beam.assign(c->desc.size(), 0);
}

// Fields and parameters are set outside captures: the host's counts and its
// copy of the beam table change with the device's, at the call.
int not_captured(ssfm_ctx* c) {
  hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
  if (hipStreamIsCapturing(c->stream, &st) != hipSuccess) (void)hipGetLastError();
  if (st != hipStreamCaptureStatusNone)
    return fail(SSFM_EHIP, "fields and parameters cannot be set while the stream is captured");
  return SSFM_OK;
}

// Beam table entries [b0, b1) to the device, now and in order on the stream:
// whatever is launched or captured after this reads them from the table, and
// a captured read keeps no copy of its own.  By value: the host table may
// change right after, and nothing waits (12 beams of 256^2, fields and
// parameters set, marched, compared: 1300 us with a copy and a wait for each
// change, now 680).
int upload_inst(ssfm_ctx* c, size_t b0, size_t b1) {
  if (int r = not_captured(c)) return r;
  HIP_TRY(launch_put<InstDev>(&c->inst[b0], int(b1 - b0), c->at<InstDev>(c->L.inst) + b0,
                              c->stream));
  return SSFM_OK;
}

// ---------------------------------------------------------------- passes
template <typename R>
PassArgs<R> base_args(ssfm_ctx* c) {
  PassArgs<R> a{};
  a.inst = c->at<InstDev>(c->L.inst);
  a.tables = c->ws + c->L.tables;
  a.screens = c->at<R>(c->L.screens);
  a.screen_steps = c->at<int64_t>(c->L.steps);
  a.step = -1;
  a.precise = c->precise ? 1 : 0;
  return a;
}

// Whether a beam of the group has a turbulence screen after context step
// `step`, so that the passes of the other steps do not look for one.  Without
// the library's own graphs any turbulent beam counts: a caller may capture
// these passes and replay them after setting fields at other steps.
bool group_has_plane(const ssfm_ctx* c, const Group& g, int64_t step) {
  if (step < 0) return false;
  for (int b = g.beam0; b < g.beam0 + g.count; ++b) {
    const InstDev& in = c->inst[b];
    if (!(in.terms & SSFM_TURB) || in.n_screens <= 0) continue;
    if (!c->use_graphs) return true;
    const auto first = c->screen_steps.begin() + in.steps_off;
    if (std::binary_search(first, first + in.n_screens, step - in.step_base)) return true;
  }
  return false;
}

// The size groups [g0, g1) and the stream that their passes go to.
struct Chain {
  size_t g0, g1;
  hipStream_t st;
};

Chain whole(ssfm_ctx* c, hipStream_t st = nullptr) {
  return {0, c->groups.size(), st ? st : c->stream};
}

// Runs body(chain) for chains that cover every size group.  Beams never
// wait for one another, so each group marches on its own stream (group 0 on
// the context's), forked and joined once around the whole run of passes: a
// group of few small beams fills a fraction of the chip, and joining the
// groups after every pass kept each step as long as its slowest launch plus
// two event hops (11 beams of 256^2 to
// 1024^2, 24 steps: 2060 us; as chains 1650).
// split = false, or a context without the streams: one chain of all groups.
template <typename F>
int each_chain(ssfm_ctx* c, bool split, F body) {
  const size_t ng = c->groups.size();
  if (!split || ng < 2 || c->gstream.size() + 1 < ng) return body(whole(c));
  HIP_TRY(hipEventRecord(c->gfork, c->stream));
  for (size_t g = 1; g < ng; ++g) HIP_TRY(hipStreamWaitEvent(c->gstream[g - 1], c->gfork, 0));
  int r = SSFM_OK;
  for (size_t g = 0; g < ng && r == SSFM_OK; ++g)
    r = body(Chain{g, g + 1, g > 0 ? c->gstream[g - 1] : c->stream});
  // joined on every path: the streams carry no work past the call
  for (size_t g = 1; g < ng; ++g) {
    HIP_TRY(hipEventRecord(c->gjoin[g - 1], c->gstream[g - 1]));
    HIP_TRY(hipStreamWaitEvent(c->stream, c->gjoin[g - 1], 0));
  }
  return r;
}

// One pass over the beams of a chain: one launch per grid-size group, in
// sequence.
template <typename R>
int run_pass(ssfm_ctx* c, int kind, PassArgs<R> a, const Chain& ch, int table = T_PROP,
             const hipEvent_t* ev = nullptr) {
  const bool col = is_col_kind(kind);
  const bool adj = kind == ROW_ADJ || kind == COL_ADJ;
  const int slot = (adj ? P_ROW_ADJ : P_ROW) + (col ? 1 : 0);
  const int32_t flags = a.flags;
  const bool screen = (adj || kind == ROW_FWD || kind == COL_FWD) && (flags & PASS_SCREEN);
  for (size_t gi = ch.g0; gi < ch.g1; ++gi) {
    const Group& g = c->groups[gi];
    a.off0 = c->inst[g.beam0].off;
    a.prop0 = g.prop + int64_t(table) * g.n;
    a.prop_stride = T_COUNT * g.n;
    a.tw = g.tw + int64_t(slot) * g.n;
    a.beam0 = g.beam0;
    a.part0 = g.part0[slot];
    a.n_tiles = g.count * (g.n / g.lines[slot]);
    a.flags = flags | ((screen && group_has_plane(c, g, a.step)) ? PASS_PLANE : 0);
    const LaunchEv le = ev ? LaunchEv{ev[2 * gi], ev[2 * gi + 1]} : LaunchEv{nullptr, nullptr};
    HIP_TRY(launch_pass<R>(kind, g.n, g.variant(slot), a, ch.st, ev ? &le : nullptr));
  }
  return SSFM_OK;
}

// Power partials of a chunk's step `slot` (see Layout).
double* power_parts(ssfm_ctx* c, int slot) {
  return c->at<double>(c->fd ? c->L.theta_rows : c->L.Wk) + size_t(slot) * 2 * c->L.part_stride;
}

// Power and peak of `steps` steps from context step `step0`, for the beams of
// a chain.
int finalize_diag(ssfm_ctx* c, const int32_t* begin_even, const int32_t* begin_odd, int steps,
                  int64_t step0, const Chain& ch) {
  const int b0 = c->groups[ch.g0].beam0;
  const Group& last = c->groups[ch.g1 - 1];
  HIP_TRY(launch_diag_finalize(power_parts(c, 0), c->L.part_stride, begin_even,
                               begin_odd, b0, last.beam0 + last.count - b0, steps,
                               c->at<double>(c->L.diag), step0, c->L.diag_cap, ch.st));
  return SSFM_OK;
}

// A timing sample (a start/stop pair per size group) from the pool; false
// if none could be made.
bool take_sample(ssfm_ctx* c, ssfm_ctx::PassSample* ps) {
  const size_t need = 2 * c->groups.size();
  if (!c->free_samples.empty()) {
    *ps = std::move(c->free_samples.back());
    c->free_samples.pop_back();
    if (ps->ev.size() == need) return true;
    for (auto x : ps->ev) (void)hipEventDestroy(x);
  }
  ps->ev.assign(need, nullptr);
  for (auto& x : ps->ev)
    if (hipEventCreate(&x) != hipSuccess) {
      for (auto y : ps->ev)
        if (y) (void)hipEventDestroy(y);
      ps->ev.clear();
      (void)hipGetLastError();  // timing is best effort: the march proceeds unsampled
      return false;
    }
  return true;
}

void clear_graphs(ssfm_ctx* c) {
  for (auto& kv : c->graphs) (void)hipGraphExecDestroy(kv.second);
  c->graphs.clear();
}

// Axis along which context step `step` diffracts first (false: rows) and
// second.  Tied to the step index, so a march cut anywhere, a recomputed
// segment and the adjoint all see the same fields.
bool first_axis_col(int64_t step) { return (step & 1) != 0; }
bool second_axis_col(int64_t step) { return (step & 1) == 0; }

// Where a march of n steps reads and writes: V_0 comes from src, the
// half-diffracted field lives in cur (whole lines per workgroup: in place),
// V_n goes to dst unless that is null, and rec(i) (0 <= i <= n), where it
// gives a buffer, gets V_i.  Recorded fields lie line by line along the axis
// of the passes that use them, which is the first axis of their step: the
// columns of one take contiguous stores and loads (kept: src is recorded).
struct MarchBuffers {
  const void* src;
  void *cur, *dst;
  bool kept;
};

// The passes that end steps i0 <= i < i1 of a march of n steps from step0 (for
// i0 = 0 also, with opens, the pass that opens it).  pend(i): step whose
// screen acts before step i diffracts (-1: none).  part: whether to reduce
// the power and peak of each step.  open, end: timing events of the opening
// and of the (single) ending pass.
template <typename R, typename Pend, typename Rec>
int enqueue_march(ssfm_ctx* c, int64_t n, int64_t step0, int64_t i0, int64_t i1, bool opens,
                  const MarchBuffers& m, Pend pend, Rec rec, bool part, const Chain& ch,
                  const ssfm_ctx::PassSample* open, const ssfm_ctx::PassSample* end) {
  const int32_t raw = c->strang ? PASS_RAW : 0;  // Strang: |U|^2 = |V|^2 summed as it is
  if (i0 == 0 && opens) {
    PassArgs<R> a = base_args<R>(c);
    a.src = m.src;
    a.dst = m.cur;
    a.rec = rec(0);
    a.step = pend(0);
    a.flags = PASS_OP2 | (a.step >= 0 ? PASS_SCREEN : 0) | (m.kept ? PASS_SRC_KEPT : 0);
    const bool col = first_axis_col(step0);
    if (int r = run_pass<R>(c, col ? COL_FWD : ROW_FWD, a, ch, T_PROP,
                            open ? open->ev.data() : nullptr))
      return r;
  }
  int64_t chunk_start = step0 + i0;
  for (int64_t i = i0; i < i1; ++i) {
    const int slot = int((i - i0) % kDiagChunk);
    const bool last = i == n - 1;
    PassArgs<R> a = base_args<R>(c);
    a.src = m.cur;
    a.dst = last ? m.dst : m.cur;
    if (part) a.part = power_parts(c, slot);
    a.flags = PASS_OP1 | raw;
    a.rec = rec(i + 1);
    if (!last) {
      a.step = pend(i + 1);
      a.flags |= PASS_SCREEN | PASS_OP2;
    }
    const bool col = second_axis_col(step0 + i);
    if (int r = run_pass<R>(c, col ? COL_FWD : ROW_FWD, a, ch, T_PROP,
                            end ? end->ev.data() : nullptr))
      return r;
    if (part && (slot == kDiagChunk - 1 || i == i1 - 1)) {
      const int32_t* begins = c->at<int32_t>(c->L.begins);
      const size_t nb = c->desc.size() + 1;
      if (int r = finalize_diag(c, begins + P_COL * nb, begins + P_ROW * nb, slot + 1, chunk_start,
                                ch))
        return r;
      chunk_start = step0 + i + 1;
    }
  }
  return SSFM_OK;
}

// Runs enqueue(chain, i0, i1, opens) for the passes that end steps i0 <= i <
// i1, as chains.  Before a sampled pass (end) the chains are joined also
// after the opening pass: the pass starts in all size groups together, so
// that its span over them is its own.
template <typename F>
int march_chains(ssfm_ctx* c, int64_t i0, int64_t i1, const ssfm_ctx::PassSample* end, F enqueue) {
  const bool apart = end && i0 == 0;
  if (apart)
    if (int r = each_chain(c, true, [&](const Chain& ch) { return enqueue(ch, 0, 0, true); }))
      return r;
  return each_chain(c, true, [&](const Chain& ch) { return enqueue(ch, i0, i1, !apart); });
}

// Steps i0 <= i < i1 of an n-step plain forward march from step0 (pending0:
// the state holds V with the screen of step0 - 1 still to apply), in place
// on the state.  Lie: the screen of the previous step acts before step i;
// Strang: the state is V = L(dz/2) U and the step's own screen does.
template <typename R>
int enqueue_propagate(ssfm_ctx* c, int64_t n, int64_t step0, bool pending0, int64_t i0,
                      int64_t i1, const ssfm_ctx::PassSample* open,
                      const ssfm_ctx::PassSample* end) {
  return march_chains(c, i0, i1, end, [&](const Chain& ch, int64_t k0, int64_t k1, bool opens) {
    void* S = c->field(c->L.S);
    auto pend = [&](int64_t i) {
      return c->strang ? step0 + i : (i == 0 && !pending0) ? -1 : step0 + i - 1;
    };
    return enqueue_march<R>(
        c, n, step0, k0, k1, opens, MarchBuffers{S, S, S, false}, pend,
        [](int64_t) -> void* { return nullptr; }, true, ch, open, end);
  });
}

// Steps i0 <= i < i1 of a finite-difference march from step step0 + i0, on
// S (U) and Wk (the row-transformed right-hand side).  The first row pass
// forms U + (dz/2) G(|U|^2) U from S; each of the fd_iters iterations is a
// column pass (the solve) and a row pass (Ubar, then the next right-hand
// side); the last row pass of a step writes U+ = 2 Ubar - U and its power
// partials and, unless the range ends, starts the next step.
template <typename R>
int enqueue_fd(ssfm_ctx* c, int64_t step0, int64_t i0, int64_t i1, const Chain& ch) {
  PassArgs<R> a = base_args<R>(c);
  a.state = c->field(c->L.S);
  a.src = c->field(c->L.S);
  a.dst = c->field(c->L.Wk);
  a.flags = 0;
  if (int r = run_pass<R>(c, ROW_FD, a, ch)) return r;
  PassArgs<R> col = base_args<R>(c);
  col.src = c->field(c->L.Wk);
  col.dst = c->field(c->L.Wk);
  a.src = c->field(c->L.Wk);
  int64_t chunk_start = step0 + i0;
  for (int64_t i = i0; i < i1; ++i) {
    const int slot = int((i - i0) % c->L.fd_chunk);
    for (int k = 1; k <= c->fd_iters; ++k) {
      if (int r = run_pass<R>(c, COL_FD, col, ch, T_FD)) return r;
      const bool fin = (k == c->fd_iters);
      a.flags = FD_SPECTRAL | (fin ? FD_FINISH : 0) | ((fin && i == i1 - 1) ? FD_LAST : 0);
      a.part = fin ? power_parts(c, slot) : nullptr;
      if (int r = run_pass<R>(c, ROW_FD, a, ch)) return r;
    }
    if (slot == c->L.fd_chunk - 1 || i == i1 - 1) {
      const int32_t* rows = c->at<int32_t>(c->L.begins) + P_ROW * (c->desc.size() + 1);
      if (int r = finalize_diag(c, rows, rows, slot + 1, chunk_start, ch)) return r;
      chunk_start = step0 + i + 1;
    }
  }
  return SSFM_OK;
}

// Runs `body` directly or through a cached graph keyed by (kind, a, b, i0, i1).
template <typename F>
int maybe_graph(ssfm_ctx* c, int kind, int64_t a, int64_t b, int64_t i0, int64_t i1, F body) {
  if (!c->use_graphs) return body();
  std::vector<int64_t> bases;
  for (const InstDev& in : c->inst)
    if ((in.terms & SSFM_TURB) && in.n_screens > 0) bases.push_back(in.step_base);
  const ssfm_ctx::GraphKey key(kind, a, b, i0, i1, std::move(bases));
  auto it = c->graphs.find(key);
  if (it == c->graphs.end()) {
    // graphs are specific to their first step; a caller marching in many
    // small chunks would grow the cache without bound, so past a limit it
    // is emptied (after the stream drains, so no cached graph still runs)
    constexpr size_t kMaxGraphs = 128;
    if (c->graphs.size() >= kMaxGraphs) {
      HIP_TRY(hipStreamSynchronize(c->stream));
      clear_graphs(c);
    }
    hipStream_t cap;
    HIP_TRY(hipStreamCreateWithFlags(&cap, hipStreamNonBlocking));
    hipStream_t saved = c->stream;
    c->stream = cap;
    hipError_t e = hipStreamBeginCapture(cap, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) {
      c->stream = saved;
      (void)hipStreamDestroy(cap);
      return fail(SSFM_EHIP, "hipStreamBeginCapture: %s", hipGetErrorString(e));
    }
    int r = body();
    hipGraph_t graph = nullptr;
    hipError_t e2 = hipStreamEndCapture(cap, &graph);
    c->stream = saved;
    (void)hipStreamDestroy(cap);
    if (r) {
      if (graph) (void)hipGraphDestroy(graph);
      return r;
    }
    if (e2 != hipSuccess) return fail(SSFM_EHIP, "hipStreamEndCapture: %s", hipGetErrorString(e2));
    hipGraphExec_t exec = nullptr;
    hipError_t e3 = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    if (e3 != hipSuccess) return fail(SSFM_EHIP, "hipGraphInstantiate: %s", hipGetErrorString(e3));
    it = c->graphs.emplace(key, exec).first;
  }
  HIP_TRY(hipGraphLaunch(it->second, c->stream));
  return SSFM_OK;
}

// Steps [0, n) of a forward march from step0 through seg(i0, i1, open, end):
// in captured graphs keyed by (kind, key, n, i0, i1) between the sampled
// passes, each of those launched directly with its timing events: the pass
// that ends a sampled step and a neighbour along the other axis (the next
// pass, else the one before).
template <typename Seg>
int run_forward(ssfm_ctx* c, int kind, int64_t key, int64_t n, int64_t step0, Seg seg) {
  for (auto& e : c->samples) c->free_samples.push_back(std::move(e));
  c->samples.clear();
  c->n_samples = 0;
  int64_t i = 0;
  auto graph_to = [&](int64_t k) -> int {
    if (k <= i) return SSFM_OK;
    const int64_t i0 = i;
    i = k;
    return maybe_graph(c, kind, key, n, i0, k, [&] { return seg(i0, k, nullptr, nullptr); });
  };
  auto timed = [&](int64_t k, bool with_open) -> int {
    ssfm_ctx::PassSample open, end;
    const bool have_open = with_open && take_sample(c, &open);
    const bool have_end = take_sample(c, &end);
    open.col = first_axis_col(step0 + k);
    end.col = second_axis_col(step0 + k);
    int r = seg(k, k + 1, have_open ? &open : nullptr, have_end ? &end : nullptr);
    if (have_open) c->samples.push_back(std::move(open));
    if (have_end) c->samples.push_back(std::move(end));
    i = k + 1;
    return r;
  };
  const int64_t m = c->timing_every;
  if (m > 0) {
    int64_t first = (m / 2 - step0 % m) % m;  // first i with (step0 + i) % m == m / 2
    if (first < 0) first += m;
    for (int64_t k = first; k < n; k += m) {
      const bool pair_before = k + 1 == n && k - 1 >= i;
      if (int r = graph_to(pair_before ? k - 1 : k)) return r;
      if (pair_before)
        if (int r = timed(k - 1, false)) return r;
      if (int r = timed(k, n == 1)) return r;
      ++c->n_samples;
      if (m > 1 && k + 1 < n)
        if (int r = timed(k + 1, false)) return r;
    }
  }
  return graph_to(n);
}

template <typename R>
int do_propagate(ssfm_ctx* c, int64_t n) {
  const int64_t step0 = c->step;
  const bool pend = c->pending;
  if (c->fd) {
    // one graph per (start step, length): the diagnostics ring slots depend
    // on the absolute step
    int r = maybe_graph(c, 3, step0, n, 0, n, [&] {
      return each_chain(c, true,
                        [&](const Chain& ch) { return enqueue_fd<R>(c, step0, 0, n, ch); });
    });
    if (r) return r;
    c->step += n;
    c->pending = false;
    c->diag_valid = std::min<int64_t>(n, c->L.diag_cap);
    c->rec_valid = false;
    c->seeded = false;
    c->seeded_beam.assign(c->desc.size(), 0);
    return SSFM_OK;
  }
  int r = run_forward(c, 0, step0 * 2 + (pend ? 1 : 0), n, step0,
                      [&](int64_t i0, int64_t i1, const ssfm_ctx::PassSample* open,
                          const ssfm_ctx::PassSample* end) {
                        return enqueue_propagate<R>(c, n, step0, pend, i0, i1, open, end);
                      });
  if (r) return r;
  c->step += n;
  c->pending = !c->strang;
  c->diag_valid = std::min<int64_t>(n, c->L.diag_cap);
  c->rec_valid = false;
  c->seeded = false;
  c->seeded_beam.assign(c->desc.size(), 0);
  return SSFM_OK;
}

// Half-step diffraction L(+-dz/2) of every beam: S -> Wk through the pass
// kernels with the half-step tables (no screen).
template <typename R>
int half_steps(ssfm_ctx* c, bool forward) {
  HIP_TRY(launch_copy<R>(c->field(c->L.S), c->field(c->L.Wk), c->L.field_elems, c->stream));
  PassArgs<R> a = base_args<R>(c);
  a.src = c->field(c->L.Wk);
  a.dst = c->field(c->L.Wk);
  a.flags = PASS_OP2;
  return each_chain(c, true, [&](const Chain& ch) {
    if (int r = run_pass<R>(c, ROW_FWD, a, ch, forward ? T_HALF : T_BACK)) return r;
    return run_pass<R>(c, COL_FWD, a, ch, forward ? T_HALF : T_BACK);
  });
}

// Lam <- L(+-dz/2) Lam in place (the half-step tables, no screen), for the
// beams of a chain.
template <typename R>
int half_step_lam(ssfm_ctx* c, bool forward, const Chain& ch) {
  PassArgs<R> a = base_args<R>(c);
  a.src = c->field(c->L.Lam);
  a.dst = c->field(c->L.Lam);
  a.flags = PASS_OP2;
  if (int r = run_pass<R>(c, ROW_FWD, a, ch, forward ? T_HALF : T_BACK)) return r;
  return run_pass<R>(c, COL_FWD, a, ch, forward ? T_HALF : T_BACK);
}

// Apply the pending screen in place (state becomes U_n).
template <typename R>
int flush_pending(ssfm_ctx* c) {
  if (!c->pending) return SSFM_OK;
  HIP_TRY(launch_flush<R>(c->field(c->L.S), c->at<InstDev>(c->L.inst), int(c->desc.size()),
                          c->L.max_n, c->at<R>(c->L.screens), c->at<int64_t>(c->L.steps),
                          c->step - 1, c->stream));
  c->pending = false;
  return SSFM_OK;
}

// Screen applied on load by step `step` of a record starting at step0: Lie
// the previous step's (none for the first), Strang the step's own.
int64_t rec_pending(const ssfm_ctx* c, int64_t step0, int64_t step) {
  if (c->strang) return step;
  return (step == step0) ? -1 : step - 1;
}

// Segments of a record of n steps.  Segment k covers s_{kM} .. s_{kM+M-1}:
// s_{kM} is checkpoint k, the others sit in segment slots (a region of
// n_stack fields).  Segments k >= first_kept are written whole by the
// forward record, each in a region of its own after the recompute banks;
// the backward recomputes the others from their checkpoints, alternating
// between banks 0 and 1.  A single-segment record is kept whole in region 0.
struct Segments {
  int64_t M, n_seg, first_kept, banks;
  int64_t region(int64_t k) const { return k >= first_kept ? banks + (k - first_kept) : k % 2; }
  bool recomputed(int64_t k) const { return k < first_kept; }
};

Segments rec_segments(const ssfm_ctx* c, int64_t n) {
  Segments g;
  g.M = std::min<int64_t>(std::max<int32_t>(c->ckpt_every, 1), n);
  g.n_seg = (n + g.M - 1) / g.M;
  if (g.n_seg == 1) {
    g.first_kept = 0;
    g.banks = 0;
  } else {
    // never more kept segments than the layout has regions for (a record
    // shorter than max_steps has no more segments than the layout)
    g.first_kept = g.n_seg - std::min<int64_t>(c->L.n_kept, g.n_seg);
    g.banks = c->L.n_banks;
  }
  return g;
}

// Where a record of n steps keeps s_i = V_i (0 <= i < n; null: not kept),
// line by line along step i's first axis.
void* rec_slot(ssfm_ctx* c, const Segments& g, int64_t i) {
  if (i % g.M == 0) return c->field(c->L.ckpt, i / g.M);
  const int64_t k = i / g.M;
  if (!g.recomputed(k)) return c->field(c->L.stack, g.region(k) * c->L.n_stack + i % g.M - 1);
  return nullptr;
}

// Steps i0 <= i < i1 of an n-step record from step0, in place on the state;
// the passes write the fields that are kept as they come by.
template <typename R>
int enqueue_record(ssfm_ctx* c, int64_t n, int64_t step0, int64_t i0, int64_t i1,
                   const ssfm_ctx::PassSample* open, const ssfm_ctx::PassSample* end) {
  const Segments g = rec_segments(c, n);
  void* S = c->field(c->L.S);
  return march_chains(c, i0, i1, end, [&](const Chain& ch, int64_t k0, int64_t k1, bool opens) {
    return enqueue_march<R>(
        c, n, step0, k0, k1, opens, MarchBuffers{S, S, S, false},
        [&](int64_t i) { return rec_pending(c, step0, step0 + i); },
        [&](int64_t i) { return i < n ? rec_slot(c, g, i) : nullptr; }, true, ch, open, end);
  });
}

template <typename R>
int do_record(ssfm_ctx* c, int64_t n) {
  if (c->max_steps <= 0 || n > c->max_steps)
    return fail(SSFM_EINVAL, "record of %lld steps exceeds max_steps %lld", (long long)n,
                (long long)c->max_steps);
  if (int r = flush_pending<R>(c)) return r;
  const int64_t step0 = c->step;
  int r = run_forward(c, 1, step0, n, step0,
                      [&](int64_t i0, int64_t i1, const ssfm_ctx::PassSample* open,
                          const ssfm_ctx::PassSample* end) {
                        return enqueue_record<R>(c, n, step0, i0, i1, open, end);
                      });
  if (r) return r;
  c->step += n;
  c->pending = !c->strang;
  c->diag_valid = std::min<int64_t>(n, c->L.diag_cap);
  c->rec_steps = n;
  c->rec_step0 = step0;
  drop_record(c);
  c->rec_valid = true;
  return SSFM_OK;
}

// Backward over the recorded march, segment by segment from the last.  A
// segment the forward did not keep whole is recomputed from its checkpoint
// (into the other bank, through the work buffer): segment k-1 after the
// adjoint of segment k on the same stream, or (overlap_recompute) on the
// auxiliary stream while the adjoint of segment k runs on the main stream,
// the two joining before the adjoint of segment k-1.  The size groups sweep
// independently: through the whole backward, or with the overlap through
// the adjoint of each segment (the recompute takes them in sequence on its
// stream: a stream capture must join every fork to its primary stream, and a
// fork of a fork would be joined to the auxiliary one instead).
template <typename R>
int enqueue_backward(ssfm_ctx* c) {
  const int64_t n = c->rec_steps, step0 = c->rec_step0;
  const Segments g = rec_segments(c, n);
  const int64_t M = g.M, n_seg = g.n_seg;
  const int64_t bank = c->L.n_stack;
  auto slot = [&](int64_t k, int64_t i) -> void* {  // slot i of segment k's region
    return c->field(c->L.stack, g.region(k) * bank + i);
  };
  auto sv = [&](int64_t k, int64_t i) -> void* {  // s_{kM+i}
    if (i == 0) return c->field(c->L.ckpt, k);
    return slot(k, i - 1);
  };
  // s_{kM+1} .. of segment k from its checkpoint: the work buffer, which
  // nothing else uses during the backward sweep, holds the half-diffracted
  // field
  auto recompute = [&](int64_t k, const Chain& ch) -> int {
    const int64_t s0 = k * M;
    const int64_t len = std::min<int64_t>(M, n - s0);
    if (len < 2) return SSFM_OK;
    return enqueue_march<R>(
        c, len - 1, step0 + s0, 0, len - 1, true,
        MarchBuffers{sv(k, 0), c->field(c->L.Wk), nullptr, true},
        [&](int64_t i) { return rec_pending(c, step0, step0 + s0 + i); },
        [&](int64_t i) { return i > 0 ? slot(k, i - 1) : nullptr; }, false, ch, nullptr,
        nullptr);
  };
  // the pass along one axis that ends adjoint step s + 1 and begins step s
  // (of the march's n; s = n opens the sweep), in place on the cotangent:
  // the adjoints of step s's first factor, of the screen before it (with
  // the stored V_s), and of the factor that precedes the screen
  auto adj_pass = [&](int64_t s, const void* v_s, const Chain& ch,
                      const ssfm_ctx::PassSample* ts) -> int {
    PassArgs<R> a = base_args<R>(c);
    a.src = c->field(c->L.Lam);
    a.dst = c->field(c->L.Lam);
    const bool col = (s == n) ? second_axis_col(step0 + n - 1) : first_axis_col(step0 + s);
    a.part = c->at<double>(col ? c->L.theta_cols : c->L.theta_rows);
    if (s < n) {
      a.flags = PASS_OP1;
      a.aux = v_s;
      a.step = rec_pending(c, step0, step0 + s);
      if (a.step >= 0) a.flags |= PASS_SCREEN;
    }
    if (s > 0) a.flags |= PASS_OP2;
    return run_pass<R>(c, col ? COL_ADJ : ROW_ADJ, a, ch, T_PROP,
                       ts ? ts->ev.data() : nullptr);
  };
  // a sampled pass: one sample of every group's events
  std::map<int64_t, size_t> sample_of;
  auto timed_adj_pass = [&](int64_t s, const void* v_s, const Chain& ch) -> int {
    auto it = sample_of.find(s);
    if (it == sample_of.end() && ch.g0 == 0) {
      ssfm_ctx::PassSample ps;
      if (take_sample(c, &ps)) {
        ps.col = (s == n) ? second_axis_col(step0 + n - 1) : first_axis_col(step0 + s);
        it = sample_of.emplace(s, c->adj_samples.size()).first;
        c->adj_samples.push_back(std::move(ps));
      }
    }
    return adj_pass(s, v_s, ch, it == sample_of.end() ? nullptr : &c->adj_samples[it->second]);
  };
  HIP_TRY(launch_fill_f64(c->at<double>(c->L.theta_rows), 8 * c->L.theta_row_parts, 0.0,
                          c->stream));
  HIP_TRY(launch_fill_f64(c->at<double>(c->L.theta_cols), 8 * c->L.theta_col_parts, 0.0,
                          c->stream));
  const int64_t every = c->timing_every;
  // Strang: the seed is the cotangent of U_N = L(-dz/2) V_N, so the march's
  // adjoint starts from L(dz/2) of it (the adjoint of the read-out)
  auto open = [&](const Chain& ch) -> int {
    if (c->strang)
      if (int r = half_step_lam<R>(c, true, ch)) return r;
    return g.recomputed(n_seg - 1) ? recompute(n_seg - 1, ch) : SSFM_OK;
  };
  auto first = [&](const Chain& ch) -> int {
    return (every > 0 && n == 1) ? timed_adj_pass(n, nullptr, ch)
                                 : adj_pass(n, nullptr, ch, nullptr);
  };
  // adjoint step i of segment k
  auto pass = [&](int64_t k, int64_t i, const Chain& ch) -> int {
    const int64_t s = k * M + i, len = std::min<int64_t>(M, n - k * M);
    // sampled steps of the first segment, and the pass after each (along
    // the other axis)
    const bool sampled = every > 0 && k == 0 && s % every == every / 2;
    const bool after = every > 0 && k == 0 && i < len - 1 && (s + 1) % every == every / 2;
    if (sampled && ch.g0 == 0) ++c->n_adj_samples;
    return (sampled || after) ? timed_adj_pass(s, sv(k, i), ch)
                              : adj_pass(s, sv(k, i), ch, nullptr);
  };
  auto segment = [&](int64_t k, const Chain& ch) -> int {
    for (int64_t i = std::min<int64_t>(M, n - k * M) - 1; i >= 0; --i)
      if (int r = pass(k, i, ch)) return r;
    return SSFM_OK;
  };
  // Strang: V_0 = L(dz/2) U_0, so dL/dU_0 = L(-dz/2) dL/dV_0
  auto close = [&](const Chain& ch) -> int {
    return c->strang ? half_step_lam<R>(c, false, ch) : SSFM_OK;
  };
  const bool overlap = c->overlap_recompute && g.first_kept > 0 && n_seg > 1;
  auto chains = [&](auto body) { return each_chain(c, true, body); };
  if (!overlap && every == 0) {
    const int r = chains([&](const Chain& ch) -> int {
      if (int q = open(ch)) return q;
      if (int q = first(ch)) return q;
      for (int64_t k = n_seg - 1; k >= 0; --k) {
        if (int q = segment(k, ch)) return q;
        if (k >= 1 && g.recomputed(k - 1))
          if (int q = recompute(k - 1, ch)) return q;
      }
      return close(ch);
    });
    if (r) return r;
  } else {
    // joined around the overlapped recompute, and around every pass of a
    // sampled segment: a sampled pass starts in all size groups together,
    // so that its span over them is its own
    const bool apart = every > 0;
    if (apart)
      if (int r = chains(open)) return r;
    if (int r = chains([&](const Chain& ch) -> int {
          if (!apart)
            if (int q = open(ch)) return q;
          return first(ch);
        }))
      return r;
    for (int64_t k = n_seg - 1; k >= 0; --k) {
      const bool rec_prev = k >= 1 && g.recomputed(k - 1);
      if (rec_prev && overlap) {
        HIP_TRY(hipEventRecord(c->ev_fork, c->stream));
        HIP_TRY(hipStreamWaitEvent(c->aux, c->ev_fork, 0));
        if (int r = recompute(k - 1, whole(c, c->aux))) return r;
        HIP_TRY(hipEventRecord(c->ev_join, c->aux));
      }
      if (every > 0 && k == 0) {
        for (int64_t i = std::min<int64_t>(M, n) - 1; i >= 0; --i)
          if (int r = chains([&](const Chain& ch) { return pass(0, i, ch); })) return r;
      } else {
        if (int r = chains([&](const Chain& ch) { return segment(k, ch); })) return r;
      }
      if (rec_prev && overlap) HIP_TRY(hipStreamWaitEvent(c->stream, c->ev_join, 0));
      if (rec_prev && !overlap)
        if (int r = chains([&](const Chain& ch) { return recompute(k - 1, ch); })) return r;
    }
    if (int r = chains(close)) return r;
  }
  const int32_t* begins = c->at<int32_t>(c->L.begins);
  const size_t nb = c->desc.size() + 1;
  HIP_TRY(launch_reduce_theta(c->at<double>(c->L.theta_rows), begins + P_ROW_ADJ * nb,
                              c->at<double>(c->L.theta_cols), begins + P_COL_ADJ * nb,
                              int(c->desc.size()), c->at<double>(c->L.theta_out), c->stream));
  return SSFM_OK;
}

template <typename R>
int do_backward(ssfm_ctx* c) {
  if (!c->rec_valid) return fail(SSFM_ESTATE, "backward needs a preceding ssfm_forward_record");
  if (!c->seeded) return fail(SSFM_ESTATE, "backward needs a cotangent (set_cotangent/fluence_loss)");
  for (auto& e : c->adj_samples) c->free_samples.push_back(std::move(e));
  c->adj_samples.clear();
  c->n_adj_samples = 0;
  // a beam without a cotangent contributes nothing to the loss: its
  // cotangent and its seed-step theta partials are zero (else the adjoint
  // would march whatever an earlier backward left there)
  for (size_t b = 0; b < c->desc.size(); ++b) {
    if (c->seeded_beam[b]) continue;
    const int64_t n2 = int64_t(c->inst[b].n) * c->inst[b].n;
    HIP_TRY(launch_fill_f64(reinterpret_cast<double*>(static_cast<char*>(c->field(c->L.Lam)) +
                                                      c->inst[b].off * c->el),
                            n2 * int64_t(c->el / 8), 0.0, c->stream));
    HIP_TRY(launch_fill_f64(c->at<double>(c->L.seed_theta) + size_t(b) * 8 * c->L.max_n,
                            8 * int64_t(c->inst[b].n), 0.0, c->stream));
  }
  // sampled timing launches the backward directly (its sampled passes
  // carry events on their own dispatches)
  int r = c->timing_every > 0 ? enqueue_backward<R>(c)
                              : maybe_graph(c, 2, c->rec_step0, c->rec_steps, 0, 0,
                                            [&] { return enqueue_backward<R>(c); });
  if (r) return r;
  c->grads_valid = true;
  return SSFM_OK;
}

// Seed (mode 0: loss; mode 1: external cotangent) for one beam.
template <typename R>
int do_seed(ssfm_ctx* c, int b, int mode, const double* target_dev, const double* g_dev) {
  const InstDev& in = c->inst[b];
  const ssfm_instance_desc& d = c->desc[b];
  const int64_t pend = c->step - 1;  // rec: the last recorded step's screen
  double* loss = c->at<double>(c->L.seed_loss);
  double* th = c->at<double>(c->L.seed_theta) + size_t(b) * 8 * c->L.max_n;
  if (mode == 0) {
    HIP_TRY(launch_sumsq(target_dev, int64_t(in.n) * in.n, c->at<double>(c->L.sumsq_part),
                         c->stream));
  }
  const double gs = (mode == 0) ? d.i_ref : std::sqrt(d.i_ref);
  const void* state = c->field(c->L.S);
  int64_t seed_pend = pend;
  if (c->strang) {
    // U_N = L(-dz/2) V_N into the work buffer; nothing pending
    seed_pend = -1;
    if (mode == 0) {
      if (int r = half_steps<R>(c, false)) return r;
      state = c->field(c->L.Wk);
    }
  }
  HIP_TRY(launch_seed<R>(mode, state, c->at<InstDev>(c->L.inst), b, in.n,
                         c->at<R>(c->L.screens), c->at<int64_t>(c->L.steps), seed_pend, target_dev,
                         c->at<double>(c->L.sumsq_part), g_dev, gs, c->field(c->L.Lam), loss, th,
                         in.n, c->stream));
  return SSFM_OK;
}


// The list of the beams' screen spectra to the device; the largest pair
// count and levels x n of the beams with subharmonics.  The subharmonic
// region is laid out over every turbulent beam in order.
int upload_spectra(ssfm_ctx* c, int* sub_pairs, int64_t* sub_table) {
  std::vector<SubBeam> list(c->desc.size(), SubBeam{});
  *sub_pairs = 0;
  *sub_table = 0;
  int64_t region_off = 0;
  for (size_t b = 0; b < c->desc.size(); ++b) {
    const ssfm_instance_desc& d = c->desc[b];
    if (!(d.terms & SSFM_TURB) || d.n_screens <= 0) continue;
    const ssfm_ctx::Spectrum& sp = c->spectrum[b];
    SubBeam& e = list[b];
    e.n = d.n;
    e.pairs = (d.n_screens + 1) / 2;
    e.k0 = uint32_t(d.seed & 0xffffffffu);
    e.k1 = uint32_t(d.seed >> 32);
    e.sp.kind = sp.kind;
    e.sp.tau = sp.tau;
    e.sp.band_q2 = band_q2(d.length, sp.kappa_h);
    e.sp.length = d.length;
    const double k0 = 2.0 * M_PI / d.wavelength;
    const bool step = sp.kind == SSFM_SPECTRUM_STEP;
    if (step) {
      e.amp0 = std::sqrt(sp.tau);
    } else if (d.cn2 > 0) {
      // sqrt(Phi(f)) df with Phi(f) = 0.023 r0^(-5/3) f^(-11/3), f = m / L,
      // df = 1 / L:  amplitude = sqrt(0.023) (L / r0)^(5/6) m^(-11/6)
      e.sp.r0 = std::pow(0.423 * k0 * k0 * d.cn2 * d.screen_dz, -0.6);
      e.amp0 = std::sqrt(0.023) * std::pow(d.length / e.sp.r0, 5.0 / 6.0);
    }
    e.tab_off = region_off;
    e.coef_off = region_off + 2 * int64_t(kMaxSubharmonicLevels) * d.n;
    region_off += subharmonic_region_doubles(d.n, e.pairs);
    if (sp.subharmonics == 0 || (!step && !(d.cn2 > 0))) continue;
    e.sp.levels = sp.subharmonics;
    *sub_pairs = std::max(*sub_pairs, e.pairs);
    *sub_table = std::max<int64_t>(*sub_table, int64_t(sp.subharmonics) * d.n);
  }
  HIP_TRY(launch_put<SubBeam>(list.data(), int(list.size()), c->at<SubBeam>(c->L.subh_beams),
                              c->stream));
  return SSFM_OK;
}

// Turbulence screens: per screen pair the row pass draws Philox/Box-Muller
// white noise shaped by the spectrum and transforms it, and the column pass
// ends the unscaled inverse DFT, adds the subharmonics and writes planes 2p
// and 2p+1.  The coefficients, means and axis tables of the subharmonics
// come up front for all beams and pairs; the size groups go independently.
// Seven screens with three levels on beams of 1024^2 to 256^2: 1045 us with
// the noise, the transforms and the subharmonics as passes of their own (a
// noise launch per beam and pair, 64 multiplies per point and level), with
// the same chains 703 us, now 540, of which 350 are the 28 read-outs.
template <typename R>
int do_gen_screens(ssfm_ctx* c) {
  int sub_pairs = 0;
  int64_t sub_table = 0;
  if (int r = upload_spectra(c, &sub_pairs, &sub_table)) return r;
  const SubBeam* spectra = c->at<SubBeam>(c->L.subh_beams);
  if (sub_pairs > 0)
    HIP_TRY(launch_subharmonic_setup(spectra, int(c->desc.size()), sub_pairs, sub_table,
                                     c->at<double>(c->L.subh), c->stream));
  return each_chain(c, true, [&](const Chain& ch) -> int {
    int pairs = 0;
    for (size_t g = ch.g0; g < ch.g1; ++g)
      for (int b = c->groups[g].beam0; b < c->groups[g].beam0 + c->groups[g].count; ++b)
        if (c->desc[b].terms & SSFM_TURB) pairs = std::max(pairs, (c->desc[b].n_screens + 1) / 2);
    for (int p = 0; p < pairs; ++p) {
      PassArgs<R> a = base_args<R>(c);
      a.aux = spectra;
      a.dst = c->field(c->L.Wk);
      a.pair = p;
      if (int r = run_pass<R>(c, ROW_INV, a, ch)) return r;
      a.src = c->field(c->L.Wk);
      a.state = c->at<double>(c->L.subh);
      a.planes_out = c->at<R>(c->L.screens);
      if (int r = run_pass<R>(c, COL_INV, a, ch)) return r;
    }
    return SSFM_OK;
  });
}

// Host twiddle tables by radix plan (whose product is the size): most passes
// of a size share one.
using TwiddleTables = std::map<std::vector<int>, std::vector<unsigned char>>;

// write(g, s, table) for every group and pass whose stage-ordered twiddles the
// device does not hold yet (tuning goes through all variants of a size).
template <typename R, typename Write>
int each_new_twiddles(ssfm_ctx* c, TwiddleTables* tables, Write write) {
  const bool fp64 = c->precision == SSFM_FP64;
  std::vector<double> tmp;
  c->tw_radices.resize(c->groups.size());
  for (size_t gi = 0; gi < c->groups.size(); ++gi) {
    const Group& g = c->groups[gi];
    for (int s = 0; s < P_SLOTS; ++s) {
      PlanInfo pi{};
      if (!plan_info(s & 1, g.n, g.variant(s), fp64, &pi))
        return fail(SSFM_EUNSUPPORTED, "no kernel plan for n=%d", g.n);
      std::vector<int> radices;
      for (const int* r = pi.radices; *r; ++r) radices.push_back(*r);
      std::vector<int>& held = c->tw_radices[gi][s];
      if (held == radices) continue;
      std::vector<unsigned char>& table = (*tables)[radices];
      if (table.empty()) {
        stage_twiddles(g.n, pi.radices, &tmp);
        append_table<R>(&table, tmp);
      }
      held.clear();  // unknown should the write fail
      if (int r = write(g, s, table)) return r;
      held = radices;
    }
  }
  return SSFM_OK;
}

// The twiddles of newly selected variants and the first partials of every
// beam (they follow the variants in use) to the device.
template <typename R>
int upload_variants(ssfm_ctx* c) {
  auto copy = [&](const Group& g, int s, const std::vector<unsigned char>& table) -> int {
    HIP_TRY(hipMemcpyAsync(c->ws + c->L.tables + (g.tw + int64_t(s) * g.n) * c->el, table.data(),
                           table.size(), hipMemcpyHostToDevice, c->stream));
    return SSFM_OK;
  };
  TwiddleTables tables;
  if (int r = each_new_twiddles<R>(c, &tables, copy)) return r;
  HIP_TRY(hipMemcpyAsync(c->ws + c->L.begins, c->begins.data(),
                         sizeof(int32_t) * c->begins.size(), hipMemcpyHostToDevice, c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));
  return SSFM_OK;
}

// Host tables and beam constants to the device: the regions from the beam
// table to the end of the tables as one image (by a copy per table, and a
// twiddle table computed for each pass, creating a context of four sizes took
// 608 us, so 396; one of 4096^2 633, 421).
template <typename R>
int upload_plan(ssfm_ctx* c) {
  const int n_inst = int(c->desc.size());
  std::vector<double> tmp;
  std::vector<unsigned char> image(c->L.tables + size_t(c->L.table_elems) * c->el - c->L.inst);
  auto place = [&](size_t at, const void* src, size_t bytes) {
    std::memcpy(image.data() + (at - c->L.inst), src, bytes);
  };
  c->inst.assign(n_inst, InstDev{});
  if (c->spectrum.size() != size_t(n_inst)) c->spectrum.assign(n_inst, ssfm_ctx::Spectrum{});
  c->screen_steps.clear();
  int64_t foff = 0, soff = 0;
  auto place_twiddles = [&](const Group& g, int s, const std::vector<unsigned char>& table) {
    place(c->L.tables + (g.tw + int64_t(s) * g.n) * c->el, table.data(), table.size());
    return SSFM_OK;
  };
  TwiddleTables twiddles;
  if (int r = each_new_twiddles<R>(c, &twiddles, place_twiddles)) return r;
  place(c->L.begins, c->begins.data(), sizeof(int32_t) * c->begins.size());
  for (const Group& g : c->groups) {
    // the group's beams: T_COUNT tables each
    std::vector<unsigned char> blob;
    for (int b = g.beam0; b < g.beam0 + g.count; ++b) {
      const ssfm_instance_desc& d = c->desc[b];
      InstDev& in = c->inst[b];
      in.n = d.n;
      in.K = (d.mpa_order >= 2) ? d.mpa_order : 2;
      in.terms = d.terms;
      in.n_screens = (d.terms & SSFM_TURB) ? d.n_screens : 0;
      in.off = foff;
      foff += int64_t(d.n) * d.n;
      in.screen_off = soff;
      soff += int64_t(in.n_screens) * d.n * d.n;
      propagator(d, &tmp);
      append_table<R>(&blob, tmp);
      tmp.assign(2 * size_t(d.n), 0.0);
      for (int m = 0; m < d.n; ++m) tmp[2 * m] = 1.0 / d.n;  // identity filter until set
      append_table<R>(&blob, tmp);
      for (int sgn = 1; sgn >= -1; sgn -= 2) {
        ssfm_instance_desc h = d;
        h.dz = sgn * 0.5 * d.dz;
        propagator(h, &tmp);
        append_table<R>(&blob, tmp);
      }
      // 1 - (i dz/4k0) Lap_h has eigenvalue 1 + i (d[mx] + d[my]) on the DFT
      // mode (mx, my) of the periodic 5-point Laplacian
      const double k0 = 2.0 * M_PI / d.wavelength;
      const double dx = d.length / d.n;
      const double coef = d.dz / (k0 * dx * dx);
      tmp.assign(2 * size_t(d.n), 0.0);
      for (int m = 0; m < d.n; ++m) {
        const double sn = std::sin(M_PI * m / d.n);
        tmp[2 * m] = coef * sn * sn;
      }
      append_table<R>(&blob, tmp);
      in.steps_off = int64_t(c->screen_steps.size());
      for (int64_t s : screen_step_list(d)) c->screen_steps.push_back(s);
      in.cK = k0 * d.n2 * d.i_ref * d.dz;
      in.cM = (d.terms & SSFM_MPA) ? (in.K - 1) * d.beta_k * std::pow(d.i_ref, in.K - 1) * d.dz : 0.0;
      in.inv2k1 = 1.0 / (2.0 * (in.K - 1));
      in.cK_f = float(in.cK);
      in.cM_f = float(in.cM);
      // x^(K-1) max(1, |cM|) <= 2^-26 (2^-55 in double): below half an ulp of
      // 1, on either side of it, with room for the powers' rounding.  A
      // coefficient that is not finite leaves nothing weak.
      const auto weak_level = [&](double half_ulp) {
        return 0.999 * std::pow(half_ulp / std::max(1.0, std::fabs(in.cM)), 1.0 / (in.K - 1));
      };
      in.x_weak = std::isfinite(in.cM) ? weak_level(0x1p-55) : -1.0;
      in.x_weak_f = std::isfinite(in.cM_f) ? float(weak_level(0x1p-26)) : -1.0f;
      in.inv2k1_f = float(in.inv2k1);
      for (int p = 0; p < 8; ++p) in.theta[p] = in.theta_f[p] = 0.0;
    }
    place(c->L.tables + g.prop * c->el, blob.data(), blob.size());
  }
  place(c->L.inst, c->inst.data(), sizeof(InstDev) * n_inst);
  if (!c->screen_steps.empty())
    place(c->L.steps, c->screen_steps.data(), sizeof(int64_t) * c->screen_steps.size());
  HIP_TRY(hipMemcpyAsync(c->ws + c->L.inst, image.data(), image.size(), hipMemcpyHostToDevice,
                         c->stream));
  HIP_TRY(hipMemsetAsync(c->field(c->L.S), 0, c->el * c->L.field_elems, c->stream));
  HIP_TRY(hipMemsetAsync(c->ws + c->L.diag, 0, sizeof(double) * 2 * c->L.diag_cap * n_inst,
                         c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));  // host vectors above are temporaries
  return SSFM_OK;
}

const Group& group_of(const ssfm_ctx* c, int b) {
  for (const Group& g : c->groups)
    if (b >= g.beam0 && b < g.beam0 + g.count) return g;
  return c->groups.front();
}

// The lens filter exp(-l_dif k^2) of beam b (1/n per pass) into its filter
// table; *blob holds the host copy until the caller synchronises.
template <typename R>
int upload_lens_filter(ssfm_ctx* c, int b, double l_dif, std::vector<unsigned char>* blob) {
  const ssfm_instance_desc& d = c->desc[b];
  std::vector<double> tab(2 * size_t(d.n), 0.0);
  const double dk = 2.0 * M_PI / d.length;
  for (int m = 0; m < d.n; ++m) {
    const int f = (m <= (d.n - 1) / 2) ? m : m - d.n;  // fftfreq order
    const double k = dk * f;
    tab[2 * m] = std::exp(-l_dif * k * k) / d.n;
  }
  append_table<R>(blob, tab);
  const Group& g = group_of(c, b);
  const int64_t off = g.prop + (int64_t(b - g.beam0) * T_COUNT + T_LENS) * g.n;
  HIP_TRY(hipMemcpyAsync(c->ws + c->L.tables + off * c->el, blob->data(), blob->size(),
                         hipMemcpyHostToDevice, c->stream));
  return SSFM_OK;
}

// Beam b of Wk (and its group's others) <- the lens filter applied to it (row
// and column passes with the filter tables in place of the propagators, no
// screen).
template <typename R>
int lens_filter_passes(ssfm_ctx* c, int b) {
  PassArgs<R> a = base_args<R>(c);
  a.src = c->field(c->L.Wk);
  a.dst = c->field(c->L.Wk);
  a.flags = PASS_OP2;
  const size_t gi = size_t(&group_of(c, b) - c->groups.data());
  const Chain ch{gi, gi + 1, c->stream};
  if (int r = run_pass<R>(c, ROW_FWD, a, ch, T_LENS)) return r;
  return run_pass<R>(c, COL_FWD, a, ch, T_LENS);
}

LensDev lens_dev(const ssfm_instance_desc& d, const ssfm_lens& l) {
  LensDev p{};
  p.i_ref = d.i_ref;
  p.w_l = l.w_l;
  p.c1 = l.c1;
  p.c2 = l.c2;
  p.n_re = l.n_re;
  p.n_im = l.n_im;
  for (int j = 0; j < 8; ++j)
    for (int k = 0; k < 4; ++k) {
      p.re[j][k] = l.re[j][k];
      p.im[j][k] = l.im[j][k];
    }
  return p;
}

// Vector-Jacobian product of the lens at u_in (device complex128 of beam b):
// filter |u|^2, pointwise cotangent and partials, filter h, final cotangent
// and the fixed-order parameter sums (partials and sums in the staging area).
template <typename R>
int do_lens_vjp(ssfm_ctx* c, int b, const ssfm_lens& l, const double* u, const double* g_out,
                double* g_in, double* grad) {
  const ssfm_instance_desc& d = c->desc[b];
  const int64_t n2 = int64_t(d.n) * d.n;
  void* wk = static_cast<char*>(c->field(c->L.Wk)) + c->inst[b].off * int64_t(c->el);
  double* part = c->at<double>(c->L.stage);
  double* sums = part + int64_t(lens_vjp_blocks(n2)) * kLensGrads;
  std::vector<unsigned char> blob;
  if (int r = upload_lens_filter<R>(c, b, l.l_dif, &blob)) return r;
  HIP_TRY(launch_lens_vjp_prep<R>(u, d.i_ref, wk, n2, c->stream));
  if (int r = lens_filter_passes<R>(c, b)) return r;
  HIP_TRY(launch_lens_vjp_point<R>(u, g_out, wk, g_in, n2, lens_dev(d, l), part, c->stream));
  if (int r = lens_filter_passes<R>(c, b)) return r;
  HIP_TRY(launch_lens_vjp_final<R>(u, wk, d.i_ref, g_in, n2, part, sums, c->stream));
  double all[kLensGrads];
  HIP_TRY(hipMemcpyAsync(all, sums, sizeof(all), hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));
  // slots: c1, c2, real segments 0..7, imaginary segments 0..7 -> packed
  int k = 0;
  grad[k++] = all[0];
  grad[k++] = all[1];
  for (int j = 0; j < l.n_re; ++j)
    for (int q = 0; q < 3; ++q) grad[k++] = all[2 + 3 * j + q];
  for (int j = 0; j < l.n_im; ++j)
    for (int q = 0; q < 3; ++q) grad[k++] = all[26 + 3 * j + q];
  return SSFM_OK;
}

// Effective lens on beam b: filter |U|^2 through the pass kernels, then the
// pointwise lens where the filtered intensity reaches the trimming level.
template <typename R>
int do_apply_lens(ssfm_ctx* c, int b, const ssfm_lens& l) {
  const ssfm_instance_desc& d = c->desc[b];
  if (int r = flush_pending<R>(c)) return r;
  std::vector<unsigned char> blob;
  if (int r = upload_lens_filter<R>(c, b, l.l_dif, &blob)) return r;
  HIP_TRY(launch_lens_prep<R>(c->field(c->L.S), c->field(c->L.Wk), c->L.field_elems, c->stream));
  if (int r = lens_filter_passes<R>(c, b)) return r;
  const LensDev p = lens_dev(d, l);
  const int64_t off = c->inst[b].off;
  HIP_TRY(launch_lens_apply<R>(static_cast<char*>(c->field(c->L.S)) + off * c->el,
                               static_cast<const char*>(c->field(c->L.Wk)) + off * c->el,
                               int64_t(d.n) * d.n, p, c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));  // the filter table above is a host temporary
  drop_record(c);
  return SSFM_OK;
}

#define SSFM_DISPATCH(ctx, fn, ...) \
  ((ctx)->precision == SSFM_FP64 ? fn<double>(__VA_ARGS__) : fn<float>(__VA_ARGS__))

// Device pointer of a caller buffer, staging host data through the
// workspace's complex128 staging area (bytes <= 16 n_max^2).
int stage_in(ssfm_ctx* c, const void* src, int32_t where, size_t bytes, const double** out) {
  if (!src) return fail(SSFM_EINVAL, "source pointer is NULL");
  if (where == SSFM_DEVICE) {
    *out = static_cast<const double*>(src);
    return SSFM_OK;
  }
  if (where != SSFM_HOST) return fail(SSFM_EINVAL, "where must be SSFM_HOST or SSFM_DEVICE");
  HIP_TRY(hipMemcpyAsync(c->ws + c->L.stage, src, bytes, hipMemcpyHostToDevice, c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));  // the caller may free src on return
  *out = c->at<double>(c->L.stage);
  return SSFM_OK;
}

template <typename R>
int store_out(ssfm_ctx* c, int b, const void* state, int64_t pending, double scale, void* dst,
              int32_t where, bool intensity) {
  if (!dst) return fail(SSFM_EINVAL, "destination pointer is NULL");
  if (where != SSFM_HOST && where != SSFM_DEVICE)
    return fail(SSFM_EINVAL, "where must be SSFM_HOST or SSFM_DEVICE");
  const int n = c->desc[b].n;
  const size_t bytes = (intensity ? 8 : 16) * size_t(n) * n;
  double* out = (where == SSFM_DEVICE) ? static_cast<double*>(dst) : c->at<double>(c->L.stage);
  HIP_TRY(launch_store_field<R>(state, c->at<InstDev>(c->L.inst), b, n, c->at<R>(c->L.screens),
                                c->at<int64_t>(c->L.steps), pending, scale, out, intensity,
                                c->stream));
  if (where == SSFM_HOST) {
    HIP_TRY(hipMemcpyAsync(dst, out, bytes, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
  }
  return SSFM_OK;
}

template <typename R>
int do_set_field(ssfm_ctx* c, int b, const void* src, int32_t where) {
  if (int r = not_captured(c)) return r;
  if (c->step > 0 || c->pending) {
    // keep the other beams exact: apply their pending screen first
    if (int r = flush_pending<R>(c)) return r;
  }
  const int n = c->desc[b].n;
  const double* dsrc;
  if (int r = stage_in(c, src, where, 16 * size_t(n) * n, &dsrc)) return r;
  // beam b starts its own step count (its screen schedule) here; the other
  // beams keep theirs.  Once every beam has been set at the same step, the
  // context count restarts at 0 (so marches from fresh fields reuse their
  // captured graphs).
  c->pending = false;
  c->diag_valid = 0;
  drop_record(c);
  c->inst[b].step_base = c->step;
  bool same = true;
  for (const InstDev& in : c->inst) same = same && (in.step_base == c->step);
  if (same) {
    const bool restart = c->step != 0;
    for (InstDev& in : c->inst) in.step_base = 0;
    c->step = 0;
    if (restart && c->inst.size() > 1)
      if (int r = upload_inst(c, 0, c->inst.size())) return r;
  }
  HIP_TRY(launch_load_field<R>(dsrc, static_cast<char*>(c->field(c->L.S)) + c->inst[b].off * c->el,
                               int64_t(n) * n, 1.0 / std::sqrt(c->desc[b].i_ref), c->inst[b],
                               c->at<InstDev>(c->L.inst) + b, c->stream));
  if (c->strang) {
    // the state of a Strang march is V = L(dz/2) U: half a step for beam b
    if (int r = half_steps<R>(c, true)) return r;
    const size_t off = size_t(c->inst[b].off) * c->el;
    HIP_TRY(launch_copy<R>(static_cast<char*>(c->field(c->L.Wk)) + off,
                           static_cast<char*>(c->field(c->L.S)) + off, int64_t(n) * n,
                           c->stream));
  }
  return SSFM_OK;
}

// Lines per workgroup of a variant (0 if it does not exist).
int plan_lines(bool column, int n, int v) {
  PlanInfo pi{};
  plan_info(column, n, v, false, &pi);
  return pi.lines;
}

// Switch size n to other variants: the partials' offsets and the twiddle
// tables follow; the layout's arrays hold any variant, so their offsets
// stay.
int apply_variants(ssfm_ctx* c, int n, const std::array<int, P_SLOTS>& var) {
  VariantMap vm;
  for (auto& g : c->groups) {
    std::array<int, P_SLOTS> v;
    std::copy(g.var, g.var + P_SLOTS, v.begin());
    vm[g.n] = (g.n == n) ? var : v;
  }
  Layout L2;
  std::vector<Group> groups;
  std::vector<int32_t> begins;
  if (int r = plan_layout(c->desc.data(), int(c->desc.size()), c->precision, c->max_steps,
                          c->ckpt_every, c->stored_segments, &vm, &groups, &begins, &L2))
    return r;
  if (L2.total != c->L.total) return fail(SSFM_EUNSUPPORTED, "variant changes the workspace layout");
  HIP_TRY(hipStreamSynchronize(c->stream));
  c->groups = groups;
  c->begins = begins;
  c->L = L2;
  clear_graphs(c);
  if (int r = SSFM_DISPATCH(c, upload_variants, c)) return r;
  return SSFM_OK;
}

// Adjoint-pass variants of size n (-1: follow the forward variants).
int do_select_adjoint(ssfm_ctx* c, int32_t n, int32_t rv, int32_t cv) {
  const bool fp64 = c->precision == SSFM_FP64;
  const int rc = plan_count(false, n), cc = plan_count(true, n);
  if (rc == 0) return fail(SSFM_EUNSUPPORTED, "grid size %d not supported", n);
  if (rv < -1 || rv >= rc || cv < -1 || cv >= cc)
    return fail(SSFM_EINVAL, "variant (%d, %d) out of range [-1, %d) x [-1, %d)", rv, cv, rc, cc);
  Group* grp = nullptr;
  for (auto& g : c->groups)
    if (g.n == n) grp = &g;
  if (!grp) return fail(SSFM_EINVAL, "no instance with n=%d in this context", n);
  PlanInfo pi{};
  if (rv >= 0) {
    if (!plan_info(false, n, rv, fp64, &pi))
      return fail(SSFM_EUNSUPPORTED, "row variant %d of n=%d is not built at this precision", rv, n);
    if (pi.lines != grp->lines[P_ROW])
      return fail(SSFM_EINVAL, "row variant %d has %d lines per workgroup, the forward one %d", rv,
                  pi.lines, grp->lines[P_ROW]);
  }
  if (cv >= 0) {
    if (!plan_info(true, n, cv, fp64, &pi))
      return fail(SSFM_EUNSUPPORTED, "column variant %d of n=%d is not built at this precision",
                  cv, n);
    if (pi.lines != grp->lines[P_COL])
      return fail(SSFM_EINVAL, "column variant %d has %d columns per workgroup, the forward one %d",
                  cv, pi.lines, grp->lines[P_COL]);
  }
  return apply_variants(c, n, {grp->var[P_ROW], grp->var[P_COL], rv, cv});
}

int do_select(ssfm_ctx* c, int32_t n, int32_t rv, int32_t cv) {
  const int rc = plan_count(false, n), cc = plan_count(true, n);
  if (rc == 0) return fail(SSFM_EUNSUPPORTED, "grid size %d not supported", n);
  if (rv < 0 || rv >= rc || cv < 0 || cv >= cc)
    return fail(SSFM_EINVAL, "variant (%d, %d) out of range [0, %d) x [0, %d)", rv, cv, rc, cc);
  const Group* grp = nullptr;
  for (auto& g : c->groups)
    if (g.n == n) grp = &g;
  if (!grp) return fail(SSFM_EINVAL, "no instance with n=%d in this context", n);
  // keep the adjoint variants while their lines per workgroup still match
  // the forward ones
  int ra = grp->var[P_ROW_ADJ], ca = grp->var[P_COL_ADJ];
  if (ra >= 0 && plan_lines(false, n, ra) != plan_lines(false, n, rv)) ra = -1;
  if (ca >= 0 && plan_lines(true, n, ca) != plan_lines(true, n, cv)) ca = -1;
  return apply_variants(c, n, {rv, cv, ra, ca});
}

}  // namespace

// ================================================================ C ABI
extern "C" {

int ssfm_version(void) { return SSFM_VERSION; }

const char* ssfm_strerror(int s) {
  switch (s) {
    case SSFM_OK: return "ok";
    case SSFM_EINVAL: return "invalid argument";
    case SSFM_EUNSUPPORTED: return "unsupported grid size or option";
    case SSFM_EHIP: return "HIP runtime error";
    case SSFM_ESTATE: return "call out of order";
    case SSFM_ENONFINITE: return "non-finite power or gradient";
    case SSFM_EWORKSPACE: return "workspace missing, misaligned or too small";
    default: return "unknown status";
  }
}

const char* ssfm_last_error(void) { return g_last_error.c_str(); }

int ssfm_workspace_bytes(const ssfm_instance_desc* desc, int32_t n_inst, int32_t precision,
                         int64_t max_steps, int32_t ckpt_every, int32_t stored_segments,
                         size_t* bytes) {
  g_last_error.clear();
  if (!bytes) return fail(SSFM_EINVAL, "bytes is NULL");
  if (int r = validate_desc(desc, n_inst, precision)) return r;
  if (max_steps < 0 || ckpt_every < 1 || stored_segments < 0)
    return fail(SSFM_EINVAL, "need max_steps >= 0, ckpt_every >= 1, stored_segments >= 0");
  Layout L;
  if (int r = plan_layout(desc, n_inst, precision, max_steps, ckpt_every, stored_segments, nullptr,
                          nullptr, nullptr, &L))
    return r;
  *bytes = L.total;
  return SSFM_OK;
}

int ssfm_checkpoint_plan(const ssfm_instance_desc* desc, int32_t n_inst, int32_t precision,
                         int64_t n_steps, size_t budget_bytes, int32_t* ckpt_every,
                         int32_t* stored_segments, int64_t* recomputed) {
  g_last_error.clear();
  if (!ckpt_every || !stored_segments) return fail(SSFM_EINVAL, "output pointer is NULL");
  if (int r = validate_desc(desc, n_inst, precision)) return r;
  if (n_steps < 1 || n_steps > INT32_MAX) return fail(SSFM_EINVAL, "need 1 <= n_steps < 2^31");
  Layout L;
  auto bytes_of = [&](int64_t m, int64_t k, size_t* out) {
    int r = plan_layout(desc, n_inst, precision, n_steps, int32_t(m), int32_t(k), nullptr,
                        nullptr, nullptr, &L);
    *out = L.total;
    return r;
  };
  size_t b = 0;
  // every pre-screen field kept: no recompute
  if (int r = bytes_of(n_steps, 0, &b)) return r;
  if (b <= budget_bytes) {
    *ckpt_every = int32_t(n_steps);
    *stored_segments = 0;
    if (recomputed) *recomputed = 0;
    return SSFM_OK;
  }
  if (n_steps < 3) return fail(SSFM_EWORKSPACE, "%zu bytes needed, budget %zu", b, budget_bytes);
  // With M < n_steps the layout is affine in its field slots (every field
  // array is a whole number of alignment units): bytes = A + F * slots,
  // slots = checkpoints + (M - 1) * (banks + kept segments).
  auto slots_of = [&](int64_t m, int64_t k) {
    const int64_t seg = (n_steps + m - 1) / m;
    const int64_t kept = std::min(k, seg);
    return seg + (m - 1) * (std::min<int64_t>(2, seg - kept) + kept);
  };
  size_t b2 = 0;
  if (int r = bytes_of(2, 0, &b2)) return r;
  const double F = double(L.field_elems) * (precision == SSFM_FP64 ? 16.0 : 8.0);
  const double A = double(b2) - F * double(slots_of(2, 0));
  const double cap = (double(budget_bytes) - A) / F;  // field slots that fit
  // Cost of (M, K): steps recomputed by the backward, plus one per segment
  // for its fork, join and checkpoint boundary; the cheapest that fits.
  int64_t best_m = -1, best_k = 0, best_rec = 0;
  double best_cost = 0.0;
  for (int64_t m = 2; m < n_steps; ++m) {
    const int64_t seg = (n_steps + m - 1) / m;
    if (double(slots_of(m, 0)) > cap) continue;
    // kept segments that fit (slots rise with K; K = seg - 1 costs what
    // K = seg costs, so it is never the choice)
    int64_t k = 0;
    if (double(slots_of(m, seg)) <= cap) {
      k = seg;
    } else {
      const double room = (cap - double(seg)) / double(m - 1) - 2.0;
      k = std::max<int64_t>(0, std::min<int64_t>(seg - 2, int64_t(std::floor(room))));
      while (k > 0 && double(slots_of(m, k)) > cap) --k;
    }
    const int64_t rec = (k == 0) ? n_steps - seg : (seg - std::min(k, seg)) * (m - 1);
    const double cost = double(rec) + double(seg);
    if (best_m < 0 || cost < best_cost) {
      best_m = m;
      best_k = k;
      best_rec = rec;
      best_cost = cost;
    }
  }
  if (best_m < 0) {
    // the smallest layout: M near sqrt(n_steps / 2), nothing kept
    size_t need = 0;
    bytes_of(std::max<int64_t>(2, int64_t(std::sqrt(0.5 * double(n_steps)))), 0, &need);
    return fail(SSFM_EWORKSPACE, "no checkpoint layout fits %zu bytes (at least %zu needed)",
                budget_bytes, need);
  }
  // the affine model is exact; confirm with the layout itself
  if (int r = bytes_of(best_m, best_k, &b)) return r;
  if (b > budget_bytes)
    return fail(SSFM_EWORKSPACE, "checkpoint layout of %zu bytes exceeds budget %zu", b,
                budget_bytes);
  *ckpt_every = int32_t(best_m);
  *stored_segments = int32_t(best_k);
  if (recomputed) *recomputed = best_rec;
  return SSFM_OK;
}

int ssfm_create(const ssfm_instance_desc* desc, int32_t n_inst, int32_t precision,
                int64_t max_steps, int32_t ckpt_every, int32_t stored_segments,
                void* workspace, size_t ws_bytes, void* stream, ssfm_ctx** out) {
  g_last_error.clear();
  if (!out) return fail(SSFM_EINVAL, "out is NULL");
  *out = nullptr;
  if (int r = validate_desc(desc, n_inst, precision)) return r;
  if (max_steps < 0 || ckpt_every < 1 || stored_segments < 0)
    return fail(SSFM_EINVAL, "need max_steps >= 0, ckpt_every >= 1, stored_segments >= 0");
  std::unique_ptr<ssfm_ctx> c(new ssfm_ctx);
  c->precision = precision;
  c->el = precision == SSFM_FP64 ? 16 : 8;
  c->caller = group_order(desc, n_inst);
  c->slot.assign(n_inst, 0);
  for (int b = 0; b < n_inst; ++b) {
    c->slot[c->caller[b]] = b;
    c->desc.push_back(desc[c->caller[b]]);
  }
  c->seeded_beam.assign(n_inst, 0);
  c->max_steps = max_steps;
  c->ckpt_every = ckpt_every;
  c->stored_segments = stored_segments;
  c->stream = static_cast<hipStream_t>(stream);
  if (int r = plan_layout(c->desc.data(), n_inst, precision, max_steps, ckpt_every,
                          stored_segments, nullptr, &c->groups, &c->begins, &c->L))
    return r;
  if (!workspace) return fail(SSFM_EWORKSPACE, "workspace is NULL");
  if (reinterpret_cast<uintptr_t>(workspace) % kAlign)
    return fail(SSFM_EWORKSPACE, "workspace must be %zu-byte aligned", kAlign);
  if (ws_bytes < c->L.total)
    return fail(SSFM_EWORKSPACE, "workspace has %zu bytes, needs %zu", ws_bytes, c->L.total);
  c->ws = static_cast<char*>(workspace);
  HIP_TRY(hipStreamCreateWithFlags(&c->aux, hipStreamNonBlocking));
  HIP_TRY(hipEventCreateWithFlags(&c->ev_fork, hipEventDisableTiming));
  HIP_TRY(hipEventCreateWithFlags(&c->ev_join, hipEventDisableTiming));
  HIP_TRY(hipEventCreateWithFlags(&c->gfork, hipEventDisableTiming));
  for (size_t g = 1; g < c->groups.size(); ++g) {
    hipStream_t sg;
    hipEvent_t ej;
    HIP_TRY(hipStreamCreateWithFlags(&sg, hipStreamNonBlocking));
    c->gstream.push_back(sg);
    HIP_TRY(hipEventCreateWithFlags(&ej, hipEventDisableTiming));
    c->gjoin.push_back(ej);
  }
  int r = SSFM_DISPATCH(c, upload_plan, c.get());
  if (r) return r;
  *out = c.release();
  return SSFM_OK;
}

int ssfm_destroy(ssfm_ctx* ctx) {
  if (!ctx) return SSFM_OK;
  (void)hipStreamSynchronize(ctx->stream);
  delete ctx;
  return SSFM_OK;
}

int ssfm_set_field(ssfm_ctx* c, int32_t inst, const void* src, int32_t where) {
  if (int r = check_inst(c, inst)) return r;
  return SSFM_DISPATCH(c, do_set_field, c, inst, src, where);
}

int ssfm_set_theta(ssfm_ctx* c, int32_t inst, const double* theta) {
  if (int r = check_inst(c, inst)) return r;
  if (!theta) return fail(SSFM_EINVAL, "theta is NULL");
  for (int p = 0; p < 8; ++p) {
    if (!std::isfinite(theta[p])) return fail(SSFM_EINVAL, "theta[%d] not finite", p);
    c->inst[inst].theta[p] = theta[p];
    c->inst[inst].theta_f[p] = float(theta[p]);
  }
  // a recorded march (its stored fields, the screen its adjoint applies)
  // belongs to the old parameters
  drop_record(c);
  return upload_inst(c, inst, inst + 1);
}

int ssfm_gen_screens(ssfm_ctx* c) {
  if (int r = check_ctx(c)) return r;
  drop_record(c);  // the recorded march used the previous screens
  return SSFM_DISPATCH(c, do_gen_screens, c);
}

int ssfm_get_screen(ssfm_ctx* c, int32_t inst, int32_t s, void* dst, int32_t where) {
  if (int r = check_inst(c, inst)) return r;
  const InstDev& in = c->inst[inst];
  if (s < 0 || s >= in.n_screens) return fail(SSFM_EINVAL, "screen %d out of range", s);
  if (!dst) return fail(SSFM_EINVAL, "dst is NULL");
  const int64_t n2 = int64_t(in.n) * in.n;
  double* out = (where == SSFM_DEVICE) ? static_cast<double*>(dst) : c->at<double>(c->L.stage);
  const size_t rel = c->el / 2;
  const void* plane = c->ws + c->L.screens + rel * size_t(in.screen_off + int64_t(s) * n2);
  if (c->precision == SSFM_FP64)
    HIP_TRY(launch_screen_to_f64<double>(static_cast<const double*>(plane), n2, out, c->stream));
  else
    HIP_TRY(launch_screen_to_f64<float>(static_cast<const float*>(plane), n2, out, c->stream));
  if (where == SSFM_HOST) {
    HIP_TRY(hipMemcpyAsync(dst, out, 8 * n2, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(hipStreamSynchronize(c->stream));
  }
  return SSFM_OK;
}

int ssfm_propagate(ssfm_ctx* c, int64_t n_steps) {
  if (int r = check_ctx(c)) return r;
  if (n_steps < 0) return fail(SSFM_EINVAL, "n_steps < 0");
  if (n_steps == 0) return SSFM_OK;
  return SSFM_DISPATCH(c, do_propagate, c, n_steps);
}

extern "C++" {
// Read-out of beam b: Lie applies the pending screen; Strang diffracts the
// state V back by half a step (U = L(-dz/2) V) in the work buffer first.
template <typename R>
int read_out(ssfm_ctx* c, int b, void* dst, int32_t where, bool intensity) {
  const double sc = std::sqrt(c->desc[b].i_ref);
  if (c->strang) {
    if (int r = half_steps<R>(c, false)) return r;
    return store_out<R>(c, b, c->field(c->L.Wk), -1, sc, dst, where, intensity);
  }
  const int64_t pend = c->pending ? c->step - 1 : -1;
  return store_out<R>(c, b, c->field(c->L.S), pend, sc, dst, where, intensity);
}
}  // extern "C++"

int ssfm_get_field(ssfm_ctx* c, int32_t inst, void* dst, int32_t where) {
  if (int r = check_inst(c, inst)) return r;
  return SSFM_DISPATCH(c, read_out, c, inst, dst, where, false);
}

int ssfm_get_intensity(ssfm_ctx* c, int32_t inst, void* dst, int32_t where) {
  if (int r = check_inst(c, inst)) return r;
  return SSFM_DISPATCH(c, read_out, c, inst, dst, where, true);
}

int ssfm_set_splitting(ssfm_ctx* c, int32_t scheme) {
  if (int r = check_ctx(c)) return r;
  if (scheme != SSFM_LIE && scheme != SSFM_STRANG && scheme != SSFM_FD)
    return fail(SSFM_EINVAL, "unknown scheme %d", scheme);
  if (scheme == SSFM_FD) {
    for (size_t b = 0; b < c->desc.size(); ++b) {
      const ssfm_instance_desc& d = c->desc[b];
      if ((d.terms & SSFM_ANSATZ) || ((d.terms & SSFM_TURB) && d.n_screens > 0))
        return fail(SSFM_EUNSUPPORTED,
                    "the finite-difference scheme covers the Kerr, plasma and multiphoton "
                    "terms only (instance %d has the ansatz or turbulence screens)", c->caller[b]);
    }
  }
  HIP_TRY(hipStreamSynchronize(c->stream));
  clear_graphs(c);
  c->strang = (scheme == SSFM_STRANG);
  c->fd = (scheme == SSFM_FD);
  HIP_TRY(hipMemsetAsync(c->field(c->L.S), 0, c->el * c->L.field_elems, c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));
  c->step = 0;
  c->pending = false;
  c->diag_valid = 0;
  drop_record(c);
  for (InstDev& in : c->inst) in.step_base = 0;
  return upload_inst(c, 0, c->inst.size());
}

namespace {
int split_step_only(ssfm_ctx* c, const char* what) {
  if (c->fd)
    return fail(SSFM_EUNSUPPORTED, "%s needs a split-step scheme (the finite-difference scheme "
                                   "marches forward only)", what);
  return SSFM_OK;
}

int lie_only(ssfm_ctx* c, const char* what) {
  if (c->strang || c->fd)
    return fail(SSFM_EUNSUPPORTED, "%s needs the Lie split-step scheme (%s marches forward only)",
                what, c->strang ? "Strang" : "the finite-difference scheme");
  return SSFM_OK;
}

}  // namespace

int ssfm_set_fd_iterations(ssfm_ctx* c, int32_t iterations) {
  if (int r = check_ctx(c)) return r;
  if (iterations < 1 || iterations > 64)
    return fail(SSFM_EINVAL, "finite-difference iterations must be in [1, 64], got %d",
                iterations);
  HIP_TRY(hipStreamSynchronize(c->stream));
  clear_graphs(c);
  c->fd_iters = iterations;
  return SSFM_OK;
}

int ssfm_get_diag(ssfm_ctx* c, int32_t inst, double* power, double* peak, int64_t n) {
  if (int r = check_inst(c, inst)) return r;
  if (n < 0 || n > c->diag_valid)
    return fail(SSFM_EINVAL, "n=%lld exceeds the %lld recorded diagnostic steps", (long long)n,
                (long long)c->diag_valid);
  if (n == 0) return SSFM_OK;
  std::vector<double> buf(2 * size_t(c->L.diag_cap));
  HIP_TRY(hipMemcpyAsync(buf.data(), c->ws + c->L.diag + sizeof(double) * 2 * c->L.diag_cap * inst,
                         sizeof(double) * 2 * c->L.diag_cap, hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));
  const ssfm_instance_desc& d = c->desc[inst];
  const double dx = d.length / d.n;
  int status = SSFM_OK;
  for (int64_t i = 0; i < n; ++i) {
    const int64_t step = c->step - n + i;
    const int64_t slot = step % c->L.diag_cap;
    const double pw = buf[2 * slot] * d.i_ref * dx * dx;
    const double pk = buf[2 * slot + 1] * d.i_ref;
    if (power) power[i] = pw;
    if (peak) peak[i] = pk;
    if (!std::isfinite(pw)) status = SSFM_ENONFINITE;
  }
  if (status) return fail(status, "non-finite power in the diagnostics of instance %d", inst);
  return SSFM_OK;
}

int ssfm_forward_record(ssfm_ctx* c, int64_t n_steps) {
  if (int r = check_ctx(c)) return r;
  if (int r = split_step_only(c, "forward_record")) return r;
  if (n_steps < 1) return fail(SSFM_EINVAL, "n_steps must be >= 1");
  return SSFM_DISPATCH(c, do_record, c, n_steps);
}

int ssfm_set_cotangent(ssfm_ctx* c, int32_t inst, const void* g, int32_t where) {
  if (int r = check_inst(c, inst)) return r;
  if (int r = split_step_only(c, "set_cotangent")) return r;
  if (!c->rec_valid) return fail(SSFM_ESTATE, "set_cotangent needs a preceding forward_record");
  const int n = c->desc[inst].n;
  const double* dg;
  if (int r = stage_in(c, g, where, 16 * size_t(n) * n, &dg)) return r;
  int r = SSFM_DISPATCH(c, do_seed, c, inst, 1, nullptr, dg);
  if (r) return r;
  if (where == SSFM_HOST) HIP_TRY(hipStreamSynchronize(c->stream));
  c->seeded = true;
  c->seeded_beam[inst] = 1;
  return SSFM_OK;
}

int ssfm_fluence_loss(ssfm_ctx* c, int32_t inst, const void* target, int32_t where, double* loss) {
  if (int r = check_inst(c, inst)) return r;
  if (int r = split_step_only(c, "fluence_loss")) return r;
  if (!c->rec_valid) return fail(SSFM_ESTATE, "fluence_loss needs a preceding forward_record");
  const int n = c->desc[inst].n;
  const double* dt;
  if (int r = stage_in(c, target, where, 8 * size_t(n) * n, &dt)) return r;
  int r = SSFM_DISPATCH(c, do_seed, c, inst, 0, dt, nullptr);
  if (r) return r;
  std::vector<double> part(n + 1);  // the rows' losses, then sum w^2
  HIP_TRY(hipMemcpyAsync(part.data(), c->ws + c->L.seed_loss, sizeof(double) * (n + 1),
                         hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));
  double s = 0.0;
  for (int i = 0; i < n; ++i) s += part[i];
  if (loss) *loss = s / part[n];
  c->seeded = true;
  c->seeded_beam[inst] = 1;
  return SSFM_OK;
}

int ssfm_fluence_mismatch(ssfm_ctx* c, int32_t inst, const void* target, int32_t where,
                          double* loss) {
  if (int r = check_inst(c, inst)) return r;
  if (!loss) return fail(SSFM_EINVAL, "loss is NULL");
  const int n = c->desc[inst].n;
  const double* dt;
  if (int r = stage_in(c, target, where, 8 * size_t(n) * n, &dt)) return r;
  // the sums go to the staging area past the target
  double* part = c->at<double>(c->L.stage) + size_t(n) * n;
  auto run = [&]<typename R>(R*) -> int {
    // the field U: the state with its pending screen (Lie), the state itself
    // (finite differences), or L(-dz/2) of it in the work buffer (Strang)
    const void* state = c->field(c->L.S);
    int64_t pend = c->pending ? c->step - 1 : -1;
    if (c->strang) {
      if (int r = half_steps<R>(c, false)) return r;
      state = c->field(c->L.Wk);
      pend = -1;
    }
    HIP_TRY(launch_mismatch<R>(state, c->at<InstDev>(c->L.inst), inst, n, c->at<R>(c->L.screens),
                               c->at<int64_t>(c->L.steps), pend, dt, c->desc[inst].i_ref, part,
                               c->stream));
    return SSFM_OK;
  };
  if (int r = (c->precision == SSFM_FP64) ? run((double*)nullptr) : run((float*)nullptr))
    return r;
  std::vector<double> h(size_t(n) + kSumParts);
  HIP_TRY(hipMemcpyAsync(h.data(), part, sizeof(double) * h.size(), hipMemcpyDeviceToHost,
                         c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));
  double s = 0.0, wsum = 0.0;
  for (int i = 0; i < n; ++i) s += h[i];
  // the order in which a workgroup sums them for ssfm_fluence_loss: a
  // butterfly over each wavefront's 64, then the wavefronts
  for (int w = 0; w < kSumParts; w += 64) {
    double* p = h.data() + n + w;
    for (int off = 32; off >= 1; off /= 2)
      for (int i = 0; i < off; ++i) p[i] += p[i + off];
    wsum += p[0];
  }
  *loss = s / wsum;
  return SSFM_OK;
}

int ssfm_backward(ssfm_ctx* c) {
  if (int r = check_ctx(c)) return r;
  if (int r = split_step_only(c, "backward")) return r;
  return SSFM_DISPATCH(c, do_backward, c);
}

int ssfm_get_grad_field(ssfm_ctx* c, int32_t inst, void* dst, int32_t where) {
  if (int r = check_inst(c, inst)) return r;
  if (!c->grads_valid) return fail(SSFM_ESTATE, "no gradient: call ssfm_backward first");
  const double sc = 1.0 / std::sqrt(c->desc[inst].i_ref);
  return SSFM_DISPATCH(c, store_out, c, inst, c->field(c->L.Lam), -1, sc, dst, where, false);
}

int ssfm_get_grad_theta(ssfm_ctx* c, int32_t inst, double* g) {
  if (int r = check_inst(c, inst)) return r;
  if (!c->grads_valid) return fail(SSFM_ESTATE, "no gradient: call ssfm_backward first");
  if (!g) return fail(SSFM_EINVAL, "g is NULL");
  double acc[8], seed_part[8];
  const int n = c->desc[inst].n;
  std::vector<double> sp(size_t(8) * n);
  HIP_TRY(hipMemcpyAsync(acc, c->ws + c->L.theta_out + sizeof(double) * 8 * inst,
                         sizeof(double) * 8, hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(hipMemcpyAsync(sp.data(), c->ws + c->L.seed_theta + sizeof(double) * 8 * c->L.max_n * inst,
                         sizeof(double) * 8 * n, hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));
  for (int p = 0; p < 8; ++p) {
    seed_part[p] = 0.0;
    for (int r = 0; r < n; ++r) seed_part[p] += sp[size_t(r) * 8 + p];
    g[p] = acc[p] + seed_part[p];
  }
  for (int p = 0; p < 8; ++p)
    if (!std::isfinite(g[p]))
      return fail(SSFM_ENONFINITE,
                  "theta gradient of instance %d is not finite: the linearised march "
                  "outgrew the precision's range", inst);
  return SSFM_OK;
}

int ssfm_block_mean(ssfm_ctx* c, const double* src, int32_t n, int32_t b, double* dst) {
  if (int r = check_ctx(c)) return r;
  if (!src || !dst) return fail(SSFM_EINVAL, "src/dst is NULL");
  if (n < 1 || b < 1 || n % b) return fail(SSFM_EINVAL, "block %d must divide n=%d", b, n);
  HIP_TRY(launch_block_mean(src, n, b, dst, c->stream));
  return SSFM_OK;
}

int ssfm_set_recompute_overlap(ssfm_ctx* c, int32_t enable) {
  if (int r = check_ctx(c)) return r;
  c->overlap_recompute = enable != 0;
  // captured backward sweeps hold the previous schedule
  clear_graphs(c);
  return SSFM_OK;
}

int ssfm_set_precise_math(ssfm_ctx* c, int32_t enable) {
  if (int r = check_ctx(c)) return r;
  c->precise = enable != 0;
  for (auto& in : c->inst) {
    if (enable) in.terms |= (1u << 8);
    else in.terms &= ~(1u << 8);
  }
  HIP_TRY(hipMemcpyAsync(c->ws + c->L.inst, c->inst.data(), sizeof(InstDev) * c->inst.size(),
                         hipMemcpyHostToDevice, c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));
  // captured steps hold the kernels chosen for the previous setting
  clear_graphs(c);
  return SSFM_OK;
}

int ssfm_use_graphs(ssfm_ctx* c, int32_t enable) {
  if (int r = check_ctx(c)) return r;
  c->use_graphs = enable != 0;
  return SSFM_OK;
}

int ssfm_plan_variants(int32_t n, int32_t precision, int32_t* n_row, int32_t* n_col) {
  if (!n_row || !n_col) return fail(SSFM_EINVAL, "n_row/n_col is NULL");
  if (precision != SSFM_FP32 && precision != SSFM_FP64) return fail(SSFM_EINVAL, "precision");
  *n_row = plan_count(false, n);
  *n_col = plan_count(true, n);
  if (*n_row == 0 || *n_col == 0) return fail(SSFM_EUNSUPPORTED, "grid size %d not supported", n);
  return SSFM_OK;
}

int ssfm_select_plan(ssfm_ctx* c, int32_t n, int32_t row_variant, int32_t col_variant) {
  if (int r = check_ctx(c)) return r;
  return do_select(c, n, row_variant, col_variant);
}

int ssfm_select_adjoint_plan(ssfm_ctx* c, int32_t n, int32_t row_variant,
                             int32_t col_variant) {
  if (int r = check_ctx(c)) return r;
  return do_select_adjoint(c, n, row_variant, col_variant);
}

int ssfm_time_adjoint_passes(ssfm_ctx* c, int32_t reps, double* ms_col, double* ms_row) {
  if (int r = check_ctx(c)) return r;
  if (reps < 1) return fail(SSFM_EINVAL, "reps must be >= 1");
  if (c->max_steps <= 0)
    return fail(SSFM_ESTATE, "adjoint passes need a context created with max_steps > 0");
  struct Events {
    hipEvent_t e[3] = {nullptr, nullptr, nullptr};
    ~Events() {
      for (auto x : e)
        if (x) (void)hipEventDestroy(x);
    }
  } ev;
  for (auto& x : ev.e) HIP_TRY(hipEventCreate(&x));
  // column pass: cotangent -> work buffer; row pass: work buffer in place,
  // the state standing in for the stored pre-screen field, at a step with
  // no turbulence screen (the ansatz partials go to the accumulators every
  // backward clears first).  Fields, cotangent and gradients are unchanged.
  auto body = [&]<typename R>(R*) -> int {
    PassArgs<R> a = base_args<R>(c);
    a.src = c->field(c->L.Lam);
    a.dst = c->field(c->L.Wk);
    a.aux = c->field(c->L.S);
    a.step = int64_t(1) << 60;
    a.flags = PASS_OP1 | PASS_SCREEN | PASS_OP2;
    PassArgs<R> b = a;
    a.part = c->at<double>(c->L.theta_cols);
    b.src = c->field(c->L.Wk);
    b.part = c->at<double>(c->L.theta_rows);
    HIP_TRY(hipEventRecord(ev.e[0], c->stream));
    for (int i = 0; i < reps; ++i)
      if (int q = run_pass<R>(c, COL_ADJ, a, whole(c))) return q;
    HIP_TRY(hipEventRecord(ev.e[1], c->stream));
    for (int i = 0; i < reps; ++i)
      if (int q = run_pass<R>(c, ROW_ADJ, b, whole(c))) return q;
    HIP_TRY(hipEventRecord(ev.e[2], c->stream));
    return SSFM_OK;
  };
  int r = (c->precision == SSFM_FP64) ? body((double*)nullptr) : body((float*)nullptr);
  if (r) return r;
  HIP_TRY(hipEventSynchronize(ev.e[2]));
  float t1 = 0, t2 = 0;
  HIP_TRY(hipEventElapsedTime(&t1, ev.e[0], ev.e[1]));
  HIP_TRY(hipEventElapsedTime(&t2, ev.e[1], ev.e[2]));
  if (ms_col) *ms_col = double(t1) / reps;
  if (ms_row) *ms_row = double(t2) / reps;
  return SSFM_OK;
}

int ssfm_time_passes(ssfm_ctx* c, int32_t reps, double* ms_row, double* ms_col,
                     double* bytes_row, double* bytes_col) {
  if (int r = check_ctx(c)) return r;
  if (reps < 1) return fail(SSFM_EINVAL, "reps must be >= 1");
  // events released on every return path
  struct Events {
    hipEvent_t e[3] = {nullptr, nullptr, nullptr};
    ~Events() {
      for (auto x : e)
        if (x) (void)hipEventDestroy(x);
    }
  } ev;
  for (auto& x : ev.e) HIP_TRY(hipEventCreate(&x));
  hipEvent_t e0 = ev.e[0], e1 = ev.e[1], e2 = ev.e[2];
  int r = SSFM_OK;
  auto body = [&]<typename R>(R*) -> int {
    PassArgs<R> a = base_args<R>(c);
    a.src = c->field(c->L.S);
    a.dst = c->field(c->L.Wk);
    a.step = int64_t(1) << 60;  // a step with no turbulence screen
    a.flags = PASS_OP1 | PASS_SCREEN | PASS_OP2;
    a.part = c->at<double>(c->L.theta_rows);
    PassArgs<R> b = a;
    b.src = c->field(c->L.Wk);
    HIP_TRY(hipEventRecord(e0, c->stream));
    for (int i = 0; i < reps; ++i)
      if (int q = run_pass<R>(c, ROW_FWD, a, whole(c))) return q;
    HIP_TRY(hipEventRecord(e1, c->stream));
    for (int i = 0; i < reps; ++i)
      if (int q = run_pass<R>(c, COL_FWD, b, whole(c))) return q;
    HIP_TRY(hipEventRecord(e2, c->stream));
    return SSFM_OK;
  };
  r = (c->precision == SSFM_FP64) ? body((double*)nullptr) : body((float*)nullptr);
  if (r == SSFM_OK) {
    HIP_TRY(hipEventSynchronize(e2));
    float t1 = 0, t2 = 0;
    HIP_TRY(hipEventElapsedTime(&t1, e0, e1));
    HIP_TRY(hipEventElapsedTime(&t2, e1, e2));
    if (ms_row) *ms_row = double(t1) / reps;
    if (ms_col) *ms_col = double(t2) / reps;
    const double b = 2.0 * double(c->el) * double(c->L.field_elems);
    if (bytes_row) *bytes_row = b;
    if (bytes_col) *bytes_col = b;
  }
  return r;
}

int ssfm_set_screen_spectrum(ssfm_ctx* c, int32_t inst, int32_t kind, double tau,
                             double kappa_h) {
  if (int r = check_inst(c, inst)) return r;
  if (kind != SSFM_SPECTRUM_KOLMOGOROV && kind != SSFM_SPECTRUM_STEP)
    return fail(SSFM_EINVAL, "unknown spectrum kind %d", kind);
  if (kind == SSFM_SPECTRUM_STEP &&
      (!(tau >= 0.0) || !std::isfinite(tau) || !(kappa_h > 0.0) || !std::isfinite(kappa_h)))
    return fail(SSFM_EINVAL, "step spectrum needs finite tau >= 0 and kappa_h > 0");
  ssfm_ctx::Spectrum& sp = c->spectrum[inst];
  sp.kind = kind;
  sp.tau = tau;
  sp.kappa_h = kappa_h;
  return SSFM_OK;
}

int ssfm_set_subharmonics(ssfm_ctx* c, int32_t inst, int32_t levels) {
  if (int r = check_inst(c, inst)) return r;
  if (levels < 0 || levels > kMaxSubharmonicLevels)
    return fail(SSFM_EINVAL, "subharmonic levels must be in [0, %d], got %d",
                kMaxSubharmonicLevels, levels);
  c->spectrum[inst].subharmonics = levels;
  return SSFM_OK;
}

namespace {
int check_lens(const ssfm_lens* lens) {
  if (!lens) return fail(SSFM_EINVAL, "lens is NULL");
  const ssfm_lens& l = *lens;
  if (!(l.l_dif >= 0.0) || !std::isfinite(l.l_dif) || !std::isfinite(l.w_l) ||
      !std::isfinite(l.c1) || l.c1 == 0.0 || !std::isfinite(l.c2))
    return fail(SSFM_EINVAL, "lens needs finite l_dif >= 0, w_l, c2 and c1 != 0");
  if (l.n_re < 0 || l.n_re > 8 || l.n_im < 0 || l.n_im > 8)
    return fail(SSFM_EINVAL, "lens segment counts must be in [0, 8]");
  for (int part = 0; part < 2; ++part) {
    const int n = part ? l.n_im : l.n_re;
    const double(*seg)[4] = part ? l.im : l.re;
    double lo = 0.0;
    for (int j = 0; j < n; ++j) {
      for (int k = 0; k < 4; ++k)
        if (!std::isfinite(seg[j][k])) return fail(SSFM_EINVAL, "lens segment not finite");
      if (!(seg[j][0] > lo))
        return fail(SSFM_EINVAL, "lens segment radii must increase from 0");
      lo = seg[j][0];
    }
  }
  return SSFM_OK;
}
}  // namespace

int ssfm_apply_lens(ssfm_ctx* c, int32_t inst, const ssfm_lens* lens) {
  if (int r = check_inst(c, inst)) return r;
  if (int r = lie_only(c, "the effective lens")) return r;
  if (int r = check_lens(lens)) return r;
  return SSFM_DISPATCH(c, do_apply_lens, c, inst, *lens);
}

int ssfm_lens_vjp(ssfm_ctx* c, int32_t inst, const ssfm_lens* lens, const void* u_in,
                  const void* g_out, void* g_in, double* grad, int32_t n_grad) {
  if (int r = check_inst(c, inst)) return r;
  if (int r = check_lens(lens)) return r;
  if (!u_in || !g_out || !g_in || !grad)
    return fail(SSFM_EINVAL, "u_in, g_out, g_in and grad must not be NULL");
  const int need = 2 + 3 * (lens->n_re + lens->n_im);
  if (n_grad < need)
    return fail(SSFM_EINVAL, "grad holds %d values, the lens has %d parameters", n_grad, need);
  return SSFM_DISPATCH(c, do_lens_vjp, c, inst, *lens, static_cast<const double*>(u_in),
                       static_cast<const double*>(g_out), static_cast<double*>(g_in), grad);
}

namespace {
// The result of a count whose n^2 labels start at base.
HotResult* hot_result_at(char* base, int32_t n) {
  return reinterpret_cast<HotResult*>(base + align_up(sizeof(int) * size_t(n) * n));
}

int count_hot_areas(const double* w, int32_t n, double threshold, int32_t periodic, int* labels,
                    HotResult* res, hipStream_t st, int64_t* count) {
  HIP_TRY(launch_hot_areas(w, n, threshold, periodic ? 1 : 0, labels, res, st));
  HotResult h{};
  HIP_TRY(hipMemcpyAsync(&h, res, sizeof(h), hipMemcpyDeviceToHost, st));
  HIP_TRY(hipStreamSynchronize(st));
  if (h.overflow) return fail(SSFM_EHIP, "hot-area labelling: a union exceeded its retry cap");
  *count = h.regions;
  return SSFM_OK;
}
}  // namespace

int ssfm_hot_areas(ssfm_ctx* c, const double* w, int32_t n, double threshold, int32_t periodic,
                   int64_t* count) {
  if (int r = check_ctx(c)) return r;
  if (!w || !count) return fail(SSFM_EINVAL, "w/count is NULL");
  if (n < 1 || n > c->L.max_n)
    return fail(SSFM_EINVAL, "n=%d must be in [1, %d] (the context's largest grid)", n,
                c->L.max_n);
  if (!std::isfinite(threshold)) return fail(SSFM_EINVAL, "threshold must be finite");
  // labels (n^2 ints) and the result live in the staging buffer
  return count_hot_areas(w, n, threshold, periodic, c->at<int>(c->L.stage),
                         hot_result_at(c->at<char>(c->L.stage), n), c->stream, count);
}

int ssfm_hot_areas_static(const double* w, int32_t n, double threshold, int32_t periodic,
                          void* stream, int64_t* count) {
  g_last_error.clear();
  if (!w || !count) return fail(SSFM_EINVAL, "w/count is NULL");
  if (n < 1 || n > kStaticMaxN)
    return fail(SSFM_EINVAL,
                "n=%d outside [1, %d], the static scratch's largest grid (larger grids: "
                "ssfm_hot_areas with a context)", n, kStaticMaxN);
  if (!std::isfinite(threshold)) return fail(SSFM_EINVAL, "threshold must be finite");
  void* base = nullptr;
  HIP_TRY(static_scratch(&base));
  char* sc = static_cast<char*>(base);
  return count_hot_areas(w, n, threshold, periodic, reinterpret_cast<int*>(sc),
                         reinterpret_cast<HotResult*>(sc + kStaticResultOff),
                         static_cast<hipStream_t>(stream), count);
}

namespace {
// The measure vector of an n x n device fluence w (see ssfm_measure_vector);
// the hot-area labels use the staging area's first half.
int measure(ssfm_ctx* c, const double* w, int32_t n, double length, double w_p,
            int32_t periodic, double* p) {
  constexpr int kParts = 256;
  const double dx = length / n;
  double* part = c->at<double>(c->L.sumsq_part) + kParts;
  HIP_TRY(launch_measure(w, n, dx, part, kParts, c->stream));
  std::vector<double> host(5 * kParts);
  HIP_TRY(hipMemcpyAsync(host.data(), part, sizeof(double) * host.size(), hipMemcpyDeviceToHost,
                         c->stream));
  int64_t count = 0;
  if (int r = ssfm_hot_areas(c, w, n, w_p, periodic, &count)) return r;  // synchronises
  double acc[4] = {0.0, 0.0, 0.0, 0.0}, mx = 0.0;
  for (int b = 0; b < kParts; ++b) {
    for (int k = 0; k < 4; ++k) acc[k] += host[5 * b + k];
    mx = std::max(mx, host[5 * b + 4]);
  }
  p[0] = acc[0] * dx * dx;  // Q(1, 0)
  p[1] = acc[1] * dx * dx;  // Q(1, 1)
  p[2] = acc[2] * dx * dx;  // Q(2, 0)
  p[3] = acc[3] * dx * dx;  // Q(2, 1)
  p[4] = mx;
  p[5] = double(count);
  return SSFM_OK;
}
}  // namespace

int ssfm_measure_vector(ssfm_ctx* c, const double* w, int32_t n, double length, double w_p,
                        int32_t periodic, double* p) {
  if (int r = check_ctx(c)) return r;
  if (!w || !p) return fail(SSFM_EINVAL, "w/p is NULL");
  if (n < 1 || n > c->L.max_n || !(length > 0.0) || !std::isfinite(w_p))
    return fail(SSFM_EINVAL, "need 1 <= n <= %d, length > 0, finite w_p", c->L.max_n);
  return measure(c, w, n, length, w_p, periodic, p);
}

int ssfm_measure_distance(ssfm_ctx* c, int32_t inst, double w_p, int32_t periodic,
                          const double* p0, double* d, double* p) {
  if (int r = check_inst(c, inst)) return r;
  if (!p0 || !d) return fail(SSFM_EINVAL, "p0/d is NULL");
  if (!std::isfinite(w_p)) return fail(SSFM_EINVAL, "w_p must be finite");
  const ssfm_instance_desc& desc = c->desc[inst];
  const int n = desc.n;
  // the fluence into the staging area's second half (the labels use the first)
  double* w = c->at<double>(c->L.stage) + size_t(c->L.max_n) * c->L.max_n;
  if (int r = SSFM_DISPATCH(c, read_out, c, inst, w, SSFM_DEVICE, true)) return r;
  double pv[SSFM_MEASURE_LEN];
  if (int r = measure(c, w, n, desc.length, w_p, periodic, pv)) return r;
  double acc = 0.0;
  for (int k = 0; k < SSFM_MEASURE_LEN; ++k) {
    const double s = (p0[k] != 0.0) ? std::fabs(p0[k]) : 1.0;
    const double q = (pv[k] - p0[k]) / s;
    acc += q * q;
  }
  *d = std::sqrt(acc);
  if (p)
    for (int k = 0; k < SSFM_MEASURE_LEN; ++k) p[k] = pv[k];
  return SSFM_OK;
}

int ssfm_moment(ssfm_ctx* c, const double* w, int32_t n, double length, double p, int32_t m,
                double* q) {
  if (int r = check_ctx(c)) return r;
  if (!w || !q) return fail(SSFM_EINVAL, "w/q is NULL");
  if (n < 1 || !(length > 0.0) || m < 0 || !std::isfinite(p))
    return fail(SSFM_EINVAL, "need n >= 1, length > 0, m >= 0, finite p");
  double* part = c->at<double>(c->L.sumsq_part);
  constexpr int kParts = 256;
  const double dx = length / n;
  HIP_TRY(launch_moment(w, n, dx, p, m, part, kParts, c->stream));
  double host[kParts];
  HIP_TRY(hipMemcpyAsync(host, part, sizeof(host), hipMemcpyDeviceToHost, c->stream));
  HIP_TRY(hipStreamSynchronize(c->stream));
  double total = 0.0;
  for (int k = 0; k < kParts; ++k) total += host[k];
  *q = total * dx * dx;
  return SSFM_OK;
}

int ssfm_set_pass_timing(ssfm_ctx* c, int32_t every) {
  if (int r = check_ctx(c)) return r;
  if (every < 0) return fail(SSFM_EINVAL, "every must be >= 0");
  if (every == c->timing_every) return SSFM_OK;
  HIP_TRY(hipStreamSynchronize(c->stream));
  clear_graphs(c);  // the step graphs are cut at the sampled steps
  for (auto& e : c->samples) c->free_samples.push_back(std::move(e));
  c->samples.clear();
  c->n_samples = 0;
  c->timing_every = every;
  return SSFM_OK;
}

namespace {
// Mean span of the sampled row passes and column passes: for each sample the
// earliest start to the latest stop over its size groups, which a sampled
// pass starts together and runs side by side.
int mean_spans(ssfm_ctx* c, const std::vector<ssfm_ctx::PassSample>& samples, double* row,
               double* col) {
  double acc[2] = {0.0, 0.0};
  int n[2] = {0, 0};
  if (!samples.empty()) {
    HIP_TRY(hipStreamSynchronize(c->stream));
    const size_t ng = c->groups.size();
    for (const auto& e : samples) {
      double lo = 0.0, hi = 0.0;
      for (size_t g = 0; g < ng; ++g) {
        float a = 0.f, b = 0.f;
        HIP_TRY(hipEventElapsedTime(&a, e.ev[0], e.ev[2 * g]));
        HIP_TRY(hipEventElapsedTime(&b, e.ev[0], e.ev[2 * g + 1]));
        lo = std::min(lo, double(a));
        hi = std::max(hi, double(b));
      }
      acc[e.col] += hi - lo;
      ++n[e.col];
    }
  }
  if (row) *row = n[0] ? acc[0] / n[0] : 0.0;
  if (col) *col = n[1] ? acc[1] / n[1] : 0.0;
  return SSFM_OK;
}
}  // namespace

int ssfm_pass_times(ssfm_ctx* c, double* ms_row, double* ms_col, int32_t* n_samples) {
  if (int r = check_ctx(c)) return r;
  if (n_samples) *n_samples = c->n_samples;
  return mean_spans(c, c->samples, ms_row, ms_col);
}

int ssfm_adjoint_pass_times(ssfm_ctx* c, double* ms_col, double* ms_row, int32_t* n_samples) {
  if (int r = check_ctx(c)) return r;
  if (n_samples) *n_samples = c->n_adj_samples;
  return mean_spans(c, c->adj_samples, ms_row, ms_col);
}

int ssfm_synchronize(ssfm_ctx* c) {
  if (int r = check_ctx(c)) return r;
  HIP_TRY(hipStreamSynchronize(c->stream));
  return SSFM_OK;
}

}  // extern "C"
