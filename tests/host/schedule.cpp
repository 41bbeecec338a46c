// The host side of libssfm on a machine without a GPU: csrc/ssfm.cpp linked
// with the HIP calls and kernel launches below, which copy host memory,
// count, and keep what is ordered before what (a vector clock per stream,
// carried by events; a wait of the host orders all that follows).  Kernels
// compute nothing.  Exit status 0 when every check holds.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>
#include <vector>

#include "internal.hpp"
#include "kernels.hpp"
#include "lens_vjp.hpp"
#include "ssfm.h"
#include "subharmonics.hpp"

using namespace ssfm;

namespace {

int g_fail = 0;
void expect(bool ok, const char* what, int line) {
  if (ok) return;
  std::fprintf(stderr, "schedule: line %d: %s (last error: %s)\n", line, what, ssfm_last_error());
  ++g_fail;
}
#define EXPECT(c) expect((c), #c, __LINE__)

using Clock = std::map<hipStream_t, int>;  // launches of each stream known to have ended
void join(Clock& a, const Clock& b) {
  for (const auto& kv : b) a[kv.first] = std::max(a[kv.first], kv.second);
}

struct Pass {
  int kind, n, at;  // at: index among its stream's launches
  bool timed;
  int32_t flags;
  int64_t step;
  hipStream_t stream;
  Clock before;  // what its start waits for
};

struct World {
  std::map<hipStream_t, Clock> streams;
  std::map<hipEvent_t, Clock> events;
  Clock host;
  std::vector<Pass> passes;
  int graphs = 0;                       // instantiated
  int copies = 0;                       // hipMemcpyAsync
  int puts = 0;                         // uploads of table entries by themselves
  hipStream_t captured = nullptr;       // a stream that its caller captures
  intptr_t next = 0x1000;
} W;

void* fresh() { return reinterpret_cast<void*>(W.next += 16); }

int launched(hipStream_t s) {
  Clock& c = W.streams[s];
  join(c, W.host);
  return ++c[s];
}

// whether pass a has ended when pass b starts
bool ends_before(const Pass& a, const Pass& b) {
  auto it = b.before.find(a.stream);
  return it != b.before.end() && it->second >= a.at;
}

}  // namespace

// ------------------------------------------------------------ HIP runtime
extern "C" {
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
  *s = static_cast<hipStream_t>(fresh());
  return hipSuccess;
}
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) {
  join(W.host, W.streams[s]);
  return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  join(W.streams[s], W.events[e]);
  return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) {
  *e = static_cast<hipEvent_t>(fresh());
  return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  W.events[e] = W.streams[s];
  join(W.events[e], W.host);
  return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) {
  *ms = 1.0f;
  return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t st) {
  launched(st);
  ++W.copies;
  std::memcpy(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t st) {
  launched(st);
  std::memset(d, v, n);
  return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t s, hipStreamCaptureStatus* st) {
  *st = (s == W.captured && s) ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipSuccess; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g) {
  *g = static_cast<hipGraph_t>(fresh());
  return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t, hipGraphNode_t*, char*, size_t) {
  ++W.graphs;
  *x = static_cast<hipGraphExec_t>(fresh());
  return hipSuccess;
}
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t s) {
  launched(s);
  return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
}

// ---------------------------------------------------------------- kernels
namespace ssfm {
int plan_default(bool, int, bool) { return 0; }
int plan_count(bool, int) { return 2; }
bool plan_info(bool, int n, int v, bool, PlanInfo* o) {
  *o = PlanInfo{};
  o->threads = 64;
  o->lines = v + 1;
  o->waves = 1;
  o->t = 64;
  o->radices[0] = n;
  return v >= 0 && v < 2;
}
template <typename R>
hipError_t launch_pass(int kind, int n, int, const PassArgs<R>& a, hipStream_t s,
                       const LaunchEv* ev) {
  launched(s);
  const Clock& c = W.streams[s];
  Pass p{kind, n, c.at(s), ev != nullptr, a.flags, a.step, s, c};
  p.before[s] = p.at - 1;
  W.passes.push_back(p);
  return hipSuccess;
}
hipError_t one(hipStream_t s) {
  launched(s);
  return hipSuccess;
}
#define STUB(R)                                                                                 \
  template hipError_t launch_pass<R>(int, int, int, const PassArgs<R>&, hipStream_t,           \
                                     const LaunchEv*);                                         \
  template <>                                                                                  \
  hipError_t launch_load_field<R>(const double*, void*, int64_t, double, const InstDev& e,     \
                                  InstDev* slot, hipStream_t s) {                              \
    *slot = e;                                                                                 \
    return one(s);                                                                             \
  }                                                                                            \
  template <>                                                                                  \
  hipError_t launch_store_field<R>(const void*, const InstDev*, int, int, const R*,            \
                                   const int64_t*, int64_t, double, double*, bool,             \
                                   hipStream_t s) {                                            \
    return one(s);                                                                             \
  }                                                                                            \
  template <>                                                                                  \
  hipError_t launch_seed<R>(int, const void*, const InstDev*, int, int, const R*,              \
                            const int64_t*, int64_t, const double*, const double*,             \
                            const double*, double, void*, double*, double*, int,               \
                            hipStream_t s) {                                                   \
    return one(s);                                                                             \
  }                                                                                            \
  template <>                                                                                  \
  hipError_t launch_copy<R>(const void*, void*, int64_t, hipStream_t s) { return one(s); }     \
  template <>                                                                                  \
  hipError_t launch_flush<R>(void*, const InstDev*, int, int, const R*, const int64_t*,        \
                             int64_t, hipStream_t s) {                                         \
    return one(s);                                                                             \
  }                                                                                            \
  template <>                                                                                  \
  hipError_t launch_mismatch<R>(const void*, const InstDev*, int, int, const R*,               \
                                const int64_t*, int64_t, const double*, double, double*,       \
                                hipStream_t s) {                                               \
    return one(s);                                                                             \
  }                                                                                            \
  template <>                                                                                  \
  hipError_t launch_screen_to_f64<R>(const R*, int64_t, double*, hipStream_t s) {              \
    return one(s);                                                                             \
  }                                                                                            \
  template <>                                                                                  \
  hipError_t launch_lens_prep<R>(const void*, void*, int64_t, hipStream_t s) { return one(s); } \
  template <>                                                                                  \
  hipError_t launch_lens_apply<R>(void*, const void*, int64_t, const LensDev&, hipStream_t s) { \
    return one(s);                                                                             \
  }                                                                                            \
  template <>                                                                                  \
  hipError_t launch_lens_vjp_prep<R>(const double*, double, void*, int64_t, hipStream_t s) {   \
    return one(s);                                                                             \
  }                                                                                            \
  template <>                                                                                  \
  hipError_t launch_lens_vjp_point<R>(const double*, const double*, void*, double*, int64_t,   \
                                      const LensDev&, double*, hipStream_t s) {                \
    return one(s);                                                                             \
  }                                                                                            \
  template <>                                                                                  \
  hipError_t launch_lens_vjp_final<R>(const double*, const void*, double, double*, int64_t,    \
                                      double*, double*, hipStream_t s) {                       \
    return one(s);                                                                             \
  }
STUB(float)
STUB(double)
template <typename T>
hipError_t launch_put(const T* src, int count, T* dst, hipStream_t s) {
  ++W.puts;
  std::copy(src, src + count, dst);
  return one(s);
}
template hipError_t launch_put<InstDev>(const InstDev*, int, InstDev*, hipStream_t);
template hipError_t launch_put<SubBeam>(const SubBeam*, int, SubBeam*, hipStream_t);
hipError_t launch_diag_finalize(const double*, int64_t, const int32_t*, const int32_t*, int, int,
                                int, double*, int64_t, int64_t, hipStream_t s) {
  return one(s);
}
hipError_t launch_reduce_theta(const double*, const int32_t*, const double*, const int32_t*, int,
                               double*, hipStream_t s) {
  return one(s);
}
hipError_t launch_sumsq(const double*, int64_t, double*, hipStream_t s) { return one(s); }
hipError_t launch_fill_f64(double*, int64_t, double, hipStream_t s) { return one(s); }
hipError_t launch_hot_areas(const double*, int, double, int, int*, HotResult*, hipStream_t s) {
  return one(s);
}
hipError_t launch_moment(const double*, int, double, double, int, double*, int, hipStream_t s) {
  return one(s);
}
hipError_t launch_measure(const double*, int, double, double*, int, hipStream_t s) {
  return one(s);
}
hipError_t launch_block_mean(const double*, int, int, double*, hipStream_t s) { return one(s); }
hipError_t launch_subharmonic_setup(const SubBeam*, int, int, int64_t, double*, hipStream_t s) {
  return one(s);
}
int lens_vjp_blocks(int64_t) { return 1; }
hipError_t static_scratch(void**) { return hipErrorInvalidValue; }
}  // namespace ssfm

// ----------------------------------------------------------------- checks
namespace {

ssfm_instance_desc beam(int n, uint32_t terms, int n_screens) {
  ssfm_instance_desc d;
  std::memset(&d, 0, sizeof(d));
  d.n = n;
  d.mpa_order = 8;
  d.terms = terms;
  d.n_screens = n_screens;
  d.length = 8e-3;
  d.dz = 0.1;
  d.wavelength = 800e-9;
  d.n2 = 3.2e-23;
  d.beta_k = 1e-120;
  d.i_ref = 5e17;
  d.cn2 = 1e-14;
  d.screen_dz = 0.3;
  d.seed = 1234;
  return d;
}

struct Context {
  ssfm_ctx* c = nullptr;
  void* ws = nullptr;
  hipStream_t stream = static_cast<hipStream_t>(fresh());
  std::vector<double> field = std::vector<double>(2 * 512 * 512, 1.0);
  Context(const std::vector<ssfm_instance_desc>& d, int64_t max_steps, int ckpt) {
    size_t bytes = 0;
    EXPECT(ssfm_workspace_bytes(d.data(), int32_t(d.size()), SSFM_FP32, max_steps, ckpt, 0,
                                &bytes) == SSFM_OK);
    ws = std::aligned_alloc(256, (bytes + 255) / 256 * 256);
    EXPECT(ssfm_create(d.data(), int32_t(d.size()), SSFM_FP32, max_steps, ckpt, 0, ws, bytes,
                       stream, &c) == SSFM_OK);
  }
  ~Context() {
    ssfm_destroy(c);
    std::free(ws);
  }
  void set(int i) { EXPECT(ssfm_set_field(c, i, field.data(), SSFM_HOST) == SSFM_OK); }
};

// Fields and parameters are refused while the context's stream is captured.
void captured() {
  Context x({beam(128, SSFM_KERR, 0)}, 0, 1);
  double theta[8] = {0.1};
  x.set(0);
  W.captured = x.stream;
  EXPECT(ssfm_set_theta(x.c, 0, theta) == SSFM_EHIP);
  EXPECT(ssfm_set_field(x.c, 0, x.field.data(), SSFM_HOST) == SSFM_EHIP);
  W.captured = nullptr;
  EXPECT(ssfm_set_theta(x.c, 0, theta) == SSFM_OK);
  x.set(0);
}

// The sampled passes among those of the given kinds, the k-th of each size
// being of one step.
void check_samples(std::vector<int> kinds, bool any) {
  std::map<int, std::vector<Pass>> by_size;
  for (const Pass& p : W.passes)
    if (std::find(kinds.begin(), kinds.end(), p.kind) != kinds.end()) by_size[p.n].push_back(p);
  EXPECT(by_size.size() == 3);
  size_t seen = 0;
  for (const auto& own : by_size)
    for (size_t k = 0; k < own.second.size(); ++k) {
      const Pass& p = own.second[k];
      if (!p.timed) continue;
      ++seen;
      for (const auto& other : by_size) {
        EXPECT(other.second[k].timed);
        for (size_t j = 0; j < k; ++j) EXPECT(ends_before(other.second[j], p));
      }
    }
  EXPECT((seen > 0) == any);
}

// The sampled passes of several grid sizes start together: each after the
// passes before it of every size, so that their spans are those of one pass.
void samples() {
  for (int every : {1, 2, 3})
    for (int ckpt : {1, 2, 6})
      for (int overlap : {0, 1})
        for (int scheme : {SSFM_LIE, SSFM_STRANG}) {
          Context x({beam(512, SSFM_KERR, 0), beam(128, SSFM_KERR, 0), beam(256, SSFM_KERR, 0)}, 6,
                    ckpt);
          EXPECT(ssfm_set_splitting(x.c, scheme) == SSFM_OK);
          EXPECT(ssfm_set_recompute_overlap(x.c, overlap) == SSFM_OK);
          EXPECT(ssfm_set_pass_timing(x.c, every) == SSFM_OK);
          for (int i = 0; i < 3; ++i) x.set(i);
          EXPECT(ssfm_use_graphs(x.c, 0) == SSFM_OK);
          W.passes.clear();
          EXPECT(ssfm_forward_record(x.c, 6) == SSFM_OK);
          check_samples({ROW_FWD, COL_FWD}, true);
          for (int i = 0; i < 3; ++i)
            EXPECT(ssfm_set_cotangent(x.c, i, x.field.data(), SSFM_HOST) == SSFM_OK);
          W.passes.clear();
          EXPECT(ssfm_backward(x.c) == SSFM_OK);
          // adjoint samples come from the first segment
          check_samples({ROW_ADJ, COL_ADJ}, every / 2 < ckpt);
        }
}

// Beams set at different steps in a repeating pattern: the marches of the
// second time round are those captured the first time, and marches whose
// turbulence screens fall on other passes have graphs of their own.
void graphs() {
  for (uint32_t turbulence : {0u, uint32_t(SSFM_TURB)}) {
    W.graphs = 0;
    Context x({beam(128, SSFM_KERR | turbulence, 3), beam(256, SSFM_KERR | turbulence, 3)}, 4, 4);
    for (int turn = 0; turn < 3; ++turn)
      for (int again : {0, 1}) {
        x.set(0);
        x.set(1);
        EXPECT(ssfm_propagate(x.c, 4) == SSFM_OK);
        x.set(again);
        EXPECT(ssfm_propagate(x.c, 4) == SSFM_OK);
      }
    EXPECT(W.graphs == (turbulence ? 3 : 2));
  }
}

// Passes launched outside the library's own graphs, which a caller may
// capture and replay after setting fields at other steps, look for their
// turbulence screens on the device.
void planes() {
  Context x({beam(128, SSFM_KERR | SSFM_TURB, 1), beam(256, SSFM_KERR, 0)}, 0, 1);
  EXPECT(ssfm_use_graphs(x.c, 0) == SSFM_OK);
  x.set(0);
  x.set(1);
  W.passes.clear();
  EXPECT(ssfm_propagate(x.c, 6) == SSFM_OK);
  for (const Pass& p : W.passes)
    EXPECT(bool(p.flags & PASS_PLANE) == (p.n == 128 && (p.flags & PASS_SCREEN)));
}

// Setting fields again before any step changes no start step: each call loads
// its field with its own entry and nothing else.
void entries() {
  Context x(std::vector<ssfm_instance_desc>(64, beam(128, SSFM_KERR, 0)), 0, 1);
  for (int i = 0; i < 64; ++i) x.set(i);
  W.puts = 0;
  for (int i = 0; i < 64; ++i) x.set(i);
  EXPECT(W.puts == 0);
  EXPECT(ssfm_propagate(x.c, 2) == SSFM_OK);
  for (int i = 0; i < 64; ++i) x.set(i);
  EXPECT(W.puts == 1);  // the restart of the step count, with the last beam
}

// A context's tables reach the device in one copy, whatever its sizes.
void create() {
  Context one({beam(128, SSFM_KERR, 0)}, 0, 1);
  EXPECT(W.copies == 1);
  W.copies = 0;
  Context four({beam(512, SSFM_TURB, 2), beam(128, 0, 0), beam(256, 0, 0), beam(128, 0, 0)}, 4, 2);
  EXPECT(W.copies == 1);
}
}  // namespace

int main(int argc, char** argv) {
  const std::string only = argc > 1 ? argv[1] : "";
  const std::pair<const char*, void (*)()> checks[] = {
      {"captured", captured},
      {"samples", samples},
      {"graphs", graphs},
      {"planes", planes},
      {"entries", entries},
      {"create", create},
  };
  for (const auto& c : checks)
    if (only.empty() || only == c.first) {
      W = World{};
      c.second();
    }
  if (g_fail) {
    std::fprintf(stderr, "schedule: %d checks failed\n", g_fail);
    return 1;
  }
  std::printf("schedule: all checks passed\n");
  return 0;
}
