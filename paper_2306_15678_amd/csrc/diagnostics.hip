// diagnostics.hip -- hot-area count and spatial moments of a fluence.
//
// Hot areas (Results: a hot area is a closed region of the fluence with
// w >= w_p, N_ha their number): 4-connected components of the thresholded
// FP64 array, optionally continuing across the periodic window edge.
// Labelling is a lock-free union-find over pixel indices: parents only ever
// decrease (atomicMin), so L[x] <= x holds throughout and every walk to a
// root ends; a union retries only after lowering one of its two labels.
// It runs in two levels: one workgroup per 32 x 32 tile joins the tile's
// pixels in LDS (horizontal runs from ballots, then one union per vertical
// contact of two runs) and writes every pixel's tile root; a second launch
// joins the roots across tile edges, one union per contact.  A region's
// count needs no further pass: every union that removes a root removes one
// region, so N = tile roots - such unions, integers summed in any order.
// Bound by the chains of label reads.  One large region of a 1024^2 fluence
// took 490 us with pixel-wise unions in global memory, whose walks grow
// with the region, and passes that compressed and counted; a lens, its
// peak, count and gradient went from 1000 to 300 us with this and with the
// parallel sums of the lens gradient.
//
// Moments (Eq. (8) family): Q(p, m) = sum w^p (x^2 + y^2)^m dx^2 on the
// cell-centred grid, FP64 partial sums per block, summed on the host in
// block order.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>

#include "kernels.hpp"

// Device scratch of the allocation-free hot-area count: labels of an n x n
// grid with n <= kStaticMaxN and the result.  One copy per GPU, held until
// the process ends; host code never uses this name as an address (it stands
// for a host-side shadow): the device address comes from hipGetSymbolAddress
// in static_scratch().
static __device__ __align__(256) unsigned char scratch[ssfm::kStaticScratchBytes];

namespace ssfm {

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch[kMaxDevices] = {};
}  // namespace

hipError_t static_scratch(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (g_scratch[dev] == nullptr) {
    // with device dev current: that device's copy of the array
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch[dev] = p;
  }
  *out = g_scratch[dev];
  return hipSuccess;
}

namespace {

constexpr int kUniteCap = 1 << 22;  // far above any chain on a 4096^2 grid

__device__ __forceinline__ int load_label(const int* lab, int x) {
  return __hip_atomic_load(lab + x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Root of hot pixel x (labels only decrease along a walk).
__device__ __forceinline__ int find_root(const int* lab, int x) {
  int p = load_label(lab, x);
  while (p != x) {
    x = p;
    p = load_label(lab, x);
  }
  return x;
}

// Joins the regions of a and b; true if that removed a root.
__device__ __forceinline__ bool unite(int* lab, int a, int b, int* overflow) {
  for (int it = 0; it < kUniteCap; ++it) {
    a = find_root(lab, a);
    b = find_root(lab, b);
    if (a == b) return false;
    if (a > b) {
      const int t = a;
      a = b;
      b = t;
    }
    // link the larger root b under a; if b was no longer a root, continue
    // from its (smaller) parent
    const int old = atomicMin(lab + b, a);
    if (old == b) return true;
    b = old;
  }
  *overflow = 1;
  return false;
}

// Deterministic reduction of NV doubles over a 256-thread block (sum or
// max); valid in thread 0.  red: shared [4][NV].
template <int NV, int THREADS, bool MAX>
__device__ __forceinline__ void block_reduce_diag(double (&v)[NV], double* red) {
  for (int off = 32; off >= 1; off >>= 1)
    for (int k = 0; k < NV; ++k) {
      const double o = __shfl_xor(v[k], off, 64);
      v[k] = MAX ? fmax(v[k], o) : v[k] + o;
    }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  if (lane == 0)
    for (int k = 0; k < NV; ++k) red[wave * NV + k] = v[k];
  __syncthreads();
  if (threadIdx.x == 0)
    for (int k = 0; k < NV; ++k) {
      double t = red[k];
      for (int q = 1; q < THREADS / 64; ++q) t = MAX ? fmax(t, red[q * NV + k]) : t + red[q * NV + k];
      v[k] = t;
    }
}

__global__ void k_hot_reset(HotResult* res) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    res->regions = 0;
    res->overflow = 0;
  }
}

constexpr int kTile = 32;  // tile side

// Adds a workgroup's sum of `v` to the region count: v uniform over each of
// the 4 wavefronts, one atomic per workgroup.
__device__ __forceinline__ void add_regions(HotResult* res, int v) {
  __shared__ int sum[4];
  if ((threadIdx.x & 63) == 0) sum[threadIdx.x >> 6] = v;
  __syncthreads();
  const int t = sum[0] + sum[1] + sum[2] + sum[3];
  if (threadIdx.x == 0 && t != 0)
    atomicAdd(reinterpret_cast<unsigned long long*>(&res->regions),
              static_cast<unsigned long long>(static_cast<long long>(t)));
}

// Labels of one tile: lane l of wave w holds, in round i, pixel (8 i + 2 w +
// l / 32, l mod 32).
__global__ void __launch_bounds__(256) k_hot_tile(const double* __restrict__ w, int n, double thr,
                                                  int* __restrict__ lab, HotResult* res) {
  __shared__ int tl[kTile * kTile];
  __shared__ uint32_t mask[kTile];
  const int x0 = int(blockIdx.x) * kTile, y0 = int(blockIdx.y) * kTile;
  const int lane = int(threadIdx.x) & 63, wave = int(threadIdx.x) >> 6;
  const int col = lane & 31, half = lane >> 5;
  uint32_t m[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = 8 * i + 2 * wave + half;
    const int x = x0 + col, y = y0 + row;
    const bool hot = x < n && y < n && w[int64_t(y) * n + x] >= thr;
    const uint64_t b = __ballot(hot);
    m[i] = half ? uint32_t(b >> 32) : uint32_t(b);
    if (col == 0) mask[row] = m[i];
    // run start: the pixel after the last cold one below col
    const uint32_t cold = ~m[i] & ((1u << col) - 1u);
    const int start = 32 - __clz(cold);
    if (hot) tl[row * kTile + col] = row * kTile + start;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = 8 * i + 2 * wave + half;
    if (row == 0) continue;
    // contacts with the row above, each at its first pixel
    const uint32_t both = m[i] & mask[row - 1];
    if (((both & ~(both << 1)) >> col) & 1u) {
      int a = (row - 1) * kTile + col, b = row * kTile + col;
      for (;;) {  // ends: each turn lowers b or joins the two
        int p;
        while ((p = __hip_atomic_load(tl + a, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) != a) a = p;
        while ((p = __hip_atomic_load(tl + b, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP)) != b) b = p;
        if (a == b) break;
        if (a > b) {
          const int t = a;
          a = b;
          b = t;
        }
        const int old = atomicMin(tl + b, a);
        if (old == b) break;
        b = old;
      }
    }
  }
  __syncthreads();
  int roots = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int row = 8 * i + 2 * wave + half;
    const int x = x0 + col, y = y0 + row;
    const bool hot = (m[i] >> col) & 1u;
    int r = row * kTile + col;
    if (hot) {
      int p;
      while ((p = tl[r]) != r) r = p;
    }
    roots += __popcll(__ballot(hot && r == row * kTile + col));
    if (x < n && y < n)
      lab[int64_t(y) * n + x] = hot ? (y0 + r / kTile) * n + x0 + r % kTile : -1;
  }
  add_regions(res, roots);
}

// Unions across tile edges.  Item (edge e, position q): the pixels on both
// sides of the edge at q, vertical edges first; edge 0 is the window's wrap
// (periodic only).  A contact that continues one at q - 1 within the same
// tiles is joined already.
__global__ void __launch_bounds__(256) k_hot_edges(int* lab, int n, int edges, int periodic,
                                                   HotResult* res) {
  const int64_t items = 2 * int64_t(edges) * n;
  int joined = 0;
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < items;
       i += int64_t(gridDim.x) * blockDim.x) {
    const bool horizontal = i >= int64_t(edges) * n;
    const int64_t k = horizontal ? i - int64_t(edges) * n : i;
    const int e = int(k / n), q = int(k - int64_t(e) * n);
    if (e == 0 && !periodic) continue;
    const int hi = e * kTile, lo = (e == 0) ? n - 1 : hi - 1;
    const int64_t step = horizontal ? 1 : n, across = horizontal ? n : 1;
    const int64_t a = lo * across + q * step, b = hi * across + q * step;
    if (load_label(lab, int(a)) < 0 || load_label(lab, int(b)) < 0) continue;
    if (q % kTile != 0 && load_label(lab, int(a - step)) >= 0 && load_label(lab, int(b - step)) >= 0)
      continue;
    if (unite(lab, int(a), int(b), &res->overflow)) ++joined;
  }
  for (int o = 32; o > 0; o >>= 1) joined += __shfl_xor(joined, o);
  add_regions(res, -joined);
}

__global__ void __launch_bounds__(256) k_moment(const double* __restrict__ w, int n, double dx,
                                                double p, int m, double* part) {
  __shared__ double red[4];
  const int64_t n2 = int64_t(n) * n;
  const bool p1 = (p == 1.0), p2 = (p == 2.0);
  double s = 0.0;
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n2;
       i += int64_t(gridDim.x) * blockDim.x) {
    const int y = int(i / n), x = int(i - int64_t(y) * n);
    const double xc = (x + 0.5 - n / 2.0) * dx, yc = (y + 0.5 - n / 2.0) * dx;
    const double r2 = xc * xc + yc * yc;
    double rm = 1.0;
    for (int k = 0; k < m; ++k) rm *= r2;
    const double wi = w[i];
    const double wp = p1 ? wi : (p2 ? wi * wi : pow(wi, p));
    s += wp * rm;
  }
  for (int o = 32; o > 0; o >>= 1) s += __shfl_xor(s, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) part[blockIdx.x] = red[0] + red[1] + red[2] + red[3];
}

// Per-block FP64 partials of the measure vector's sums over an n x n
// fluence: [sum w, sum w r^2, sum w^2, sum w^2 r^2, max w] (grid-stride,
// then a fixed tree per block).
__global__ void __launch_bounds__(256) k_measure(const double* __restrict__ w, int n, double dx,
                                                 double* part) {
  __shared__ double red[4 * 5];
  const int64_t n2 = int64_t(n) * n;
  double s[4] = {0.0, 0.0, 0.0, 0.0}, mx[1] = {0.0};
  for (int64_t i = blockIdx.x * int64_t(blockDim.x) + threadIdx.x; i < n2;
       i += int64_t(gridDim.x) * blockDim.x) {
    const int y = int(i / n), x = int(i - int64_t(y) * n);
    const double xc = (x + 0.5 - n / 2.0) * dx, yc = (y + 0.5 - n / 2.0) * dx;
    const double r2 = xc * xc + yc * yc;
    const double wi = w[i], w2 = wi * wi;
    s[0] += wi;
    s[1] += wi * r2;
    s[2] += w2;
    s[3] += w2 * r2;
    mx[0] = fmax(mx[0], wi);
  }
  block_reduce_diag<4, 256, false>(s, red);
  block_reduce_diag<1, 256, true>(mx, red + 16);
  if (threadIdx.x == 0) {
    for (int k = 0; k < 4; ++k) part[5 * blockIdx.x + k] = s[k];
    part[5 * blockIdx.x + 4] = mx[0];
  }
}

}  // namespace

hipError_t launch_measure(const double* w, int n, double dx, double* part, int n_part,
                          hipStream_t s) {
  hipLaunchKernelGGL(k_measure, dim3(n_part), dim3(256), 0, s, w, n, dx, part);
  return hipGetLastError();
}

hipError_t launch_hot_areas(const double* w, int n, double threshold, int periodic, int* labels,
                            HotResult* res, hipStream_t s) {
  const int edges = (n + kTile - 1) / kTile;
  const int64_t items = 2 * int64_t(edges) * n;
  hipLaunchKernelGGL(k_hot_reset, dim3(1), dim3(64), 0, s, res);
  hipLaunchKernelGGL(k_hot_tile, dim3(edges, edges), dim3(256), 0, s, w, n, threshold, labels, res);
  hipLaunchKernelGGL(k_hot_edges, dim3(int(std::min<int64_t>((items + 255) / 256, 4096))),
                     dim3(256), 0, s, labels, n, edges, periodic, res);
  return hipGetLastError();
}

hipError_t launch_moment(const double* w, int n, double dx, double p, int m, double* part,
                         int n_part, hipStream_t s) {
  hipLaunchKernelGGL(k_moment, dim3(n_part), dim3(256), 0, s, w, n, dx, p, m, part);
  return hipGetLastError();
}

}  // namespace ssfm
