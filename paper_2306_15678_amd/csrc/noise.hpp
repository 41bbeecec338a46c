// noise.hpp -- the turbulence screens' random numbers (Philox4x32-10 and
// Box-Muller, FP64) and their spectrum on the FFT grid.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

#include "subharmonics.hpp"

namespace ssfm {

// Philox4x32-10 (Salmon et al., SC'11): ten rounds of two 32x32->64-bit
// multiplies, key advanced by the Weyl constants between rounds.
__device__ __forceinline__ void philox4x32_10(uint32_t c[4], uint32_t k0, uint32_t k1) {
  const uint32_t M0 = 0xD2511F53u, M1 = 0xCD9E8D57u;
  const uint32_t W0 = 0x9E3779B9u, W1 = 0xBB67AE85u;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r > 0) {
      k0 += W0;
      k1 += W1;
    }
    const uint64_t p0 = uint64_t(M0) * c[0];
    const uint64_t p1 = uint64_t(M1) * c[2];
    const uint32_t hi0 = uint32_t(p0 >> 32), lo0 = uint32_t(p0);
    const uint32_t hi1 = uint32_t(p1 >> 32), lo1 = uint32_t(p1);
    const uint32_t n0 = hi1 ^ c[1] ^ k0, n2 = hi0 ^ c[3] ^ k1;
    c[0] = n0;
    c[1] = lo1;
    c[2] = n2;
    c[3] = lo0;
  }
}

// Complex Gaussian of unit variance per part, from counter c.
__device__ __forceinline__ void gaussian_pair(uint32_t (&c)[4], uint32_t k0, uint32_t k1,
                                              double* re, double* im) {
  philox4x32_10(c, k0, k1);
  const double u1 = (double(c[0]) + 0.5) * 2.3283064365386962890625e-10;
  const double u2 = (double(c[1]) + 0.5) * 2.3283064365386962890625e-10;
  const double rr = sqrt(-2.0 * log(u1));
  double sn, cs;
  sincospi(2.0 * u2, &sn, &cs);
  *re = rr * cs;
  *im = rr * sn;
}

// x^(-11/12) for whole 1 <= x < 2^24: the FP32 estimate (relative error
// below 2e-6) and two Newton steps for y^12 x^11 = 1, whose error is 6.5
// times the last one's square (11 multiplies a step; the library's pow takes
// a hundred operations).
__device__ __forceinline__ double pow_m11_12(double x) {
  double y = double(__builtin_amdgcn_exp2f(-11.0f / 12.0f * __builtin_amdgcn_logf(float(x))));
  const double x2 = x * x, x4 = x2 * x2, x11 = x4 * x4 * x2 * x;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const double y2 = y * y, y4 = y2 * y2;
    y = fma(y * (1.0 / 12.0), fma(-(y4 * y4 * y4), x11, 1.0), y);
  }
  return y;
}

// Spectrum sample c sqrt(Phi(f)) df of pair `pair` at FFT index (row, col).
// Kolmogorov: Phi(f) df^2 = amp0^2 m^(-11/3) with m = |(signed col, signed
// row)|; step: amp0 where 0 < m^2 <= band_q2.  m^2 is an exact integer (at
// most n^2 / 2).
__device__ __forceinline__ void noise_sample(const SubBeam& sb, int n, int row, int col, int pair,
                                             double* re, double* im) {
  uint32_t c[4] = {uint32_t(col), uint32_t(row), uint32_t(pair), 0u};
  double g_re, g_im;
  gaussian_pair(c, sb.k0, sb.k1, &g_re, &g_im);
  const int mx = (col <= n / 2) ? col : col - n;
  const int my = (row <= n / 2) ? row : row - n;
  const double m2 = double(mx * mx + my * my);
  double a;
  if (sb.sp.kind == 1)
    a = (m2 > 0.0 && m2 <= sb.sp.band_q2) ? sb.amp0 : 0.0;
  else
    a = (m2 > 0.0) ? sb.amp0 * pow_m11_12(m2) : 0.0;
  *re = a * g_re;
  *im = a * g_im;
}

}  // namespace ssfm
