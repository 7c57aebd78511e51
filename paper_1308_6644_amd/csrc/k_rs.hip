// Rayleigh-Sommerfeld diffraction by direct summation over point pairs
// (Eq. 10 with the integral over the source replaced by a weighted sum), the
// accuracy reference the paper measures NU-ASM and NU-FRE against.  O(M1 M2)
// and bound by the vector ALUs: every pair costs a square root, a sine and a
// cosine, and a float64 phase.
//
// Work split on gfx950: one workgroup holds 64 destinations (one per lane)
// and eight waves; each wave sums an eighth of the sources, read with scalar
// loads (every lane of a wave needs the same source at the same time, so the
// source stream costs no LDS and no vector memory traffic), and the eight
// partial sums meet in LDS at the end.
#include "launch.h"

namespace nuasm {

constexpr int kRsWaves = 8;   // waves per workgroup, each over an eighth of the sources
constexpr int kRsBlock = 64;  // sources per float32 partial sum (then added in float64)
constexpr int kRsUnroll = 8;  // sources whose scalar loads are issued together

// One pair's term of the sum, w (z/r)(1 - i k r) exp(i k r)/r^2, up to the
// factor that the caller multiplies the sum by.  Lengths are in units of 1/p, p
// the power of two that brings |z| into [1/2, 1) as zs (scaling by it is
// exact): (dx, dy) is the pair's distance, R = sqrt(zs^2 + dx^2 + dy^2).
// Either way the phase is |z|/l, reduced to c0 on the host, plus the path
// difference (r - |z|)/l, which is formed in float64 without cancellation and
// reduced by whole cycles before the float32 sine and cosine.
//
// FAR = false, |z|/l <= kRsNear: with y0, the float32 estimate of 1/R (relative
// error d, at most 2e-7), R2 y0 - zs is the path difference D up to d R, the
// residual e = rho^2 - D (D + 2 zs) holds the rest to the last digit, and
// h = e y0 / 2 corrects it to 1.5 d^2 R, which the float32 term 1.5 h^2 y0 takes
// to d^3 R.  Error: a few 2^-53 of the path difference and 3e-20 |z|/l; emulated
// on the CPU, |z|/l from 20 to 1e5 and windows of 0.1 mm to 4 m: 2e-16 of the
// path difference at most, where the FAR form has 3e-14.
// FAR = true, in units of |z|: D = rho^2 / (1 + s), s = R = sqrt(1 + rho^2), from
// the estimates of 1/s and of 1/(1 + s) by a Newton step each (1e-14 of D).  It
// stays below the d^3 term where |z|/l is large and the path difference small
// (|z|/l = 2e8, a window of 1 mm: 2e-16 cycles, and 6e-12 by the other).
//
// The amplitude needs float32 only.  With y = 1/R (its square corrected by h),
// z/r^3 = a3 y^3 and k z/r^2 = ak y^2, the term is ak y^2 ((a3/ak) y - i) (w e).
// 65536 x 65536 pairs: 4.66 ms with the FAR form and the amplitude as separate
// products, 3.83 with (|z|/l) s in the place of the path difference, whose error
// is 1e-14 of |z|/l (1e-9 cycles at 1e5), 4.14 so (1.04e12 pairs/s).
template <bool FAR>
__device__ __forceinline__ void rs_add(double dx, double dy, float2 w, const RsConst& k, float& sr, float& si) {
  const double rho2 = fma(dx, dx, dy * dy);
  float cycf, y, y2;  // y: 1/R, and its square
  if constexpr (FAR) {
    const double u = fma(rho2, k.inv_zs2, 1.0);
    double v = (double)__builtin_amdgcn_rsqf((float)u);
    v = v * fma(-0.5 * u, v * v, 1.5);
    const double d = fma(u, v, 1.0);
    double q = (double)__builtin_amdgcn_rcpf((float)d);
    q = q * fma(-d, q, 2.0);
    const double cyc = fma(rho2 * k.inv_lz, q, k.c0);
    cycf = (float)(cyc - rint(cyc));
    y = (float)v;
    y2 = y * y;
  } else {
    const double R2 = rho2 + k.zs2;
    y = __builtin_amdgcn_rsqf((float)R2);
    const double y0 = (double)y;
    const double D0 = fma(R2, y0, -k.zs);
    const double h2 = fma(-D0, D0 + k.two_zs, rho2) * y0;  // 2 h
    const double cyc = fma(fma(0.5, h2, D0), k.inv_l, k.c0);
    const float h2f = (float)h2, t = h2f * y;
    cycf = fmaf(k.corr * h2f, t, (float)(cyc - rint(cyc)));
    y2 = y * y;
    y2 = fmaf(t, y2, y2);
  }
  const float2 e = cis_rev(cycf);
  const float b = k.ratio * y;
  // P = w e; P (b - i) = (P.x b + P.y, P.y b - P.x)
  const float pr = fmaf(w.x, e.x, -(w.y * e.y)), pi = fmaf(w.x, e.y, w.y * e.x);
  sr = fmaf(fmaf(pr, b, pi), y2, sr);
  si = fmaf(fmaf(pi, b, -pr), y2, si);
}

template <bool FAR>
__global__ void __launch_bounds__(64 * kRsWaves)
k_rs_direct(const double* __restrict__ x1, const double* __restrict__ y1, const float2* __restrict__ c,
            int64_t M1, const double* __restrict__ x2, const double* __restrict__ y2, int64_t M2, RsConst k,
            float2* __restrict__ out) {
  __shared__ double2 part[kRsWaves][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t j = (int64_t)blockIdx.x * 64 + lane;
  const bool live = j < M2;
  const double X = ((live ? x2[j] : 0.0) + k.ox) * k.p;
  const double Y = ((live ? y2[j] : 0.0) + k.oy) * k.p;
  const int64_t per = (M1 + kRsWaves - 1) / kRsWaves;
  const int64_t i0 = min(M1, (int64_t)wave * per);
  const int64_t i1 = min(M1, i0 + per);
  double accr = 0.0, acci = 0.0;
  float sr = 0.f, si = 0.f;
  auto pair = [&](double sx, double sy, float2 w) {
    rs_add<FAR>(fma(-sx, k.p, X), fma(-sy, k.p, Y), w, k, sr, si);
  };
  int64_t i = i0;
  // full groups of kRsUnroll sources: their scalar loads are issued together
  // ahead of the arithmetic; the float32 partial sums go into float64 every
  // kRsBlock sources
  int n = 0;
  for (; i + kRsUnroll <= i1; i += kRsUnroll) {
    double sx[kRsUnroll], sy[kRsUnroll];
    float2 sw[kRsUnroll];
#pragma unroll
    for (int u = 0; u < kRsUnroll; ++u) {
      sx[u] = x1[i + u];
      sy[u] = y1[i + u];
      sw[u] = c[i + u];
    }
#pragma unroll
    for (int u = 0; u < kRsUnroll; ++u) pair(sx[u], sy[u], sw[u]);
    if (++n == kRsBlock / kRsUnroll) {
      accr += (double)sr;
      acci += (double)si;
      sr = si = 0.f;
      n = 0;
    }
  }
  for (; i < i1; ++i) pair(x1[i], y1[i], c[i]);
  accr += (double)sr;
  acci += (double)si;
  part[wave][lane] = make_double2(accr, acci);
  __syncthreads();
  if (wave == 0 && live) {
    double r = 0.0, i = 0.0;
#pragma unroll
    for (int w = 0; w < kRsWaves; ++w) {
      r += part[w][lane].x;
      i += part[w][lane].y;
    }
    out[j] = make_float2((float)(r * k.scale), (float)(i * k.scale));
  }
}

hipError_t launch_rs_direct(const double* x1, const double* y1, const float2* c, int64_t M1, const double* x2,
                            const double* y2, int64_t M2, const RsConst& k, float2* out, hipStream_t st) {
  if (M2 <= 0) return hipSuccess;
  const int64_t grid = (M2 + 63) / 64;
  if (!k.far)
    hipLaunchKernelGGL(k_rs_direct<false>, dim3((unsigned)grid), dim3(64 * kRsWaves), 0, st, x1, y1, c, M1, x2, y2,
                       M2, k, out);
  else
    hipLaunchKernelGGL(k_rs_direct<true>, dim3((unsigned)grid), dim3(64 * kRsWaves), 0, st, x1, y1, c, M1, x2, y2,
                       M2, k, out);
  return hipGetLastError();
}

}  // namespace nuasm
