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
constexpr double kRsNear = 1e5;  // largest |z|/l summed by the shorter form of the phase
constexpr int kRsUnroll = 8;  // sources whose scalar loads are issued together

// One pair's term of the sum, w (z/r)(1 - i k r) exp(i k r)/r^2 with
// r = sqrt(rho^2 + z^2), divided by k z/z^2 (the caller multiplies the sum).
// (dx, dy) is the pair's distance over |z| and s = r/|z| = sqrt(u),
// u = 1 + dx^2 + dy^2.
//
// FAR = false, |z|/l <= kRsNear: the phase k r / (2 pi) = (|z|/l) s is formed
// in float64 and reduced by whole cycles before the float32 sine and cosine.
// s comes from the float32 estimate y0 of 1/sqrt(u) (relative error d <= 1e-7)
// by one residual correction, s0 = u y0, s = s0 + (u - s0^2) y0/2, whose error
// is 1.5 d^2 <= 1.4e-14 (1.3e-15 rms): 1.4e-9 cycles at |z|/l = 1e5, a twentieth
// of the float32 argument's own rounding.  The product with |z|/l is reduced by
// a fused multiply-add and rounds once.
// FAR = true: that product would keep too few digits, so (r - |z|)/l is formed
// without cancellation as rho^2 / (l |z| (1 + s)), 1/(1 + s) from the float32
// estimate by one Newton step, and |z|/l enters as its fraction c0.
//
// The amplitude needs float32 only.  With y = 1/s (corrected: the estimate's
// error is (u - s0^2) y0^2 / 2), z/r^3 = a3 y^3 and k z/r^2 = ak y^2, the term is
// ak y^2 ((a3/ak) y - i) (w e).
// 35 issue slots a pair where the FAR form alone took 43 (an instruction each,
// two a transcendental): 65536 x 65536 pairs 4.66 -> 3.86 ms
// (1.11e12 pairs/s, 90 % of vector issue).
template <bool FAR>
__device__ __forceinline__ void rs_add(double dx, double dy, float2 w, const RsConst& k, float& sr, float& si) {
  const double rho2 = fma(dx, dx, dy * dy);
  const double u = FAR ? 1.0 + rho2 : fma(dx, dx, fma(dy, dy, 1.0));
  const float y0f = __builtin_amdgcn_rsqf((float)u);
  const double y0 = (double)y0f;
  double cyc;
  float yf;
  if constexpr (FAR) {
    const double y = y0 * fma(-0.5 * u, y0 * y0, 1.5);
    const double d = fma(u, y, 1.0);
    double q = (double)__builtin_amdgcn_rcpf((float)d);
    q = q * fma(-d, q, 2.0);
    cyc = fma(rho2 * k.zl, q, k.c0);
    cyc -= rint(cyc);
    yf = (float)y;
  } else {
    const double s0 = u * y0;
    const double eh = fma(-s0, s0, u) * (0.5 * y0);
    const double s = s0 + eh;
    cyc = fma(k.zl, s, -rint(k.zl * s));
    yf = fmaf((float)eh, y0f * y0f, y0f);
  }
  const float2 e = cis_rev((float)cyc);
  const float y2 = yf * yf, b = k.ratio * yf;
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
  const double X = ((live ? x2[j] : 0.0) + k.ox) * k.inv_az;
  const double Y = ((live ? y2[j] : 0.0) + k.oy) * k.inv_az;
  const int64_t per = (M1 + kRsWaves - 1) / kRsWaves;
  const int64_t i0 = min(M1, (int64_t)wave * per);
  const int64_t i1 = min(M1, i0 + per);
  double accr = 0.0, acci = 0.0;
  float sr = 0.f, si = 0.f;
  auto pair = [&](double sx, double sy, float2 w) {
    rs_add<FAR>(fma(-sx, k.inv_az, X), fma(-sy, k.inv_az, Y), w, k, sr, si);
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
  if (k.zl <= kRsNear)
    hipLaunchKernelGGL(k_rs_direct<false>, dim3((unsigned)grid), dim3(64 * kRsWaves), 0, st, x1, y1, c, M1, x2, y2,
                       M2, k, out);
  else
    hipLaunchKernelGGL(k_rs_direct<true>, dim3((unsigned)grid), dim3(64 * kRsWaves), 0, st, x1, y1, c, M1, x2, y2,
                       M2, k, out);
  return hipGetLastError();
}

}  // namespace nuasm
