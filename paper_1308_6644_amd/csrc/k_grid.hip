// Spreading and interpolation for a non-uniform plane that is a uniform grid
// of its own pitch (scaled diffraction, the case NU-ASM generalises).  The
// weights psi(tx - tau_x(a)) psi(ty - tau_y(b)) of such a plane factor over
// the axes, so both operations split into two 1-D gather passes and need no
// binning at all:
//   interpolation  R[ty][a] = sum_j psi_x(a, j) G[ty][i0x(a) + j]        (x pass)
//                  u[b][a]  = sum_j psi_y(b, j) R[i0y(b) + j][a]         (y pass)
//   spreading      S[b][tx] = sum_{a: tx in taps(a)} psi(tx - tau_x(a)) c[b][a]
//                  G[ty][tx] = sum_{b: ty in taps(b)} psi(ty - tau_y(b)) S[b][tx]
// Lanes run along x in every pass, so every global access is a contiguous
// row segment.
#include <algorithm>
#include <cmath>

#include "launch.h"

namespace nuasm {

constexpr int kGridRows = 8;  // rows per wave in the passes along x

// First tap and offset (i0 - tau) of grid index k on one axis (centre c, n
// points): the rule of the binned points, clamped to the closed window.
__device__ __forceinline__ void grid_tap(const GridPts& p, int k, int n, double c, int w, int* i0, float* d) {
  double xp = (c + (double)(k - n / 2) * p.pitch) * p.inv_g;
  xp = fmin(fmax(xp, -p.half_n), p.half_n);
  const double t = 2.0 * xp + p.tau0;
  const double f = ceil(t - 0.5 * w);
  *i0 = (int)f;
  *d = (float)(f - t);
}

// Both passes of the interpolation in one kernel: a workgroup makes 64 columns
// by `rb` rows of the output.  Lane = grid column a.  x pass: the support rows
// the output rows' taps touch, interpolated along x at the lane's column, into
// LDS (row r by wave r % 4); y pass: each output row from its w rows of LDS,
// with weights and first taps evaluated once per workgroup.  The intermediate
// R never goes to memory.  The support rows are a contiguous run while the
// output rows are closer than w cells, and w rows per output row beyond that;
// grid_interp_rows picks rb so that they fit kGridLdsRows.  Bound by the cache
// reads of the x pass (w overlapping loads an element).
// 2048 x 2048 points from the 2064 x 2064 support, w = 7: 15.8 + 24.5 us as
// two launches, 22.0 as one (reads and writes 68 MB: 3.1 TB/s).
constexpr int kGridLdsRows = 48;
constexpr int kGridMaxRb = 64;

template <int W>
__global__ void __launch_bounds__(256) k_grid_interp(const float2* __restrict__ G, float2* __restrict__ out,
                                                     GridPts p, int rb, int sparse) {
  __shared__ float2 R[kGridLdsRows][64];
  __shared__ float wy[kGridMaxRb][W];
  __shared__ int iy[kGridMaxRb];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int a = blockIdx.x * 64 + lane;
  const int b0 = blockIdx.y * rb, nb = min(rb, p.ny - b0);
  // weights and first taps of the output rows, one (row, tap) pair per thread
  for (int e = t; e < nb * W; e += 256) {
    const int b = e / W, j = e - b * W;
    int i0;
    float d;
    grid_tap(p, b0 + b, p.ny, p.cy, W, &i0, &d);
    wy[b][j] = es_kernel_fast(d + (float)j, p.two_over_w, p.beta_log2e);
    if (j == 0) iy[b] = i0;
  }
  __syncthreads();
  const int r0 = iy[0];
  const int nr = min(sparse ? nb * W : iy[nb - 1] - r0 + W, kGridLdsRows);
  {
    // lanes past the last column repeat it (their result is not stored)
    int i0;
    float d;
    grid_tap(p, min(a, p.nx - 1), p.nx, p.cx, W, &i0, &d);
    float wt[W];
#pragma unroll
    for (int j = 0; j < W; ++j) wt[j] = es_kernel_fast(d + (float)j, p.two_over_w, p.beta_log2e);
    for (int r = wave; r < nr; r += 4) {
      const int ty = sparse ? iy[r / W] + r % W : r0 + r;
      const float2* row = G + (size_t)min(max(ty, 0), p.L - 1) * p.L + i0;
      float2 acc = czero();
#pragma unroll
      for (int j = 0; j < W; ++j) {
        const float2 g = row[j];
        acc.x = fmaf(wt[j], g.x, acc.x);
        acc.y = fmaf(wt[j], g.y, acc.y);
      }
      R[r][lane] = acc;
    }
  }
  __syncthreads();
  if (a >= p.nx) return;
  for (int b = wave; b < nb; b += 4) {
    const int q = min(sparse ? b * W : iy[b] - r0, kGridLdsRows - W);
    float2 acc = czero();
#pragma unroll
    for (int j = 0; j < W; ++j) {
      const float2 v = R[q + j][lane];
      acc.x = fmaf(wy[b][j], v.x, acc.x);
      acc.y = fmaf(wy[b][j], v.y, acc.y);
    }
    out[(size_t)(b0 + b) * p.nx + a] = acc;
  }
}

// Output rows per workgroup, and whether their support rows are kept apart
// (rows at least w cells apart share none).  Rows s cells apart have first
// taps at most (rb - 1) s + 1 apart.
static void grid_interp_rows(const GridPts& p, int w, int* rb, int* sparse) {
  const double s = 2.0 * p.pitch * p.inv_g;
  *sparse = s >= (double)w ? 1 : 0;
  if (*sparse) {
    *rb = kGridLdsRows / w;
    return;
  }
  const double fit = std::floor((double)(kGridLdsRows - w - 2) / s) + 1.0;
  *rb = (int)std::min<double>(kGridMaxRb, std::max(1.0, fit));
}

// Grid indices whose taps may contain support cell t on one axis: tau(k) is
// increasing in k with step s = 2 pitch / g cells, and the taps of k cover
// [ceil(tau - w/2), ceil(tau - w/2) + w), so a range widened by one index on
// each side holds them all; membership is then tested exactly.
__device__ __forceinline__ void grid_candidates(const GridPts& p, int t, int n, double c, int w, int* k0, int* k1) {
  const double s = 2.0 * p.pitch * p.inv_g;
  const double tau_first = 2.0 * ((c + (double)(0 - n / 2) * p.pitch) * p.inv_g) + p.tau0;
  const double lo = (t - 0.5 * w - tau_first) / s;
  const double hi = (t + 0.5 * w - tau_first) / s;
  *k0 = max(0, (int)floor(lo) - 1);
  *k1 = min(n - 1, (int)ceil(hi) + 1);
}

// x pass of the spreading: lane = support column tx, each wave kGridRows
// grid rows; the candidate columns and their weights are shared by the rows.
template <int W>
__global__ void __launch_bounds__(256) k_grid_spread_x(const float2* __restrict__ c, float2* __restrict__ S,
                                                       GridPts p) {
  const int tx = blockIdx.x * 64 + (threadIdx.x & 63);
  const int b0 = (blockIdx.y * 4 + (threadIdx.x >> 6)) * kGridRows;
  if (tx >= p.L || b0 >= p.ny) return;
  const int nb = min(kGridRows, p.ny - b0);
  float2 acc[kGridRows];
#pragma unroll
  for (int r = 0; r < kGridRows; ++r) acc[r] = czero();
  int k0, k1;
  grid_candidates(p, tx, p.nx, p.cx, W, &k0, &k1);
  for (int a = k0; a <= k1; ++a) {
    int i0;
    float d;
    grid_tap(p, a, p.nx, p.cx, W, &i0, &d);
    const int j = tx - i0;
    if (j < 0 || j >= W) continue;
    const float wt = es_kernel_fast(d + (float)j, p.two_over_w, p.beta_log2e);
#pragma unroll
    for (int r = 0; r < kGridRows; ++r) {
      if (r < nb) {
        const float2 v = c[(size_t)(b0 + r) * p.nx + a];
        acc[r].x = fmaf(wt, v.x, acc[r].x);
        acc[r].y = fmaf(wt, v.y, acc[r].y);
      }
    }
  }
#pragma unroll
  for (int r = 0; r < kGridRows; ++r)
    if (r < nb) S[(size_t)(b0 + r) * p.L + tx] = acc[r];
}

// y pass of the spreading: lane = support column tx, one support row ty per
// wave; every support cell is written (zero where no grid row reaches).
template <int W>
__global__ void __launch_bounds__(256) k_grid_spread_y(const float2* __restrict__ S, float2* __restrict__ G,
                                                       GridPts p) {
  const int tx = blockIdx.x * 64 + (threadIdx.x & 63);
  const int ty = blockIdx.y * 4 + (threadIdx.x >> 6);
  if (tx >= p.L || ty >= p.L) return;
  float2 acc = czero();
  int k0, k1;
  grid_candidates(p, ty, p.ny, p.cy, W, &k0, &k1);
  for (int b = k0; b <= k1; ++b) {
    int i0;
    float d;
    grid_tap(p, b, p.ny, p.cy, W, &i0, &d);
    const int j = ty - i0;
    if (j < 0 || j >= W) continue;
    const float wt = es_kernel_fast(d + (float)j, p.two_over_w, p.beta_log2e);
    const float2 v = S[(size_t)b * p.L + tx];
    acc.x = fmaf(wt, v.x, acc.x);
    acc.y = fmaf(wt, v.y, acc.y);
  }
  G[(size_t)ty * p.L + tx] = acc;
}

#define NUASM_GRID_DISPATCH_W(w, CALL) \
  switch (w) {                         \
    case 2: CALL(2); break;            \
    case 3: CALL(3); break;            \
    case 4: CALL(4); break;            \
    case 5: CALL(5); break;            \
    case 6: CALL(6); break;            \
    case 7: CALL(7); break;            \
    case 8: CALL(8); break;            \
    case 9: CALL(9); break;            \
    case 10: CALL(10); break;          \
    case 11: CALL(11); break;          \
    case 12: CALL(12); break;          \
    case 13: CALL(13); break;          \
    case 14: CALL(14); break;          \
    case 15: CALL(15); break;          \
    case 16: CALL(16); break;          \
    default: return hipErrorInvalidValue; \
  }

hipError_t launch_grid_interp(int w, const float2* fine, float2* out, const GridPts& p, hipStream_t st) {
  if (p.nx <= 0 || p.ny <= 0) return hipSuccess;
  int rb = 1, sparse = 0;
  grid_interp_rows(p, w, &rb, &sparse);
  const dim3 grid((p.nx + 63) / 64, (p.ny + rb - 1) / rb);
#define CALL(W) \
  hipLaunchKernelGGL(k_grid_interp<W>, grid, dim3(256), 0, st, fine, out, p, rb, sparse)
  NUASM_GRID_DISPATCH_W(w, CALL)
#undef CALL
  return hipGetLastError();
}

hipError_t launch_grid_spread(int w, const float2* vals, float2* S, float2* fine, const GridPts& p, hipStream_t st) {
  const dim3 gx((p.L + 63) / 64, (p.ny + 4 * kGridRows - 1) / (4 * kGridRows));
  const dim3 gy((p.L + 63) / 64, (p.L + 3) / 4);
#define CALL(W)                                                                    \
  {                                                                                \
    if (p.ny > 0 && p.nx > 0) {                                                    \
      hipLaunchKernelGGL(k_grid_spread_x<W>, gx, dim3(256), 0, st, vals, S, p);    \
      hipError_t e = hipGetLastError();                                            \
      if (e != hipSuccess) return e;                                               \
    }                                                                              \
    GridPts q = p;                                                                 \
    if (p.ny <= 0 || p.nx <= 0) q.ny = 0;                                          \
    hipLaunchKernelGGL(k_grid_spread_y<W>, gy, dim3(256), 0, st, S, fine, q);      \
  }
  NUASM_GRID_DISPATCH_W(w, CALL)
#undef CALL
  return hipGetLastError();
}

}  // namespace nuasm
