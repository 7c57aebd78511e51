// Grid passes of the two pipelines on gfx950: pruned row FFTs, the fused
// column pass (FFT -> deconvolution x transfer function x Rect -> inverse FFT),
// and the final row passes.  Data stay in registers between the LDS exchanges
// of a transform (reg_fft); HBM is touched once per pass.
//
// Index conventions (centred, as in Eqs. 3, 6 and 9): a plane element [b][a]
// of an N' x N' array holds n = (a - N'/2, b - N'/2); frequency k = a - N'/2.
// The non-uniform sums run on the spectral grid K'' of N'' modes (N'' = N',
// or smaller when the band of Eq. 4 is narrow) and a fine grid of nf = 2 N''
// cells per axis; the non-uniform window occupies fine cells
// [N''/2, 3N''/2), and only the support rows/columns [s0, s0 + L),
// L = N'' + 16, are ever stored.
//
// Half-length transforms.  Every transform of the fine grid has half its
// cells (but for the 16 cells of margin) or half its modes empty, and so has
// the transform of a zero-padded N x N plane: a transform of length 2 n is run
// as two of length n, of the even and of the odd outputs (reg_fft, HALF), one
// after the other in half the LDS, which leaves room for twice the rows or
// columns in a workgroup.
//
// Intermediate layout.  Between a row pass and a column pass the array is
// stored in strips of 2^cs columns, the column pass's own: element (row, col)
// of an array of R rows at ((col >> cs) R + row) 2^cs + col mod 2^cs.  A column
// workgroup then reads and writes one contiguous block, and a row workgroup of
// C rows segments of C 2^cs elements, where row-major columns of one or two
// elements had cost a 64-byte request each.  Before (full-length transforms in
// LDS, row-major arrays, in-band strips alone launched) and now, us a launch:
//   N' = 2048, half the columns in band  t1_cols  27.5  23.8   t1_rows      17.0  18.6
//   N' = 2048, all columns               t2_cols  38.2  30.3   t2_rows_inv  18.9  19.3
//                                        t3_cols  ~38   27.4   t1_rows_inv  16.0  14.1
//   N' = 4096, 2522 columns              t1_cols 168.5  61.2   t1_rows      74.3  73.0
//                                        t2_cols 134.5  64.1   t2_rows_inv  76.3  89.1
//   N' = 8192, N'' = 2048, 2020 columns  t2_cols  91.5  48.8   t2_rows      75.4  79.3
// The passes are bound by vector instruction issue (about 70 % at N' = 2048)
// and the latency of their exchanges; the largest by cache requests.
#include <algorithm>

#include "group.h"
#include "launch.h"

namespace nuasm {

// Row passes: C rows per workgroup by transforms of length 2^LOG, eight
// elements a thread; TL: log2 of the twiddle table's length.  ELEMS complex
// values per workgroup (at least one row): small workgroups, which need fewer
// waves at a barrier, suit the passes that write or read wide segments
// (N'' = 2048, 2064 rows: t1_rows 20.0 us with two rows a workgroup, 19.1 with
// one); the cropped pass, whose columns may come in strips of two, takes two
// rows for 32-byte segments (N' = 4096: 30.8 us with one, 23 with two).
constexpr int kRowElems = 2048, kCropRowElems = 4096;

template <int LOG, int TL, int ELEMS = kRowElems>
struct RowCfg {
  static constexpr int N = 1 << LOG;
  static constexpr int C0 = ELEMS / N;
  static constexpr int CMIN = N < 32 ? 512 / N : 1;  // at least a wave
  static constexpr int C = C0 > 16 ? (CMIN > 16 ? CMIN : 16) : (C0 < 1 ? 1 : C0);
  static constexpr int NT = C * N / 8;
  static constexpr int DATA = lds_elems(C * N);
  static constexpr int LDS = (DATA + Tw2<TL>::SIZE) * 8;
};

// Column passes: C adjacent columns per workgroup, C * 2^LOG complex values in
// LDS (LOG: the longest transform): workgroups of 512 threads, three or four
// to a CU (N' = 2048, full band: t2_cols 38 us with 8192 values and 1024
// threads, 31 with 4096, 41 with 2048).
constexpr int kColElems = 4096;

constexpr int col_log(int log) {
  int l = 0;
  while (l < 4 && (kColElems >> (log + l + 1)) >= 1) ++l;
  return l;
}

template <int LOG, int TL>
struct ColCfg {
  static constexpr int CS = col_log(LOG), C = 1 << CS;
  static constexpr int NT = C * (1 << LOG) / 8;
  static constexpr int DATA = lds_elems(C << LOG);
  static constexpr int LDS = (DATA + Tw2<TL>::SIZE) * 8;
};

constexpr int imax(int a, int b) { return a > b ? a : b; }

// Longest transform of the three column passes (their strip widths follow).
constexpr int t1_cols_log(int lpf, int lp) { return imax(lpf, lp); }
// Whether the type-2 column pass runs its forward transform by half-length
// ones.  That takes half the LDS and one dependent transform more: it pays where
// a whole column fills a workgroup's LDS.  t2_cols and the row pass that reads
// its strips, split and whole, us a launch: N' = 512, N'' = 256 12.6 + 7.6 and
// 9.9 + 7.2 (full-length transforms throughout: 11.8 + 7.2), N' = 2048, N'' = 1024
// 18.7 + 14.7 and 17.0 + 14.7, N' = 4096, N'' = 2048 40.5 + 20.7 and 38.2 + 25.6,
// N' = 8192, N'' = 4096 140 + 86 and 163 + 86.
constexpr bool t2_split(int lpf, int lp, bool halfin) { return halfin && lpf < lp && lp >= 12; }
constexpr int t2_cols_log(int lpf, int lp, bool halfin) { return t2_split(lpf, lp, halfin) ? imax(lpf, lp - 1) : lp; }
// Strip widths of the arrays a column pass reads (cs) and writes (cv), whole
// multiples of its C columns.  A strip wider than C costs the column pass
// partial requests and saves them in the row pass: four columns balance the
// two, but for the array written by workgroups of one column, which take two
// (N' = 4096: t2_cols 90 us with strips of four, 64 with two; t2_rows_inv 80
// and 87).
static void set_strips(GridGeom* g, int log) {
  const int c = col_log(log);
  g->cs = imax(2, c);
  g->cv = c == 0 ? 1 : imax(2, c);
}
void set_t1_strips(GridGeom* g, int logNp) { set_strips(g, t1_cols_log(logNp, logNp)); }
void set_t2_strips(GridGeom* g, int logNpf, int logNp) { set_strips(g, t2_cols_log(logNpf, logNp, g->Nin < g->Np)); }
void set_t3_strips(GridGeom* g, int logNpf) { set_strips(g, logNpf); }

// Element (row, col) of an array of `rows` rows stored in strips of 2^cs columns.
__device__ __forceinline__ size_t strip_at(int rows, int cs, int row, int col) {
  return (((size_t)(col >> cs) * rows + row) << cs) + (col & ((1 << cs) - 1));
}

// Columns col (even) and col + 1 of a row (cs is 2 at least).
__device__ __forceinline__ void strip_store2(float2* __restrict__ a, int rows, int cs, int row, int col, float2 v0,
                                             float2 v1) {
  *reinterpret_cast<float4*>(a + strip_at(rows, cs, row, col)) = make_float4(v0.x, v0.y, v1.x, v1.y);
}

__device__ __forceinline__ bool in_band(int k, int lo, int hi) { return k >= lo && k <= hi; }

// Column passes launch the strips of C columns (of n, frequency k_x at column
// k_x + n/2) that meet the band of Eq. 4, and no others: the first one and
// their number.  The column range dealt to the XCDs is then the band's own.
// (With every strip launched and the ones outside the band leaving at once,
// the band, a run of consecutive strips, sat on a few of the eight XCDs:
// N' = 2048 with half the columns in band 36.6 us, N' = 8192 with 2020 in
// band 284 us, one launch.)
// (The n columns hold the band: K'' is chosen to, and a band empty along
// either axis comes here empty along x, with no strip.)
__host__ __device__ __forceinline__ int band_strip0(const GridGeom& g, int n, int C) { return (g.kxlo + n / 2) / C; }
static int band_strips(const GridGeom& g, int n, int C) {
  return g.kxlo > g.kxhi ? 0 : (g.kxhi + n / 2) / C - band_strip0(g, n, C) + 1;
}

// float64 square root from the hardware seed (v_rsq_f64) refined by Newton
// steps: each step squares the relative error, so two steps from the ~2^-23
// seed are far below 2^-53; a final residual correction gives sqrt to about
// one ulp.
__device__ __forceinline__ double sqrt_nr(double r) {
  double y = __builtin_amdgcn_rsq(r);
  y = y * (1.5 - 0.5 * r * y * y);
  y = y * (1.5 - 0.5 * r * y * y);
  const double s = r * y;
  return s + 0.5 * y * (r - s * s);
}

// Transfer function of Eq. 4 (ASM) or Eq. 5 (Fresnel) at integer frequency
// (kx, ky), without the Rect.  The ASM phase is formed in cycles:
// z sqrt(1/l^2 - df^2 k^2) = z/l - (z/l)(1 - sqrt(1 - t)), t = (l df)^2 k^2.
// sqrt(1 - t) is accurate to about one ulp of 1, so the subtracted term is
// off by about (z/l) 2^-53 cycles however large z/l is (1e-10 cycles at
// z/l = 2e6); z/l itself enters only as its fraction c0.  The phase is then
// reduced to [-1/2, 1/2] before the float32 sine and cosine.  Evanescent
// frequencies (t > 1) give 0.
__device__ __forceinline__ float2 transfer_at(const Spectral& sp, int Np, int kx, int ky) {
  float2 h;
  if (sp.tf == 1) {
    h = cmul(sp.fre_x[kx + Np / 2], sp.fre_y[ky + Np / 2]);
  } else if (sp.phase_fp64) {
    const double k2 = (double)kx * kx + (double)ky * ky;
    const double u = 1.0 - sp.ql2 * k2;
    if (u < 0.0) return czero();
    const double s = u > 0.0 ? sqrt_nr(u) : 0.0;
    double cyc = sp.c0 + sp.ax * kx + sp.ay * ky - sp.zl * (1.0 - s);
    cyc -= rint(cyc);
    h = cis_rev((float)cyc);
  } else {
    const float k2 = (float)kx * (float)kx + (float)ky * (float)ky;
    const float r = sp.inv_lam2f - sp.qf * k2;
    if (r < 0.0f) return czero();
    float cyc = sp.axf * (float)kx + sp.ayf * (float)ky + sp.zf * sqrtf(r);
    cyc -= rintf(cyc);
    h = cis_rev(cyc);
  }
  if (sp.conj) h.y = -h.y;
  return h;
}

__device__ __forceinline__ float2 csel(bool ok, float2 v) { return ok ? v : czero(); }

// The fine support along one axis as the input of the half-length transforms
// of length N = N'': element u = i0 + m N/8 gathers the cells u and u + N of
// the fine axis that lie in the support.  at(i) reads support cell i.  main[m]
// is cell u + N for m < 4 and u for m >= 4 (always inside the support), and
// edge[m] the other one, inside it for 2 kPad of the u only.
template <int N, class At>
__device__ __forceinline__ void load_support(int i0, const At& at, float2 (&main)[8], float2 (&edge)[8]) {
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    const int u = i0 + m * (N / 8);
    edge[m] = czero();
    if (m < 4) {
      main[m] = at(u + N / 2 + kPad);
      if ((m + 1) * (N / 8) > N / 2 - kPad && u >= N / 2 - kPad) edge[m] = at(u - N / 2 + kPad);
    } else {
      main[m] = at(u - N / 2 + kPad);
      if (m * (N / 8) < N / 2 + kPad && u < N / 2 + kPad) edge[m] = at(u + N / 2 + kPad);
    }
  }
}

// Input of the half-length transform of parity p: cells u + N enter with
// (-1)^p.
__device__ __forceinline__ void fold_support(int p, const float2 (&main)[8], const float2 (&edge)[8], float2 (&x)[8]) {
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    const float2 hi = m < 4 ? main[m] : edge[m], lo = m < 4 ? edge[m] : main[m];
    x[m] = p ? csub(lo, hi) : cadd(lo, hi);
  }
}

// Whether element m of eight (i0 + m N/8, taken as signed, [-N/2, N/2)) can lie
// in [-K/2, K/2).
constexpr bool mode_kept(int m, int N, int K) { return (m < 4 ? m : 7 - m) * (N / 8) < K / 2; }

// ----------------------------------------------------------------- type 1
// Fine support rows -> nf-point FFT along x -> keep k_x in K'', times 1/psihat.
// T(i, k_x) = sum_l G[i][l] exp(-2 pi i k_x (s0 + l) / nf) / psihat(k_x).
template <int LOG>
__device__ __forceinline__ void t1_rows_body(const RowArgs& a, int bid, int nbid) {
  const float2* __restrict__ fine = a.in;
  float2* __restrict__ T = a.out;
  const GridGeom& g = a.g;
  const float* __restrict__ dinv = a.dinv;
  constexpr int N = 1 << LOG, TL = LOG + 1;
  using Cfg = RowCfg<LOG, TL>;
  constexpr int C = Cfg::C, NT = Cfg::NT;
  extern __shared__ float2 s[];
  float2* tw = s + Cfg::DATA;
  const int tid = (int)threadIdx.x, i0 = tid / C;
  const int L = g.L, row = xcd_remap(bid, nbid) * C + tid % C;
  const float2* src = fine + (size_t)min(row, L - 1) * L;
  float2 x[8], h[8], main[8], edge[8];
  load_support<N>(i0, [&](int i) { return src[i]; }, main, edge);
  load_tw2<TL, NT>(tw, tw_for(a.tw, TL));
  fold_support(0, main, edge, h);
  reg_fft<LOG, C, NT, -1, false, TL>(s, tw, tid, h);
  fold_support(1, main, edge, x);
  reg_fft<LOG, C, NT, -1, true, TL>(s, tw, opaque_tid(), x);
  if (row >= L) return;
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    if (m >= 2 && m < 6) continue;  // outside K''
    const int q = i0 + m * (N / 8), kx = 2 * (m < 4 ? q : q - N), ax = kx + N / 2;
    if (kx + 1 >= g.kxlo && kx <= g.kxhi)
      strip_store2(T, L, g.cs, row, ax, cscale(h[m], dinv[ax]), cscale(x[m], dinv[ax + 1]));
  }
}

// Columns of T -> nf-point FFT along y -> keep k_y in the spectral grid K''
// (N'' modes, a superset of the band of Eq. 4; N'' = N' unless the band
// is narrow) -> times H(k) Rect(k) / psihat(k_y) / N'^2 -> embedded in K ->
// N'-point inverse FFT along y.  T holds the columns k_x + N''/2; V has N'
// columns, k_x + N'/2, and N' rows (the central N when cropping).  The (-1)^k
// factors of the centred fine grid and of the centred inverse DFT cancel
// (N'/2 is even); the remaining output sign (-1)^n_y is applied here.
template <int LPF, int LP>
__device__ __forceinline__ void t1_cols_body(const ColArgs& a, int bid, int nbid) {
  const GridGeom& g = a.g;
  const Spectral& sp = a.sp;
  constexpr int N = 1 << LPF, NP = 1 << LP, TL = imax(LPF + 1, LP);
  using Cfg = ColCfg<t1_cols_log(LPF, LP), TL>;
  constexpr int C = Cfg::C, NT = Cfg::NT, NA = C * N / 8;
  extern __shared__ float2 s[];
  float2* tw = s + Cfg::DATA;
  const int a0 = (band_strip0(g, N, C) + xcd_remap(bid, nbid)) * C;
  const int kx0 = a0 - N / 2;
  const int tid = (int)threadIdx.x, c = tid % C, i0 = tid / C, kx = kx0 + c;
  const int L = g.L;
  const bool inx = in_band(kx, g.kxlo, g.kxhi);
  float2 x[8], h[8], main[8], edge[8];
  if (NA == NT || tid < NA) {
    const float2* src = a.in + strip_at(L, g.cs, 0, a0) + c;
    load_support<N>(i0, [&](int i) { return csel(inx, src[i << g.cs]); }, main, edge);
  }
  load_tw2<TL, NT>(tw, tw_for(a.tw, TL));
  // H Rect / psihat / N'^2 at mode 2 q + p of element m
  auto spectral = [&](int m, int p, float2 v) -> float2 {
    const int q = i0 + m * (N / 8), ky = 2 * (m < 4 ? q : q - N) + p;
    if (!inx || !in_band(ky, g.kylo, g.kyhi)) return czero();
    return cscale(cmul(v, transfer_at(sp, NP, kx, ky)), sp.dinv[ky + N / 2] * sp.scale);
  };
  fold_support(0, main, edge, h);
  reg_fft<LPF, C, NT, -1, false, TL>(s, tw, tid, h);
  if (NA == NT || tid < NA) {
#pragma unroll
    for (int m = 0; m < 8; ++m)
      if (m < 2 || m >= 6) h[m] = spectral(m, 0, h[m]);
  }
  fold_support(1, main, edge, x);
  reg_fft<LPF, C, NT, -1, true, TL>(s, tw, opaque_tid(), x);
  __syncthreads();
  if (NA == NT || tid < NA) {
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      if (m >= 2 && m < 6) continue;  // outside K''
      const int q = i0 + m * (N / 8), ay = 2 * (m < 4 ? q : q - N) + NP / 2;
      s[pidx(ay * C + c)] = h[m];
      s[pidx((ay + 1) * C + c)] = spectral(m, 1, x[m]);
    }
  }
  if constexpr (N < NP) {
    // K outside K'': [0, (N' - N'')/2) and [(N' + N'')/2, N')
    constexpr int H = (NP - N) / 2;
    for (int e = tid; e < 2 * H * C; e += NT) {
      const int u = e / C, ay = u < H ? u : u + N;
      s[pidx(ay * C + c)] = czero();
    }
  }
  __syncthreads();
  const int t2 = opaque_tid(), j0 = t2 / C, c2 = t2 % C;
#pragma unroll
  for (int m = 0; m < 8; ++m) x[m] = s[pidx((j0 + m * (NP / 8)) * C + c2)];
  reg_fft<LP, C, NT, +1, false, TL>(s, tw, t2, x);
  // V: this strip's columns, with the (-1)^n_y sign
  const int nrows = g.crop ? NP / 2 : NP, row0 = g.crop ? NP / 4 : 0;
  float2* dst = a.out + strip_at(nrows, g.cv, 0, a0 - N / 2 + NP / 2) + c2;
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    const int by = j0 + m * (NP / 8), r = by - row0;
    if (r >= 0 && r < nrows) dst[r << g.cv] = (by & 1) ? make_float2(-x[m].x, -x[m].y) : x[m];
  }
}

// Rows of V -> N'-point inverse FFT along x -> times (-1)^n_x -> plane
// (N' x N'), or, when cropping, the central N x N: the outputs
// [N'/4, 3N'/4) of each parity from half-length transforms.
template <int LP>
__device__ __forceinline__ void t1_rows_inv_body(const RowArgs& a, int bid, int nbid) {
  const float2* __restrict__ V = a.in;
  float2* __restrict__ out = a.out;
  const GridGeom& g = a.g;
  constexpr int N = 1 << LP;
  using Cfg = RowCfg<LP, LP>;
  constexpr int C = Cfg::C, NT = Cfg::NT;
  extern __shared__ float2 s[];
  float2* tw = s + Cfg::DATA;
  const int tid = (int)threadIdx.x, i0 = tid / C;
  const int row = xcd_remap(bid, nbid) * C + tid % C, rowc = min(row, N - 1);
  float2 x[8];
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    const int ax = i0 + m * (N / 8);
    x[m] = csel(in_band(ax - N / 2, g.kxlo, g.kxhi), V[strip_at(N, g.cv, rowc, ax)]);
  }
  load_tw2<LP, NT>(tw, tw_for(a.tw, LP));
  reg_fft<LP, C, NT, +1, false, LP>(s, tw, tid, x);
  if (row >= N) return;
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    const int bx = i0 + m * (N / 8);
    out[(size_t)row * N + bx] = (bx & 1) ? make_float2(-x[m].x, -x[m].y) : x[m];
  }
}

template <int LP>
__device__ __forceinline__ void t1_rows_inv_crop_body(const RowArgs& a, int bid, int nbid) {
  const float2* __restrict__ V = a.in;
  float2* __restrict__ out = a.out;
  const GridGeom& g = a.g;
  constexpr int LOG = LP - 1, N = 1 << LOG, TL = LP;
  using Cfg = RowCfg<LOG, TL, kCropRowElems>;
  constexpr int C = Cfg::C, NT = Cfg::NT;
  extern __shared__ float2 s[];
  float2* tw = s + Cfg::DATA;
  const int tid = (int)threadIdx.x, i0 = tid / C;
  const int row = xcd_remap(bid, nbid) * C + tid % C, rowc = min(row, N - 1);
  float2 h[8], x[8];
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    // modes u and u + N of the N'-point transform
    const int u = i0 + m * (N / 8);
    const float2 lo = csel(in_band(u - N, g.kxlo, g.kxhi), V[strip_at(N, g.cv, rowc, u)]);
    const float2 hi = csel(in_band(u, g.kxlo, g.kxhi), V[strip_at(N, g.cv, rowc, u + N)]);
    h[m] = cadd(lo, hi);
    x[m] = csub(lo, hi);
  }
  load_tw2<TL, NT>(tw, tw_for(a.tw, TL));
  reg_fft<LOG, C, NT, +1, false, TL>(s, tw, tid, h);
  reg_fft<LOG, C, NT, +1, true, TL>(s, tw, opaque_tid(), x);
  if (row >= N) return;
  // outputs 2 q (sign +) and 2 q + 1 (sign -) of the central N columns; the
  // caller's plane may be aligned to one element only
  float2* dst = out + (size_t)row * N;
  const bool wide = ((uintptr_t)out & 15) == 0;
#pragma unroll
  for (int m = 2; m < 6; ++m) {
    const int ox = 2 * (i0 + m * (N / 8)) - N / 2;
    if (wide) {
      *reinterpret_cast<float4*>(dst + ox) = make_float4(h[m].x, h[m].y, -x[m].x, -x[m].y);
    } else {
      dst[ox] = h[m];
      dst[ox + 1] = make_float2(-x[m].x, -x[m].y);
    }
  }
}

// ----------------------------------------------------------------- type 2
// Rows of the Nin x Nin plane, zero-padded circularly to N' -> FFT along x ->
// times (-1)^k_x / psihat(k_x), T(row, k_x + N'/2).  HALFIN: Nin = N, by
// half-length transforms of the even and odd modes; else Nin = N'.
template <int LP, bool HALFIN>
__device__ __forceinline__ void t2_rows_body(const RowArgs& a, int bid, int nbid) {
  const float2* __restrict__ u1 = a.in;
  float2* __restrict__ T = a.out;
  const GridGeom& g = a.g;
  const float* __restrict__ dinv = a.dinv;
  constexpr int LOG = HALFIN ? LP - 1 : LP, N = 1 << LOG, NP = 1 << LP, TL = LP;
  using Cfg = RowCfg<LOG, TL>;
  constexpr int C = Cfg::C, NT = Cfg::NT;
  extern __shared__ float2 s[];
  float2* tw = s + Cfg::DATA;
  const int tid = (int)threadIdx.x, i0 = tid / C;
  const int row = xcd_remap(bid, nbid) * C + tid % C;
  const float2* src = u1 + (size_t)min(row, N - 1) * N;
  float2 x[8];
  // element u: sample u of the row's upper half, or u - N of its lower half
#pragma unroll
  for (int m = 0; m < 8; ++m) x[m] = src[i0 + m * (N / 8) + (m < 4 ? N / 2 : -N / 2)];
  load_tw2<TL, NT>(tw, tw_for(a.tw, TL));
  if constexpr (HALFIN) {
    float2 h[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      h[m] = x[m];
      if (m >= 4) x[m] = make_float2(-x[m].x, -x[m].y);
    }
    reg_fft<LOG, C, NT, -1, false, TL>(s, tw, tid, h);
    reg_fft<LOG, C, NT, -1, true, TL>(s, tw, opaque_tid(), x);
    if (row >= N) return;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const int q = i0 + m * (N / 8), kx = 2 * (m < 4 ? q : q - N), ax = kx + NP / 2;
      if (kx + 1 >= g.kxlo && kx <= g.kxhi)
        strip_store2(T, N, g.cs, row, ax, cscale(h[m], dinv[ax]), cscale(x[m], -dinv[ax + 1]));
    }
  } else {
    reg_fft<LOG, C, NT, -1, false, TL>(s, tw, tid, x);
    if (row >= N) return;
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const int t = i0 + m * (N / 8), kx = m < 4 ? t : t - N, ax = kx + N / 2;
      if (in_band(kx, g.kxlo, g.kxhi)) T[strip_at(N, g.cs, row, ax)] = cscale(x[m], (kx & 1) ? -dinv[ax] : dinv[ax]);
    }
  }
}

// The modes k of element m (signed, [-N''/2, N''/2)) as the input of the
// half-length inverse transform of parity p: negative modes enter with (-1)^p.
__device__ __forceinline__ void fold_modes(const float2 (&v)[8], float2 (&x)[8]) {
#pragma unroll
  for (int m = 0; m < 8; ++m) x[m] = m < 4 ? v[m] : make_float2(-v[m].x, -v[m].y);
}

// Support rows 2 q - s0 and 2 q + 1 - s0 of a column strip (outputs 2 q and
// 2 q + 1 of the nf-point inverse transform): lanes of a pair of columns
// exchange halves, so that each stores two columns of one row.
template <int N, int C>
__device__ __forceinline__ void store_support_rows(float2* __restrict__ strip, int L, int cs, int tid, const float2 (&h)[8],
                                                   const float2 (&x)[8]) {
  const int c = tid % C, i0 = tid / C;
  constexpr int s0 = N / 2 - kPad;
#pragma unroll
  for (int m = 1; m < 7; ++m) {
    const int i = 2 * (i0 + m * (N / 8)) - s0;
    if constexpr (C > 1) {
      const bool odd = c & 1;
      const float2 give = odd ? h[m] : x[m];
      const float2 got = make_float2(pair_swap(give.x), pair_swap(give.y));
      const float4 v = odd ? make_float4(got.x, got.y, x[m].x, x[m].y) : make_float4(h[m].x, h[m].y, got.x, got.y);
      if (i >= 0 && i < L)
        *reinterpret_cast<float4*>(strip + ((i + (odd ? 1 : 0)) << cs) + (c & ~1)) = v;
    } else if (i >= 0 && i < L) {
      strip[i << cs] = h[m];
      strip[(i + 1) << cs] = x[m];
    }
  }
}

// Columns of T (Nin rows, N' columns k_x + N'/2) -> N'-point FFT along y ->
// the modes k_y of the spectral grid K'' (N'' modes, a superset of the band
// of Eq. 4) times H(k) Rect(k) (-1)^k_y / psihat(k_y) / N'^2 -> inverse
// nf-point FFT along y (nf = 2 N'') -> the support rows [s0, s0 + L), N''
// columns k_x + N''/2.  HALFIN: Nin = N.  With a narrow band (N'' < N') the
// modes of the forward transform, at full length or by half-length transforms
// (t2_split), reach the inverse one through LDS; otherwise it runs at full
// length, which leaves every mode in the register where the inverse
// transforms want it.
template <int LPF, int LP, bool HALFIN>
__device__ __forceinline__ void t2_cols_body(const ColArgs& a, int bid, int nbid) {
  const GridGeom& g = a.g;
  const Spectral& sp = a.sp;
  constexpr int N = 1 << LPF, NP = 1 << LP, TL = imax(LPF + 1, LP);
  constexpr bool SPLIT = t2_split(LPF, LP, HALFIN);
  using Cfg = ColCfg<t2_cols_log(LPF, LP, HALFIN), TL>;
  constexpr int C = Cfg::C, NT = Cfg::NT, NA = C * N / 8;
  extern __shared__ float2 s[];
  float2* tw = s + Cfg::DATA;
  const int a0 = (band_strip0(g, NP, C) + xcd_remap(bid, nbid)) * C;
  const int kx0 = a0 - NP / 2;
  const int tid = (int)threadIdx.x, c = tid % C, i0 = tid / C, kx = kx0 + c;
  const bool inx = in_band(kx, g.kxlo, g.kxhi);
  const int Nin = HALFIN ? NP / 2 : NP;
  const float2* src = a.in + strip_at(Nin, g.cs, 0, a0) + c;
  auto row = [&](int r) { return csel(inx, src[r << g.cs]); };
  auto spectral = [&](int ky, float2 v) -> float2 {
    if (!inx || !in_band(ky, g.kylo, g.kyhi)) return czero();
    return cscale(cmul(v, transfer_at(sp, NP, kx, ky)),
                  sp.dinv[ky + N / 2] * sp.scale * ((ky & 1) ? -1.0f : 1.0f));
  };
  float2 v[8];  // modes i0 + m N''/8 of the inverse transforms
  if constexpr (SPLIT) {
    constexpr int LH = LP - 1, H = 1 << LH, NF = C * H / 8;
    float2 h[8], x[8];
    const bool act = NF == NT || tid < NF;
    if (act) {
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        h[m] = row(i0 + m * (H / 8) + (m < 4 ? H / 2 : -H / 2));
        x[m] = m < 4 ? h[m] : make_float2(-h[m].x, -h[m].y);
      }
    }
    load_tw2<TL, NT>(tw, tw_for(a.tw, TL));
    reg_fft<LH, C, NT, -1, false, TL>(s, tw, tid, h);
    reg_fft<LH, C, NT, -1, true, TL>(s, tw, opaque_tid(), x);
    __syncthreads();
    if (act) {
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        // even mode ky, odd mode ky + 1; K'' keeps q in [-N''/4, N''/4)
        if (!mode_kept(m, H, N / 2)) continue;
        const int q = i0 + m * (H / 8), ky = 2 * (m < 4 ? q : q - H);
        if (ky < -N / 2 || ky >= N / 2) continue;
        s[pidx((ky & (N - 1)) * C + c)] = spectral(ky, h[m]);
        s[pidx(((ky + 1) & (N - 1)) * C + c)] = spectral(ky + 1, x[m]);
      }
    }
    __syncthreads();
  } else {
    float2 x[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const int t = i0 + m * (NP / 8);
      if (HALFIN)
        x[m] = m < 2 ? row(t + NP / 4) : m >= 6 ? row(t - NP + NP / 4) : czero();
      else
        x[m] = row(m < 4 ? t + NP / 2 : t - NP / 2);
    }
    load_tw2<TL, NT>(tw, tw_for(a.tw, TL));
    reg_fft<LP, C, NT, -1, false, TL>(s, tw, tid, x);
    if constexpr (LPF < LP) __syncthreads();
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const int t = i0 + m * (NP / 8), ky = m < 4 ? t : t - NP;
      if constexpr (LPF == LP) {
        v[m] = spectral(ky, x[m]);
      } else if (mode_kept(m, NP, N)) {
        if (ky >= -N / 2 && ky < N / 2) s[pidx((ky & (N - 1)) * C + c)] = spectral(ky, x[m]);
      }
    }
    if constexpr (LPF < LP) __syncthreads();
  }
  if constexpr (LPF < LP) {
    if (NA == NT || tid < NA) {
#pragma unroll
      for (int m = 0; m < 8; ++m) v[m] = s[pidx((i0 + m * (N / 8)) * C + c)];
    }
  }
  float2 x[8];
  fold_modes(v, x);
  const int t2 = opaque_tid();
  reg_fft<LPF, C, NT, +1, false, TL>(s, tw, t2, v);
  reg_fft<LPF, C, NT, +1, true, TL>(s, tw, t2, x);
  if (NA == NT || t2 < NA) store_support_rows<N, C>(a.out + strip_at(g.L, g.cv, 0, kx0 + N / 2), g.L, g.cv, t2, v, x);
}

// Support rows of V -> embed k_x into nf -> inverse nf-point FFT along x ->
// keep support columns: the fine grid the interpolation reads.
template <int LOG>
__device__ __forceinline__ void t2_rows_inv_body(const RowArgs& a, int bid, int nbid) {
  const float2* __restrict__ V = a.in;
  float2* __restrict__ fine = a.out;
  const GridGeom& g = a.g;
  constexpr int N = 1 << LOG, TL = LOG + 1;
  using Cfg = RowCfg<LOG, TL>;
  constexpr int C = Cfg::C, NT = Cfg::NT;
  extern __shared__ float2 s[];
  float2* tw = s + Cfg::DATA;
  const int tid = (int)threadIdx.x, i0 = tid / C;
  const int L = g.L, row = xcd_remap(bid, nbid) * C + tid % C, rowc = min(row, L - 1);
  float2 h[8], x[8];
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    const int ax = i0 + m * (N / 8) + (m < 4 ? N / 2 : -N / 2);
    h[m] = csel(in_band(ax - N / 2, g.kxlo, g.kxhi), V[strip_at(L, g.cv, rowc, ax)]);
  }
  load_tw2<TL, NT>(tw, tw_for(a.tw, TL));
  fold_modes(h, x);
  reg_fft<LOG, C, NT, +1, false, TL>(s, tw, tid, h);
  reg_fft<LOG, C, NT, +1, true, TL>(s, tw, opaque_tid(), x);
  if (row >= L) return;
  // outputs 2 q and 2 q + 1 that lie in the support
  float2* dst = fine + (size_t)row * L;
#pragma unroll
  for (int m = 1; m < 7; ++m) {
    const int i = 2 * (i0 + m * (N / 8)) - (N / 2 - kPad);
    if (i >= 0 && i < L) *reinterpret_cast<float4*>(dst + i) = make_float4(h[m].x, h[m].y, x[m].x, x[m].y);
  }
}

// ----------------------------------------------------------------- type 3
// Column pass of NU-ASM_3 / NU-FRE_3 (non-uniform source and destination),
// between the type-1 row pass over the source's fine support and the type-2
// inverse row pass over the destination's: columns of T -> nf-point FFT along
// y -> keep k_y in K'' -> times H(k) Rect(k) N'^-2
// and the three deconvolutions not applied elsewhere, 1/psihat(k_y) of the
// spreading, 1/psihat(k_y) and 1/psihat(k_x) of the interpolation -> inverse
// nf-point FFT along y -> the support rows [s0, s0 + L).  Both grids are fine
// grids, so the (-1)^k factors of the window offset cancel between the
// forward and the inverse transform on each axis.
template <int LPF>
__global__ void __launch_bounds__((ColCfg<LPF, LPF + 1>::NT))
k_t3_cols(const float2* __restrict__ T, float2* __restrict__ V, GridGeom g, Spectral sp,
          const float2* __restrict__ twall) {
  constexpr int N = 1 << LPF, TL = LPF + 1;
  using Cfg = ColCfg<LPF, TL>;
  constexpr int C = Cfg::C, NT = Cfg::NT;
  extern __shared__ float2 s[];
  float2* tw = s + Cfg::DATA;
  const int a0 = (band_strip0(g, N, C) + xcd_remap((int)blockIdx.x, (int)gridDim.x)) * C;
  const int tid = (int)threadIdx.x, c = tid % C, i0 = tid / C, kx = a0 - N / 2 + c;
  const int L = g.L;
  const bool inx = in_band(kx, g.kxlo, g.kxhi);
  float2 x[8], h[8], main[8], edge[8];
  const float2* src = T + strip_at(L, g.cs, 0, a0) + c;
  load_support<N>(i0, [&](int i) { return csel(inx, src[i << g.cs]); }, main, edge);
  load_tw2<TL, NT>(tw, tw_for(twall, TL));
  const float dx = inx ? sp.dinv[kx + N / 2] * sp.scale : 0.f;
  auto spectral = [&](int m, int p, float2 v) -> float2 {
    const int q = i0 + m * (N / 8), ky = 2 * (m < 4 ? q : q - N) + p;
    if (!inx || !in_band(ky, g.kylo, g.kyhi)) return czero();
    const float dy = sp.dinv[ky + N / 2];
    return cscale(cmul(v, transfer_at(sp, g.Np, kx, ky)), dy * dy * dx);
  };
  fold_support(0, main, edge, h);
  reg_fft<LPF, C, NT, -1, false, TL>(s, tw, tid, h);
#pragma unroll
  for (int m = 0; m < 8; ++m)
    if (m < 2 || m >= 6) h[m] = spectral(m, 0, h[m]);
  fold_support(1, main, edge, x);
  reg_fft<LPF, C, NT, -1, true, TL>(s, tw, opaque_tid(), x);
  __syncthreads();
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    if (m >= 2 && m < 6) continue;  // outside K''
    const int q = i0 + m * (N / 8), u = (2 * q) & (N - 1);  // mode 2 q mod N''
    s[pidx(u * C + c)] = h[m];
    s[pidx((u + 1) * C + c)] = spectral(m, 1, x[m]);
  }
  __syncthreads();
#pragma unroll
  for (int m = 0; m < 8; ++m) h[m] = s[pidx((i0 + m * (N / 8)) * C + c)];
  fold_modes(h, x);
  const int t2 = opaque_tid();
  reg_fft<LPF, C, NT, +1, false, TL>(s, tw, t2, h);
  reg_fft<LPF, C, NT, +1, true, TL>(s, tw, t2, x);
  store_support_rows<N, C>(V + strip_at(L, g.cv, 0, a0), L, g.cv, t2, h, x);
}

// ----------------------------------------------------------- test kernels
// Batched 1-D transforms of length 2^LOGN by the half-length transforms of the
// even and odd outputs.
template <int LOGN, int DIR>
__global__ void __launch_bounds__((RowCfg<LOGN - 1, LOGN>::NT))
k_fft_rows(const float2* __restrict__ in, float2* __restrict__ out, int64_t batch,
           const float2* __restrict__ twall) {
  constexpr int LOG = LOGN - 1, N = 1 << LOG;
  using Cfg = RowCfg<LOG, LOGN>;
  constexpr int C = Cfg::C, NT = Cfg::NT;
  extern __shared__ float2 s[];
  float2* tw = s + Cfg::DATA;
  const int tid = (int)threadIdx.x, i0 = tid / C;
  const int64_t r = (int64_t)blockIdx.x * C + tid % C;
  const float2* src = in + (r < batch ? r : batch - 1) * 2 * N;
  float2 h[8], x[8];
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    const int u = i0 + m * (N / 8);
    const float2 lo = src[u], hi = src[u + N];
    h[m] = cadd(lo, hi);
    x[m] = csub(lo, hi);
  }
  load_tw2<LOGN, NT>(tw, tw_for(twall, LOGN));
  reg_fft<LOG, C, NT, DIR, false, LOGN>(s, tw, tid, h);
  reg_fft<LOG, C, NT, DIR, true, LOGN>(s, tw, opaque_tid(), x);
  if (r >= batch) return;
#pragma unroll
  for (int m = 0; m < 8; ++m) {
    const int q = i0 + m * (N / 8);
    out[r * 2 * N + 2 * q] = h[m];
    out[r * 2 * N + 2 * q + 1] = x[m];
  }
}

__global__ void k_transfer_table(GridGeom g, Spectral sp, float2* __restrict__ out) {
  const int Np = g.Np;
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= (int64_t)Np * Np) return;
  const int ay = (int)(e / Np), ax = (int)(e % Np);
  const int kx = ax - Np / 2, ky = ay - Np / 2;
  float2 h = czero();
  if (in_band(kx, g.kxlo, g.kxhi) && in_band(ky, g.kylo, g.kyhi)) h = transfer_at(sp, Np, kx, ky);
  out[e] = h;
}

// One axis of the Fresnel transfer function (Eq. 5) in float64:
// out[k + N'/2] = amp * sum_{m in K} exp(i pi (m g + o)^2 / (lambda z)) exp(-2 pi i k m / N').
// Both phases are reduced to whole cycles exactly (k m mod N' in integers)
// before the float64 sincospi.  One workgroup per output frequency; its 256
// threads split the N' terms and meet in an LDS tree.
constexpr int kFresnelThreads = 256;

__global__ void __launch_bounds__(kFresnelThreads)
k_fresnel_axis(int Np, double g, double two_lam_z, double o, double2 amp, float2* __restrict__ out) {
  __shared__ double2 part[kFresnelThreads];
  const int a = blockIdx.x;
  const int64_t k = a - Np / 2;
  double re = 0.0, im = 0.0;
  for (int m = -Np / 2 + (int)threadIdx.x; m < Np / 2; m += kFresnelThreads) {
    const double xm = m * g + o;
    double c = xm * xm / two_lam_z;
    c -= rint(c);
    const int64_t km = (k * m) % Np;
    double cyc = c - (double)km / (double)Np;
    double sn, cs;
    sincospi(2.0 * cyc, &sn, &cs);
    re += cs;
    im += sn;
  }
  part[threadIdx.x] = make_double2(re, im);
  __syncthreads();
  for (int h = kFresnelThreads / 2; h > 0; h >>= 1) {
    if ((int)threadIdx.x < h) {
      part[threadIdx.x].x += part[threadIdx.x + h].x;
      part[threadIdx.x].y += part[threadIdx.x + h].y;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    re = part[0].x;
    im = part[0].y;
    out[a] = make_float2((float)(re * amp.x - im * amp.y), (float)(re * amp.y + im * amp.x));
  }
}

// --------------------------------------------------------------- launchers
template <typename K>
static hipError_t set_lds(K kernel, int bytes) {
  if (bytes > 64 * 1024)
    return hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  return hipSuccess;
}

#define NUASM_DISPATCH_NP(logNp, CALL)                  \
  switch (logNp) {                                      \
    case 5: CALL(5); break;                             \
    case 6: CALL(6); break;                             \
    case 7: CALL(7); break;                             \
    case 8: CALL(8); break;                             \
    case 9: CALL(9); break;                             \
    case 10: CALL(10); break;                           \
    case 11: CALL(11); break;                           \
    case 12: CALL(12); break;                           \
    case 13: CALL(13); break;                           \
    default: return hipErrorInvalidValue;               \
  }

hipError_t launch_t1_rows(int logNp, const float2* fine, float2* T, GridGeom g, const float* dinv,
                          const float2* tw, hipStream_t st) {
  const RowArgs a{fine, T, g, dinv, tw};
#define CALL(LP)                                                                                 \
  {                                                                                              \
    using Cfg = RowCfg<LP, LP + 1>;                                                              \
    return launch_or_record<RowArgs, t1_rows_body<LP>, Cfg::NT>(a, (g.L + Cfg::C - 1) / Cfg::C,  \
                                                                Cfg::LDS, st);                   \
  }
  NUASM_DISPATCH_NP(logNp, CALL)
#undef CALL
  return hipErrorInvalidValue;
}

// Column passes: the spectral grid N'' = 2^logNpf may be N', N'/2, N'/4 or
// N'/8 (at least 32).
template <int LPF, int LP>
static hipError_t t1_cols_at(const float2* T, float2* V, const GridGeom& g, const Spectral& sp, const float2* tw,
                             hipStream_t st) {
  using Cfg = ColCfg<t1_cols_log(LPF, LP), imax(LPF + 1, LP)>;
  return launch_or_record<ColArgs, t1_cols_body<LPF, LP>, Cfg::NT>(
      ColArgs{T, V, g, sp, tw}, band_strips(g, 1 << LPF, Cfg::C), Cfg::LDS, st);
}

template <int LPF, int LP, bool HALFIN>
static hipError_t t2_cols_in(const float2* T, float2* V, const GridGeom& g, const Spectral& sp, const float2* tw,
                             hipStream_t st) {
  using Cfg = ColCfg<t2_cols_log(LPF, LP, HALFIN), imax(LPF + 1, LP)>;
  return launch_or_record<ColArgs, t2_cols_body<LPF, LP, HALFIN>, Cfg::NT>(
      ColArgs{T, V, g, sp, tw}, band_strips(g, 1 << LP, Cfg::C), Cfg::LDS, st);
}

template <int LPF, int LP>
static hipError_t t2_cols_at(const float2* T, float2* V, const GridGeom& g, const Spectral& sp, const float2* tw,
                             hipStream_t st) {
  return g.Nin < g.Np ? t2_cols_in<LPF, LP, true>(T, V, g, sp, tw, st)
                      : t2_cols_in<LPF, LP, false>(T, V, g, sp, tw, st);
}

template <int LP, bool T1>
static hipError_t cols_by_reduction(int d, const float2* T, float2* V, const GridGeom& g, const Spectral& sp,
                                    const float2* tw, hipStream_t st) {
#define NUASM_COLS_AT(D)                                                    \
  if constexpr (LP - D >= 5) {                                              \
    if (d == D)                                                             \
      return T1 ? t1_cols_at<LP - D, LP>(T, V, g, sp, tw, st)               \
                : t2_cols_at<LP - D, LP>(T, V, g, sp, tw, st);              \
  }
  NUASM_COLS_AT(0)
  NUASM_COLS_AT(1)
  NUASM_COLS_AT(2)
  NUASM_COLS_AT(3)
#undef NUASM_COLS_AT
  return hipErrorInvalidValue;
}

hipError_t launch_t1_cols(int logNpf, int logNp, const float2* T, float2* V, GridGeom g, Spectral sp,
                          const float2* tw, hipStream_t st) {
  const int d = logNp - logNpf;
#define CALL(LP) return cols_by_reduction<LP, true>(d, T, V, g, sp, tw, st)
  NUASM_DISPATCH_NP(logNp, CALL)
#undef CALL
  return hipErrorInvalidValue;
}

hipError_t launch_t1_rows_inv(int logNp, const float2* V, float2* out, GridGeom g, const float2* tw,
                              hipStream_t st) {
  const RowArgs a{V, out, g, nullptr, tw};
#define CALL(LP)                                                                                             \
  {                                                                                                          \
    using Full = RowCfg<LP, LP>;                                                                             \
    using Crop = RowCfg<LP - 1, LP, kCropRowElems>;                                                                         \
    constexpr int NP = 1 << LP;                                                                              \
    if (g.crop)                                                                                              \
      return launch_or_record<RowArgs, t1_rows_inv_crop_body<LP>, Crop::NT>(                                 \
          a, (NP / 2 + Crop::C - 1) / Crop::C, Crop::LDS, st);                                               \
    return launch_or_record<RowArgs, t1_rows_inv_body<LP>, Full::NT>(a, (NP + Full::C - 1) / Full::C, Full::LDS, st); \
  }
  NUASM_DISPATCH_NP(logNp, CALL)
#undef CALL
  return hipErrorInvalidValue;
}

hipError_t launch_t2_rows(int logNp, const float2* u1, float2* T, GridGeom g, const float* dinv,
                          const float2* tw, hipStream_t st) {
  const RowArgs a{u1, T, g, dinv, tw};
#define CALL(LP)                                                                                                 \
  {                                                                                                              \
    using Full = RowCfg<LP, LP>;                                                                                 \
    using Half = RowCfg<LP - 1, LP>;                                                                             \
    if (g.Nin < g.Np)                                                                                            \
      return launch_or_record<RowArgs, t2_rows_body<LP, true>, Half::NT>(a, (g.Nin + Half::C - 1) / Half::C,     \
                                                                         Half::LDS, st);                         \
    return launch_or_record<RowArgs, t2_rows_body<LP, false>, Full::NT>(a, (g.Nin + Full::C - 1) / Full::C,      \
                                                                        Full::LDS, st);                          \
  }
  NUASM_DISPATCH_NP(logNp, CALL)
#undef CALL
  return hipErrorInvalidValue;
}

hipError_t launch_t2_cols(int logNpf, int logNp, const float2* T, float2* V, GridGeom g, Spectral sp,
                          const float2* tw, hipStream_t st) {
  const int d = logNp - logNpf;
#define CALL(LP) return cols_by_reduction<LP, false>(d, T, V, g, sp, tw, st)
  NUASM_DISPATCH_NP(logNp, CALL)
#undef CALL
  return hipErrorInvalidValue;
}

hipError_t launch_t2_rows_inv(int logNp, const float2* V, float2* fine, GridGeom g, const float2* tw,
                              hipStream_t st) {
  const RowArgs a{V, fine, g, nullptr, tw};
#define CALL(LP)                                                                                    \
  {                                                                                                 \
    using Cfg = RowCfg<LP, LP + 1>;                                                                 \
    return launch_or_record<RowArgs, t2_rows_inv_body<LP>, Cfg::NT>(a, (g.L + Cfg::C - 1) / Cfg::C, \
                                                                    Cfg::LDS, st);                  \
  }
  NUASM_DISPATCH_NP(logNp, CALL)
#undef CALL
  return hipErrorInvalidValue;
}

hipError_t launch_t3_cols(int logNp, const float2* T, float2* V, GridGeom g, Spectral sp,
                          const float2* tw, hipStream_t st) {
#define CALL(LP)                                                                         \
  {                                                                                      \
    using Cfg = ColCfg<LP, LP + 1>;                                                      \
    hipError_t e = set_lds(k_t3_cols<LP>, Cfg::LDS);                                     \
    if (e != hipSuccess) return e;                                                       \
    const int grid = band_strips(g, 1 << LP, Cfg::C);                                    \
    if (grid <= 0) return hipSuccess;                                                    \
    hipLaunchKernelGGL(k_t3_cols<LP>, dim3(grid), dim3(Cfg::NT), Cfg::LDS, st, T, V, g, sp, tw); \
  }
  NUASM_DISPATCH_NP(logNp, CALL)
#undef CALL
  return hipGetLastError();
}

hipError_t launch_fft_rows(int logn, int64_t batch, int sign, const float2* in, float2* out,
                           const float2* tw, hipStream_t st) {
#define CALL2(LN, D)                                                                     \
  {                                                                                      \
    using Cfg = RowCfg<LN - 1, LN>;                                                      \
    hipError_t e = set_lds(k_fft_rows<LN, D>, Cfg::LDS);                                 \
    if (e != hipSuccess) return e;                                                       \
    const int64_t grid = (batch + Cfg::C - 1) / Cfg::C;                                  \
    hipLaunchKernelGGL((k_fft_rows<LN, D>), dim3((unsigned)grid), dim3(Cfg::NT), Cfg::LDS, st, in, out, batch, tw); \
  }
#define CALL(LN) \
  if (sign < 0) CALL2(LN, -1) else CALL2(LN, 1)
  switch (logn) {
    case 5: CALL(5); break;
    case 6: CALL(6); break;
    case 7: CALL(7); break;
    case 8: CALL(8); break;
    case 9: CALL(9); break;
    case 10: CALL(10); break;
    case 11: CALL(11); break;
    case 12: CALL(12); break;
    case 13: CALL(13); break;
    case 14: CALL(14); break;
    default: return hipErrorInvalidValue;
  }
#undef CALL
#undef CALL2
  return hipGetLastError();
}

hipError_t launch_transfer_table(const GridGeom& g, const Spectral& sp, float2* out, hipStream_t st) {
  const int64_t n = (int64_t)g.Np * g.Np;
  hipLaunchKernelGGL(k_transfer_table, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, g, sp, out);
  return hipGetLastError();
}

hipError_t launch_fresnel_axis(int Np, double g, double two_lam_z, double o, double2 amp,
                               float2* out, hipStream_t st) {
  hipLaunchKernelGGL(k_fresnel_axis, dim3(Np), dim3(kFresnelThreads), 0, st, Np, g, two_lam_z, o, amp, out);
  return hipGetLastError();
}

}  // namespace nuasm
