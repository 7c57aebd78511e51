// Device helpers shared by the gfx950 kernels: complex arithmetic, the
// register-level DFT butterflies, the LDS Stockham FFT, and the
// exponential-of-semicircle spreading kernel.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace nuasm {

// ------------------------------------------------------------ complex math
__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
__device__ __forceinline__ float2 cscale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }
__device__ __forceinline__ float2 cconj(float2 a) { return make_float2(a.x, -a.y); }
__device__ __forceinline__ float2 czero() { return make_float2(0.f, 0.f); }

// exp(2 pi i x) for x in [-1/2, 1/2] cycles from the hardware sine and cosine,
// which take their argument in revolutions (v_sin_f32 / v_cos_f32; measured
// error below 1.3e-7 over that range, against 5.5e-8 for sincospif).
__device__ __forceinline__ float2 cis_rev(float x) {
  return make_float2(__builtin_amdgcn_cosf(x), __builtin_amdgcn_sinf(x));
}

// cos / sin of 2 pi m / 16 for m = 0..8 (exact decimal expansions)
__device__ __forceinline__ float cos16(int m) {
  switch (m) {
    case 0: return 1.0f;
    case 1: return 0.92387953251128675613f;
    case 2: return 0.70710678118654752440f;
    case 3: return 0.38268343236508977173f;
    case 4: return 0.0f;
    case 5: return -0.38268343236508977173f;
    case 6: return -0.70710678118654752440f;
    case 7: return -0.92387953251128675613f;
    default: return -1.0f;
  }
}
__device__ __forceinline__ float sin16(int m) { return cos16(m < 4 ? 4 - m : m - 4) * (m <= 8 ? 1.f : -1.f); }

// w * exp(DIR * 2 pi i m / 16), m compile-time after unrolling.
template <int DIR>
__device__ __forceinline__ float2 rot16(int m, float2 v) {
  if (m == 0) return v;
  if (m == 4) return DIR < 0 ? make_float2(v.y, -v.x) : make_float2(-v.y, v.x);
  const float c = cos16(m);
  const float s = DIR < 0 ? -sin16(m) : sin16(m);
  return make_float2(c * v.x - s * v.y, c * v.y + s * v.x);
}

// (a, b) -> (a + w b, a - w b): the sum in four fused multiply-adds, the
// difference as 2 a less the sum in two.
__device__ __forceinline__ void bfly(float2& a, float2& b, float2 w) {
  const float2 r = make_float2(fmaf(-w.y, b.y, fmaf(w.x, b.x, a.x)), fmaf(w.y, b.x, fmaf(w.x, b.y, a.y)));
  b = make_float2(fmaf(2.f, a.x, -r.x), fmaf(2.f, a.y, -r.y));
  a = r;
}
// the same with w = 1, and with w = exp(DIR i pi / 2)
__device__ __forceinline__ void bfly1(float2& a, float2& b) {
  const float2 r = cadd(a, b);
  b = csub(a, b);
  a = r;
}
template <int DIR>
__device__ __forceinline__ void bfly_i(float2& a, float2& b) {
  const float2 t = DIR < 0 ? make_float2(b.y, -b.x) : make_float2(-b.y, b.x);
  const float2 r = cadd(a, t);
  b = csub(a, t);
  a = r;
}

// X[k] = sum_j x[j] w^j exp(DIR 2 pi i j k / R) in place, natural order, for
// R = 2, 4, 8, by radix-2 decimation in time.  The twiddles of the pass are
// taken inside the butterflies (w, w^2, w^4 and their rotations), six
// operations each: 72 for R = 8 and 16 for the powers, where separate products
// by w .. w^7 and a plain transform took 84 and 24.
// PH: the pass has no twiddles of its own (w = exp(DIR 2 pi i PH / 16), PH = 0,
// or 1 for the half-shifted first pass of radix 8); else w is given, and w4 = w^4
// for radix 8.
template <int R, int DIR, int PH>
__device__ __forceinline__ void dft_tw(float2 (&x)[R], float2 w, float2 w4) {
  if constexpr (R == 2) {
    bfly(x[0], x[1], w);
  } else if constexpr (R == 4) {
    const float2 w2 = cmul(w, w);
    float2 e0 = x[0], e1 = x[2], o0 = x[1], o1 = x[3];
    bfly(e0, e1, w2);
    bfly(o0, o1, w2);
    bfly(e0, o0, w);
    bfly(e1, o1, rot16<DIR>(4, w));
    x[0] = e0;
    x[1] = e1;
    x[2] = o0;
    x[3] = o1;
  } else {
    static_assert(R == 8, "radix 2, 4 or 8");
    // x[j]: even half (0, 4), (2, 6), odd half (1, 5), (3, 7)
    const float2 one = make_float2(1.f, 0.f);
    if constexpr (PH == 0) {
      bfly1(x[0], x[4]);
      bfly1(x[2], x[6]);
      bfly1(x[1], x[5]);
      bfly1(x[3], x[7]);
      bfly1(x[0], x[2]);
      bfly_i<DIR>(x[4], x[6]);
      bfly1(x[1], x[3]);
      bfly_i<DIR>(x[5], x[7]);
      bfly1(x[0], x[1]);
      bfly(x[4], x[5], rot16<DIR>(2, one));
      bfly_i<DIR>(x[2], x[3]);
      bfly(x[6], x[7], rot16<DIR>(6, one));
    } else {
      float2 w1 = w, w2;
      if constexpr (PH > 0) {
        w1 = rot16<DIR>(PH, one);
        w2 = rot16<DIR>(2 * PH, one);
        bfly_i<DIR>(x[0], x[4]);
        bfly_i<DIR>(x[2], x[6]);
        bfly_i<DIR>(x[1], x[5]);
        bfly_i<DIR>(x[3], x[7]);
        static_assert(PH <= 1, "w^4 is a quarter turn");
      } else {
        w2 = cmul(w, w);
        bfly(x[0], x[4], w4);
        bfly(x[2], x[6], w4);
        bfly(x[1], x[5], w4);
        bfly(x[3], x[7], w4);
      }
      const float2 w2i = rot16<DIR>(4, w2);
      bfly(x[0], x[2], w2);
      bfly(x[4], x[6], w2i);
      bfly(x[1], x[3], w2);
      bfly(x[5], x[7], w2i);
      const float2 w1e = PH > 0 ? rot16<DIR>(2 + PH, one) : rot16<DIR>(2, w1);
      bfly(x[0], x[1], w1);
      bfly(x[4], x[5], w1e);
      bfly(x[2], x[3], rot16<DIR>(4, w1));
      bfly(x[6], x[7], rot16<DIR>(4, w1e));
    }
    // (x0, x4, x2, x6 | x1, x5, x3, x7) hold X0, X1, X2, X3 | X4, X5, X6, X7
    const float2 t1 = x[4], t2 = x[2], t3 = x[6], t4 = x[1], t6 = x[3];
    x[1] = t1;
    x[2] = t2;
    x[3] = t3;
    x[4] = t4;
    x[6] = t6;
  }
}

// LDS index with one pad slot per 16 complex elements: breaks the stride-16
// bank pattern of the first Stockham pass.
__host__ __device__ constexpr int pidx(int e) { return e + (e >> 4); }
__host__ __device__ constexpr int lds_elems(int n) { return n + (n >> 4) + 1; }

// Two-level twiddle table for length N = 2^LOGN, held in LDS:
// hi[i] = exp(-2 pi i 64 i / N) for i < HI, lo[j] = exp(-2 pi i j / N) for
// j < 64, so exp(-2 pi i m / N) = hi[m >> 6] * lo[m & 63] for every m < N
// (one complex product, about one float32 ulp).  Staging it costs SIZE
// entries instead of N and keeps twiddles out of global memory.
template <int LOGN>
struct Tw2 {
  static constexpr int N = 1 << LOGN;
  static constexpr int HI = N >= 64 ? N / 64 : 1;
  static constexpr int SIZE = HI + 64;
};

// Fill dst[0 .. Tw2::SIZE) from the global table tw[m] = exp(-2 pi i m / N).
template <int LOGN, int NT>
__device__ __forceinline__ void load_tw2(float2* __restrict__ dst, const float2* __restrict__ tw) {
  using T = Tw2<LOGN>;
  for (int e = threadIdx.x; e < T::SIZE; e += NT)
    dst[e] = e < T::HI ? tw[(e * 64) & (T::N - 1)] : tw[(e - T::HI) & (T::N - 1)];
}

template <int LOGN>
__device__ __forceinline__ float2 tw2_get(const float2* __restrict__ t, int m) {
  return cmul(t[m >> 6], t[Tw2<LOGN>::HI + (m & 63)]);
}

// Stockham transforms of C interleaved columns of length N = 2^LOGN whose data
// live in registers between the passes' LDS exchanges.  Thread t < NA = C N / 8
// of the workgroup's NT works on column c = t % C and owns the eight elements
// i0 + m N / 8, m = 0 .. 7, i0 = t / C, before the transform and after it: a
// caller loads its first pass's inputs straight into registers, uses the
// outputs from registers, and chains two transforms of one length without an
// exchange.  Passes of radix 8 with a 4 or 2 tail (two or four butterflies a
// thread); the exchanges use element e of column c at pidx(e C + c).
//
// HALF: the transform at the frequencies k + 1/2,
//   X[k] = sum_t x[t] exp(DIR 2 pi i t (k + 1/2) / N).
// Decimation in time carries the half through every pass (the sub-transforms
// are half-shifted too), so it only changes the twiddles' index from k to
// k + 1/2.  A transform of length 2 N whose input or output is half zero then
// splits into two of length N, plain and half-shifted, one after the other in
// half the LDS: with x zero outside N elements, X[2 q + p] is the transform of
// x at q + p / 2.
//
// tw: LDS two-level table (Tw2) of length 2^TL, TL > LOGN for HALF.  The LDS
// may still be in use by other threads when a transform begins (its first
// pass waits before it writes); nothing is left in LDS at the end, but other
// threads may still be reading.
// Largest LOGN whose w^4 is a table value too, and not the square of a square
// (five roundings, at four times the first one's weight).  Error of
// transforms of twice the length on random data, with squares and so: 256
// 1.31e-7 and 1.11e-7, 1024 2.55e-7 and 1.74e-7, 2048 2.67e-7 and 1.81e-7; of a
// plane with few modes (N = 256, Fresnel, z = 0.43 m), whose errors add up
// rather than average out, 9.1e-7 and 7.6e-7 (8.4e-7 with full-length
// transforms and the twiddles as separate factors).  The same number of
// products and one or two LDS reads more: no difference in time up to 2^10
// (N' = 2048, Fresnel type 2 of 2^20 points 112.1 and 111.5 us), 1 % at 2^11 and
// beyond (114.5 and 116), where squares already err less than those factors did.
constexpr int kTableW4 = 10;

template <int LOGN, int C, int NT, int DIR, bool HALF, int TL, int P, int REM>
__device__ __forceinline__ void reg_fft_pass(float2* __restrict__ s, const float2* __restrict__ tw, int tid,
                                             float2 (&x)[8]) {
  constexpr int N = 1 << LOGN, LR = REM >= 3 ? 3 : REM, R = 1 << LR, NR = N / R, PER = 8 / R;
  constexpr int NA = C * N / 8, TWS = N / (P * R);
  constexpr bool FIRST = P == 1, LAST = REM == LR;
  static_assert(!FIRST || R == 8, "the first pass is radix 8");
  static_assert(!FIRST || !LAST, "at least two passes");
  static_assert(!HALF || TL > LOGN, "half-shifted twiddles need the table of twice the length");
  static_assert(NA <= NT, "eight elements per thread");
  const bool act = NA == NT || tid < NA;
  const int c = tid % C, i0 = tid / C;
  if (act) {
#pragma unroll
    for (int q = 0; q < PER; ++q) {
      const int i = i0 + q * (N / 8);
      const int k = i & (P - 1);
      float2 y[R];
      if constexpr (FIRST) {
#pragma unroll
        for (int j = 0; j < R; ++j) y[j] = x[j];
        dft_tw<R, DIR, HALF ? 1 : 0>(y, czero(), czero());
      } else {
        if constexpr ((NR * C) % 16 == 0) {
          // inputs NR * C elements apart: one padded address and constant
          // offsets when the stride is a whole number of pad groups
          const int p0 = pidx(i * C + c);
#pragma unroll
          for (int j = 0; j < R; ++j) y[j] = s[p0 + j * pidx(NR * C)];
        } else {
#pragma unroll
          for (int j = 0; j < R; ++j) y[j] = s[pidx((i + j * NR) * C + c)];
        }
        // exp(-2 pi i (k + HALF/2) TWS / N)
        const int idx = TL > LOGN ? ((2 * k + (HALF ? 1 : 0)) * TWS) << (TL > LOGN ? TL - LOGN - 1 : 0) : k * TWS;
        float2 w = tw2_get<TL>(tw, idx);
        if (DIR > 0) w.y = -w.y;
        float2 w4 = czero();
        if constexpr (R == 8 && LOGN <= kTableW4) {
          w4 = tw2_get<TL>(tw, (4 * idx) & ((1 << TL) - 1));
          if (DIR > 0) w4.y = -w4.y;
        } else if constexpr (R == 8) {
          w4 = cmul(w, w);
          w4 = cmul(w4, w4);
        }
        dft_tw<R, DIR, -1>(y, w, w4);
      }
      // register j * PER + q: in the last pass that is element i0 + m N / 8,
      // m = q + j 8 / R
#pragma unroll
      for (int j = 0; j < R; ++j) x[j * PER + q] = y[j];
    }
  }
  if constexpr (!LAST) {
    __syncthreads();
    if (act) {
#pragma unroll
      for (int q = 0; q < PER; ++q) {
        const int i = i0 + q * (N / 8);
        const int k = i & (P - 1);
        const int base = (i - k) * R + k;
        if constexpr ((P * C) % 16 == 0) {
          const int p0 = pidx(base * C + c);
#pragma unroll
          for (int j = 0; j < R; ++j) s[p0 + j * pidx(P * C)] = x[j * PER + q];
        } else {
#pragma unroll
          for (int j = 0; j < R; ++j) s[pidx((base + j * P) * C + c)] = x[j * PER + q];
        }
      }
    }
    __syncthreads();
    reg_fft_pass<LOGN, C, NT, DIR, HALF, TL, P * R, REM - LR>(s, tw, tid, x);
  }
}

template <int LOGN, int C, int NT, int DIR, bool HALF, int TL>
__device__ __forceinline__ void reg_fft(float2* __restrict__ s, const float2* __restrict__ tw, int tid,
                                        float2 (&x)[8]) {
  reg_fft_pass<LOGN, C, NT, DIR, HALF, TL, 1, LOGN>(s, tw, tid, x);
}

// Exchange between lanes of a pair (quad permutation 1, 0, 3, 2).
__device__ __forceinline__ float pair_swap(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xb1, 0xf, 0xf, false));
}

// A copy of the thread index that the compiler cannot tie to the first: a
// kernel with several transforms recomputes its LDS addresses in each instead
// of keeping them all live.
__device__ __forceinline__ int opaque_tid() {
  int t = (int)threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// ------------------------------------------------- spreading kernel (ES)
// psi(d) = exp(beta (sqrt(1 - (2d/w)^2) - 1)) for |d| <= w/2, 0 outside
// (Barnett, Magland and af Klinteberg, SIAM J. Sci. Comput. 2019).
__device__ __forceinline__ float es_kernel(float d, float two_over_w, float beta) {
  const float t = d * two_over_w;
  const float r = 1.0f - t * t;
  return r > 0.0f ? expf(beta * (sqrtf(r) - 1.0f)) : 0.0f;
}

// es_kernel with the hardware exp2 and square root (v_exp_f32, v_sqrt_f32):
// absolute error below 3e-8 of the kernel's peak value 1.
__device__ __forceinline__ float es_kernel_fast(float d, float two_over_w, float beta_log2e) {
  const float t = d * two_over_w;
  const float r = 1.0f - t * t;
  return r > 0.0f ? __builtin_amdgcn_exp2f(beta_log2e * (__builtin_amdgcn_sqrtf(r) - 1.0f)) : 0.0f;
}

// The weights of all W taps of one axis with one or two operations less each:
// d is the first tap's offset, tap m lies at d + m.
template <int W>
__device__ __forceinline__ void es_weights(float d, float two_over_w, float beta_log2e, float (&w)[W]) {
  const float u = d * two_over_w;
#pragma unroll
  for (int m = 0; m < W; ++m) {
    const float t = fmaf((float)m, two_over_w, u);
    const float r = fmaf(-t, t, 1.0f);
    const float e = __builtin_amdgcn_exp2f(fmaf(beta_log2e, __builtin_amdgcn_sqrtf(r), -beta_log2e));
    w[m] = r > 0.0f ? e : 0.0f;
  }
}

// Bin record: one (point, bin) pair.  lx, ly: first tap relative to the bin
// origin (int8 each), bit 16: the bin holds the point's first tap; dx, dy:
// offset of the first tap from the point in fine cells; idx: caller's point
// index.
struct __align__(16) BinRec {
  int32_t packed;
  float dx, dy;
  int32_t idx;
};

__device__ __forceinline__ int rec_lx(int32_t p) { return (int)(int8_t)(p & 0xff); }
__device__ __forceinline__ int rec_ly(int32_t p) { return (int)(int8_t)((p >> 8) & 0xff); }
__device__ __forceinline__ bool rec_primary(int32_t p) { return (p >> 16) & 1; }

// blockIdx -> work index such that consecutive work items land on the same
// XCD (the dispatcher deals workgroups round-robin over the 8 XCDs, each with
// its own L2).  `count` must be the grid size.
__device__ __forceinline__ int xcd_remap(int bid, int count) {
  constexpr int XCD = 8;
  const int per = count / XCD;
  if (per == 0 || bid >= per * XCD) return bid;
  return (bid % XCD) * per + bid / XCD;
}

}  // namespace nuasm
