// Device helpers shared by the kernel files: complex arithmetic, FFT
// butterflies and LDS stages, cross-lane exchanges, reductions and the
// pointwise pieces of Alg. 1.
#pragma once

#include <cfloat>
#include <climits>

#include "host_math.h"
#include "shot_internal.h"

namespace shot {

template <typename T>
__device__ __forceinline__ cpx<T> cadd(cpx<T> a, cpx<T> b) { return {a.x + b.x, a.y + b.y}; }
template <typename T>
__device__ __forceinline__ cpx<T> csub(cpx<T> a, cpx<T> b) { return {a.x - b.x, a.y - b.y}; }
template <typename T>
__device__ __forceinline__ cpx<T> cmul(cpx<T> a, cpx<T> b) {
  return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
template <typename T>
__device__ __forceinline__ cpx<T> cscale(cpx<T> a, T s) { return {a.x * s, a.y * s}; }
// multiply by s*i (s = +-1)
template <typename T>
__device__ __forceinline__ cpx<T> cmul_si(cpx<T> a, T s) { return {-s * a.y, s * a.x}; }

// ---------------------------------------------------------------------------
// Mixed-radix Stockham FFT in LDS, radices 2, 3, 4, 5.  sign = -1 forward,
// +1 inverse (unnormalised).  All threads of the block must call it.  Returns
// the buffer that holds the result (natural order).
// ---------------------------------------------------------------------------
// cos and sin of 2 pi e / R, e = 0 .. R-1: the internal twiddles of the
// register-level composite radices
template <int R>
struct UnitRoots;
template <>
struct UnitRoots<8> {
  static constexpr double c[8] = {1.0, 0.70710678118654752440, 0.0, -0.70710678118654752440,
                                  -1.0, -0.70710678118654752440, 0.0, 0.70710678118654752440};
  static constexpr double s[8] = {0.0, 0.70710678118654752440, 1.0, 0.70710678118654752440,
                                  0.0, -0.70710678118654752440, -1.0, -0.70710678118654752440};
};
template <>
struct UnitRoots<9> {
  static constexpr double c[9] = {1.0, 0.76604444311897803520, 0.17364817766693034885, -0.5,
                                  -0.93969262078590838405, -0.93969262078590838405, -0.5,
                                  0.17364817766693034885, 0.76604444311897803520};
  static constexpr double s[9] = {0.0, 0.64278760968653932632, 0.98480775301220805937, 0.86602540378443864676,
                                  0.34202014332566873304, -0.34202014332566873304, -0.86602540378443864676,
                                  -0.98480775301220805937, -0.64278760968653932632};
};

template <typename T, int R>
__device__ __forceinline__ void butterfly(cpx<T>* v, T s) {
  if constexpr (R == 2) {
    cpx<T> a = v[0], b = v[1];
    v[0] = cadd(a, b);
    v[1] = csub(a, b);
  } else if constexpr (R == 4) {
    cpx<T> t0 = cadd(v[0], v[2]), t1 = csub(v[0], v[2]);
    cpx<T> t2 = cadd(v[1], v[3]), t3 = cmul_si(csub(v[1], v[3]), s);
    v[0] = cadd(t0, t2);
    v[2] = csub(t0, t2);
    v[1] = cadd(t1, t3);
    v[3] = csub(t1, t3);
  } else if constexpr (R == 3) {
    const T c = (T)-0.5, sn = s * (T)0.86602540378443864676;
    cpx<T> t = cadd(v[1], v[2]), d = csub(v[1], v[2]);
    cpx<T> base = {v[0].x + c * t.x, v[0].y + c * t.y};
    cpx<T> rot = cmul_si(d, sn);  // i * sn * d
    v[0] = cadd(v[0], t);
    v[1] = cadd(base, rot);
    v[2] = csub(base, rot);
  } else if constexpr (R == 5) {
    const T c1 = (T)0.30901699437494742410, c2 = (T)-0.80901699437494742410;
    const T s1 = s * (T)0.95105651629515357212, s2 = s * (T)0.58778525229247312917;
    cpx<T> t1 = cadd(v[1], v[4]), d1 = csub(v[1], v[4]);
    cpx<T> t2 = cadd(v[2], v[3]), d2 = csub(v[2], v[3]);
    cpx<T> b1 = {v[0].x + c1 * t1.x + c2 * t2.x, v[0].y + c1 * t1.y + c2 * t2.y};
    cpx<T> b2 = {v[0].x + c2 * t1.x + c1 * t2.x, v[0].y + c2 * t1.y + c1 * t2.y};
    cpx<T> e1 = {s1 * d1.x + s2 * d2.x, s1 * d1.y + s2 * d2.y};
    cpx<T> e2 = {s2 * d1.x - s1 * d2.x, s2 * d1.y - s1 * d2.y};
    cpx<T> r1 = cmul_si(e1, (T)1), r2 = cmul_si(e2, (T)1);
    v[0] = cadd(v[0], cadd(t1, t2));
    v[1] = cadd(b1, r1);
    v[4] = csub(b1, r1);
    v[2] = cadd(b2, r2);
    v[3] = csub(b2, r2);
  } else if constexpr (R == 8 || R == 9) {
    // R = R1 R2 in registers: with r = R2 r1 + r2 and q = q1 + R1 q2,
    // X[q] = sum_r2 w_R2^(r2 q2) w_R^(r2 q1) sum_r1 w_R1^(r1 q1) v[R2 r1 + r2]
    constexpr int R1 = R == 9 ? 3 : 4, R2 = R / R1;
    cpx<T> y[R2][R1];
#pragma unroll
    for (int r2 = 0; r2 < R2; ++r2) {
#pragma unroll
      for (int r1 = 0; r1 < R1; ++r1) y[r2][r1] = v[R2 * r1 + r2];
      butterfly<T, R1>(y[r2], s);
    }
#pragma unroll
    for (int r2 = 1; r2 < R2; ++r2)
#pragma unroll
      for (int q1 = 1; q1 < R1; ++q1) {
        const int e = r2 * q1;  // w_R^e = cos(2 pi e / R) + i s sin(2 pi e / R)
        y[r2][q1] = cmul(y[r2][q1], cpx<T>{(T)UnitRoots<R>::c[e], s * (T)UnitRoots<R>::s[e]});
      }
#pragma unroll
    for (int q1 = 0; q1 < R1; ++q1) {
      cpx<T> z[R2];
#pragma unroll
      for (int r2 = 0; r2 < R2; ++r2) z[r2] = y[r2][q1];
      butterfly<T, R2>(z, s);
#pragma unroll
      for (int q2 = 0; q2 < R2; ++q2) v[q1 + R1 * q2] = z[q2];
    }
  }
}

template <typename T, int R>
__device__ __forceinline__ void stockham_stage(const cpx<T>* __restrict__ src, cpx<T>* __restrict__ dst,
                                               int N, int Ns, const cpx<T>* __restrict__ tw, T sign) {
  const int NR = N / R;
  const int twstride = N / (Ns * R);
  for (int b = threadIdx.x; b < NR; b += blockDim.x) {
    const int k = b % Ns;
    cpx<T> v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = src[b + r * NR];
#pragma unroll
    for (int r = 1; r < R; ++r) {
      cpx<T> w = tw[r * k * twstride];
      w.y *= -sign;  // table holds exp(-2 pi i k/N); inverse uses the conjugate
      v[r] = cmul(v[r], w);
    }
    butterfly<T, R>(v, sign);
    const int base = (b / Ns) * Ns * R + k;
#pragma unroll
    for (int r = 0; r < R; ++r) dst[base + r * Ns] = v[r];
  }
}

// Stockham stage of any radix R (the primes above 5 of ring lengths that are
// not 2,3,5-smooth): each thread forms whole outputs, output q of butterfly b
// being sum_r src[b + r N/R] w^{r (k N/(Ns R) + q N/R)} with w the length-N
// root, so every term costs one table lookup.
template <typename T>
__device__ __forceinline__ void stockham_stage_generic(const cpx<T>* __restrict__ src, cpx<T>* __restrict__ dst, int N, int Ns,
                                       int R, const cpx<T>* __restrict__ tw, T sign) {
  const int NR = N / R;
  const int twstride = N / (Ns * R);
  for (int o = threadIdx.x; o < N; o += blockDim.x) {
    const int q = o / NR, b = o - q * NR;
    const int k = b % Ns;
    const int e = k * twstride + q * NR;
    cpx<T> acc = {(T)0, (T)0};
    int idx = 0;  // r * e mod N, advanced by e (< N, so one subtraction wraps it)
    int r = 0;
    // eight terms per step: their LDS reads are all in flight before the first use
    for (; r + 8 <= R; r += 8) {
      int ix[8];
      cpx<T> v[8], w[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        ix[j] = idx;
        idx += e;
        idx = idx >= N ? idx - N : idx;
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        v[j] = src[b + (r + j) * NR];
        w[j] = tw[ix[j]];
      }
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        w[j].y *= -sign;  // table holds exp(-2 pi i k/N); inverse uses the conjugate
        acc = cadd(acc, cmul(v[j], w[j]));
      }
    }
    for (; r < R; ++r) {
      cpx<T> w = tw[idx];
      w.y *= -sign;
      acc = cadd(acc, cmul(src[b + r * NR], w));
      idx += e;
      idx = idx >= N ? idx - N : idx;
    }
    dst[(b / Ns) * Ns * R + k + q * Ns] = acc;
  }
}

template <typename T>
__device__ __forceinline__ cpx<T>* fft_lds(cpx<T>* a, cpx<T>* b, int N, const int* fac, int nfac,
                           const cpx<T>* __restrict__ tw, T sign) {
  int Ns = 1;
  cpx<T>* src = a;
  cpx<T>* dst = b;
  for (int s = 0; s < nfac; ++s) {
    const int R = fac[s];
    switch (R) {
      case 2: stockham_stage<T, 2>(src, dst, N, Ns, tw, sign); break;
      case 3: stockham_stage<T, 3>(src, dst, N, Ns, tw, sign); break;
      case 4: stockham_stage<T, 4>(src, dst, N, Ns, tw, sign); break;
      case 5: stockham_stage<T, 5>(src, dst, N, Ns, tw, sign); break;
      default: stockham_stage_generic<T>(src, dst, N, Ns, R, tw, sign); break;
    }
    __syncthreads();
    cpx<T>* t = src;
    src = dst;
    dst = t;
    Ns *= R;
  }
  return src;
}

// Compile-time factorisation (same radix order as the host: 4, 2, 3, 5) for
// the common transform lengths: every stage's length, stride and twiddle step
// become constants, so the index arithmetic needs no runtime division.
struct FacList {
  int n;
  int r[12];
};
__host__ __device__ constexpr FacList factorize(int N) {
  FacList f{0, {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0}};
  const int rs[4] = {4, 2, 3, 5};
  for (int i = 0; i < 4; ++i)
    while (N % rs[i] == 0 && f.n < 12) {
      f.r[f.n++] = rs[i];
      N /= rs[i];
    }
  return f;
}
// The compile-time stages fuse a radix 4 with the radix 2 and pairs of
// radix 3 into register-level radix-8 and radix-9 stages: fewer LDS passes
// and barriers, and every stage of a 1440-point row fits one pass of 512
// threads (4, 8, 9, 5 instead of 4, 4, 2, 3, 3, 5; three heavier stages
// 16, 10, 9 leave too few threads busy and measured slower).
__host__ __device__ constexpr FacList fuse_factors(FacList f) {
  FacList g{0, {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0}};
  int n4 = 0, n2 = 0, n3 = 0, n5 = 0;
  for (int i = 0; i < f.n; ++i) {
    if (f.r[i] == 4) ++n4;
    else if (f.r[i] == 2) ++n2;
    else if (f.r[i] == 3) ++n3;
    else ++n5;
  }
  const int n8 = (n4 > 0 && n2 > 0) ? 1 : 0;
  for (int i = 0; i < n4 - n8; ++i) g.r[g.n++] = 4;
  for (int i = 0; i < n8; ++i) g.r[g.n++] = 8;
  for (int i = 0; i < n2 - n8; ++i) g.r[g.n++] = 2;
  for (int i = 0; i < n3 / 2; ++i) g.r[g.n++] = 9;
  for (int i = 0; i < n3 % 2; ++i) g.r[g.n++] = 3;
  for (int i = 0; i < n5; ++i) g.r[g.n++] = 5;
  return g;
}
__host__ __device__ constexpr int fac_prefix(FacList f, int s) {
  int p = 1;
  for (int i = 0; i < s; ++i) p *= f.r[i];
  return p;
}

template <typename T, int R, int N, int Ns>
__device__ __forceinline__ void stockham_stage_c(const cpx<T>* __restrict__ src, cpx<T>* __restrict__ dst,
                                                 const cpx<T>* __restrict__ tw, T sign) {
  constexpr int NR = N / R;
  constexpr int twstride = N / (Ns * R);
  for (int b = threadIdx.x; b < NR; b += blockDim.x) {
    const int k = b % Ns;
    cpx<T> v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = src[b + r * NR];
#pragma unroll
    for (int r = 1; r < R; ++r) {
      cpx<T> w = tw[r * k * twstride];
      w.y *= -sign;
      v[r] = cmul(v[r], w);
    }
    butterfly<T, R>(v, sign);
    const int base = (b / Ns) * Ns * R + k;
#pragma unroll
    for (int r = 0; r < R; ++r) dst[base + r * Ns] = v[r];
  }
}

template <typename T, int N, int S>
__device__ __forceinline__ void fft_stages_c(cpx<T>*& src, cpx<T>*& dst, const cpx<T>* tw, T sign) {
  constexpr FacList F = fuse_factors(factorize(N));
  if constexpr (S < F.n) {
    constexpr int R = F.r[S];
    constexpr int Ns = fac_prefix(F, S);
    stockham_stage_c<T, R, N, Ns>(src, dst, tw, sign);
    __syncthreads();
    cpx<T>* t = src;
    src = dst;
    dst = t;
    fft_stages_c<T, N, S + 1>(src, dst, tw, sign);
  }
}

// Length chosen at compile time (NC > 0) or at run time (NC == 0).
template <typename T, int NC>
__device__ __forceinline__ cpx<T>* fft_any(cpx<T>* a, cpx<T>* b, int N, const int* fac, int nfac,
                                           const cpx<T>* tw, T sign) {
  if constexpr (NC > 0) {
    cpx<T>* src = a;
    cpx<T>* dst = b;
    fft_stages_c<T, NC, 0>(src, dst, tw, sign);
    return src;
  } else {
    return fft_lds<T>(a, b, N, fac, nfac, tw, sign);
  }
}

// ---------------------------------------------------------------------------
// Cross-lane exchanges without LDS round trips: DPP row permutes for lane
// bits 0-3, permlane swaps (gfx950) for bits 4 and 5.
// ---------------------------------------------------------------------------
__device__ __forceinline__ float dpp_f(float v, int ctrl_sel) {
  int x = __float_as_int(v);
  int r;
  switch (ctrl_sel) {
    case 0: r = __builtin_amdgcn_update_dpp(0, x, 0x140, 0xf, 0xf, false); break;  // row_mirror (bit 3)
    case 1: r = __builtin_amdgcn_update_dpp(0, x, 0x141, 0xf, 0xf, false); break;  // row_half_mirror (bit 2)
    case 2: r = __builtin_amdgcn_update_dpp(0, x, 0x4e, 0xf, 0xf, false); break;   // quad_perm [2,3,0,1] (bit 1)
    default: r = __builtin_amdgcn_update_dpp(0, x, 0xb1, 0xf, 0xf, false); break;  // quad_perm [1,0,3,2] (bit 0)
  }
  return __int_as_float(r);
}

__device__ __forceinline__ double dpp_d(double v, int ctrl_sel) {
  const unsigned long long u = __double_as_longlong(v);
  float lo = __int_as_float((int)(u & 0xffffffffull)), hi = __int_as_float((int)(u >> 32));
  const unsigned long long rl = (unsigned)__float_as_int(dpp_f(lo, ctrl_sel));
  const unsigned long long rh = (unsigned)__float_as_int(dpp_f(hi, ctrl_sel));
  return __longlong_as_double((long long)(rl | (rh << 32)));
}

// new value = X(lane) + X(lane ^ 32) for lanes < 32, Y(lane ^ 32) + Y(lane) above.
__device__ __forceinline__ float swap_add32(float X, float Y) {
  auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(X), __float_as_uint(Y), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float swap_add16(float X, float Y) {
  auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(X), __float_as_uint(Y), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ double swap_add32(double X, double Y) {
  const unsigned long long x = __double_as_longlong(X), y = __double_as_longlong(Y);
  auto lo = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)y, false, false);
  auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  const double a = __longlong_as_double((long long)((unsigned long long)lo[0] | ((unsigned long long)hi[0] << 32)));
  const double b = __longlong_as_double((long long)((unsigned long long)lo[1] | ((unsigned long long)hi[1] << 32)));
  return a + b;
}
__device__ __forceinline__ double swap_add16(double X, double Y) {
  const unsigned long long x = __double_as_longlong(X), y = __double_as_longlong(Y);
  auto lo = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)y, false, false);
  auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(y >> 32), false, false);
  const double a = __longlong_as_double((long long)((unsigned long long)lo[0] | ((unsigned long long)hi[0] << 32)));
  const double b = __longlong_as_double((long long)((unsigned long long)lo[1] | ((unsigned long long)hi[1] << 32)));
  return a + b;
}

// v of the lane and of its partner across lane bit 4 (permlane16) or bit 5
// (permlane32), returned as (value of the lower lane, value of the upper lane)
// so that both partners see the same ordered pair.
__device__ __forceinline__ void lane_pair16(double v, double& lo, double& hi) {
  const unsigned long long x = __double_as_longlong(v);
  auto a = __builtin_amdgcn_permlane16_swap((unsigned)x, (unsigned)x, false, false);
  auto b = __builtin_amdgcn_permlane16_swap((unsigned)(x >> 32), (unsigned)(x >> 32), false, false);
  lo = __longlong_as_double((long long)((unsigned long long)a[0] | ((unsigned long long)b[0] << 32)));
  hi = __longlong_as_double((long long)((unsigned long long)a[1] | ((unsigned long long)b[1] << 32)));
}
__device__ __forceinline__ void lane_pair32(double v, double& lo, double& hi) {
  const unsigned long long x = __double_as_longlong(v);
  auto a = __builtin_amdgcn_permlane32_swap((unsigned)x, (unsigned)x, false, false);
  auto b = __builtin_amdgcn_permlane32_swap((unsigned)(x >> 32), (unsigned)(x >> 32), false, false);
  lo = __longlong_as_double((long long)((unsigned long long)a[0] | ((unsigned long long)b[0] << 32)));
  hi = __longlong_as_double((long long)((unsigned long long)a[1] | ((unsigned long long)b[1] << 32)));
}

// Wave-wide all-reduction with a commutative op (sum, min, max): at every
// step a lane and its partner combine the same two values, so all 64 lanes
// end with the identical, run-to-run deterministic result.
template <typename Op>
__device__ __forceinline__ double wave_allreduce(double v, Op op) {
  v = op(v, dpp_d(v, 3));  // lane ^ 1
  v = op(v, dpp_d(v, 2));  // lane ^ 2
  v = op(v, dpp_d(v, 1));  // mirror within 8 lanes
  v = op(v, dpp_d(v, 0));  // mirror within 16 lanes
  double lo, hi;
  lane_pair16(v, lo, hi);
  v = op(lo, hi);
  lane_pair32(v, lo, hi);
  return op(lo, hi);
}
struct OpAdd {
  __device__ double operator()(double a, double b) const { return a + b; }
};
struct OpMin {
  __device__ double operator()(double a, double b) const { return fmin(a, b); }
};
struct OpMax {
  __device__ double operator()(double a, double b) const { return fmax(a, b); }
};
__device__ __forceinline__ double wave_sum(double v) { return wave_allreduce(v, OpAdd()); }
__device__ __forceinline__ double wave_min(double v) { return wave_allreduce(v, OpMin()); }
__device__ __forceinline__ double wave_max(double v) { return wave_allreduce(v, OpMax()); }

// ---------------------------------------------------------------------------
// Deterministic block reduction: every thread receives the same value (the
// wave partials are combined in wave order by each thread).
// ---------------------------------------------------------------------------

__device__ double block_sum(double v, double* sh) {
  v = wave_sum(v);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = (blockDim.x + 63) >> 6;
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double r = 0.0;
  for (int i = 0; i < nw; ++i) r += sh[i];
  return r;
}

// Sums of r[0] and r[3], minimum of r[1], maximum of r[2] over the block,
// combined in wave order (as block_sum) with one pair of barriers; sh holds
// 4 doubles per wave.
__device__ void block_reduce4(double* r, double* sh) {
  r[0] = wave_sum(r[0]);
  r[1] = wave_min(r[1]);
  r[2] = wave_max(r[2]);
  r[3] = wave_sum(r[3]);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = (blockDim.x + 63) >> 6;
  __syncthreads();
  if (lane == 0)
    for (int i = 0; i < 4; ++i) sh[4 * w + i] = r[i];
  __syncthreads();
  double a = 0.0, b = INFINITY, c = -INFINITY, d = 0.0;
  for (int i = 0; i < nw; ++i) {
    a += sh[4 * i];
    b = fmin(b, sh[4 * i + 1]);
    c = fmax(c, sh[4 * i + 2]);
    d += sh[4 * i + 3];
  }
  r[0] = a;
  r[1] = b;
  r[2] = c;
  r[3] = d;
}

__device__ double block_min(double v, double* sh) {
  v = wave_min(v);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = (blockDim.x + 63) >> 6;
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double r = sh[0];
  for (int i = 1; i < nw; ++i) r = fmin(r, sh[i]);
  return r;
}

__device__ double block_max(double v, double* sh) {
  v = wave_max(v);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, nw = (blockDim.x + 63) >> 6;
  __syncthreads();
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double r = sh[0];
  for (int i = 1; i < nw; ++i) r = fmax(r, sh[i]);
  return r;
}

// Non-finite outputs count as -inf so that the ratio of that half is -inf.
template <typename T>
__device__ __forceinline__ void track_minmax(double& mn, double& mx, T v) {
  const double d = isfinite(v) ? (double)v : -INFINITY;
  mn = fmin(mn, d);
  mx = fmax(mx, d);
}

template <typename T>
__device__ __forceinline__ bool bad_kernel_value(T x) {
  return !(x > (T)0) || !isfinite(x);
}

// Term u^(-eps/tau) of the unbalanced gauge sums (Alg. 1), taken in the field
// precision: a float32 scaling gives a float32 power (about one ulp, as the
// scaling itself carries); a float64 power of it cost more than the rest of
// an unbalanced row launch.  The sums themselves stay float64.
template <typename T>
__device__ __forceinline__ double gauge_term(T u, double eot) {
  return (double)pow(u, (T)(-eot));
}

// The unbalanced update x -> x^lam (lam = tau/(tau+eps)) and the new value's
// gauge-sum term x^(-lam eps/tau), both from one base-2 logarithm in float32:
// exp2(lam log2 x) is within about |log2 x| ulp of the correctly rounded power
// (about 1e-6 relative for scalings within 2^+-16), and the term's exponent is
// damped by eps/tau.  Zero, infinite and negative x give what the powers give.
// float64 fields keep the library powers.
template <typename T>
__device__ __forceinline__ T unbalanced_update(T x, double lam, double eot, double& term) {
  if constexpr (sizeof(T) == 4) {
    const float y = (float)lam * log2f(x);
    term = (double)exp2f(-(float)eot * y);
    return exp2f(y);
  } else {
    const T xn = pow(x, (T)lam);
    term = gauge_term(xn, eot);
    return xn;
  }
}

template <typename T>
__device__ __forceinline__ T* ubuf_of(const RowArgs<T>& A, int k) { return (k & 1) ? A.ubuf1 : A.ubuf0; }
template <typename T>
__device__ __forceinline__ T* vbuf_of(const RowArgs<T>& A, int k) { return (k & 1) ? A.vbuf1 : A.vbuf0; }

// What a U half that forms the previous iteration's gauge anyway keeps of it for
// the reverse sweep (one thread per item; a launch of its own took 4.5 us).
template <typename T>
__device__ __forceinline__ void store_gauge(const RowArgs<T>& A, int it, double g, double s0, double s1) {
  if (!A.gout) return;
  double* o = A.gout + (size_t)A.gstride * it;
  o[0] = g;
  if (A.gstride == 3) {
    o[1] = s0;
    o[2] = s1;
  }
}

// Gauge g_k: after iteration k the Alg. 1 scalings are u_k = u_hat/g_k and
// v_k = g_k v_hat, with g_k = s = sum u_hat (balanced) or exp(-c/eps) with
// c = tau/2 (log sum a p u_hat^(-eps/tau) - log sum a q v_hat^(-eps/tau)).
template <typename T>
__device__ double gauge(const RowArgs<T>& A, const ItemDev& I, int it, int k, double* sh) {
  const double* R = A.red + ((size_t)(k & 1) * A.nitems_all + it) * (size_t)A.hs * RED_SLOTS;
  double s0 = 0.0, s1 = 0.0;
  for (int q = threadIdx.x; q < A.h; q += blockDim.x) {
    s0 += R[(size_t)q * RED_SLOTS + 0];
    s1 += R[(size_t)q * RED_SLOTS + 1];
  }
  s0 = block_sum(s0, sh);
  s1 = block_sum(s1, sh);
  const double g = I.balanced ? s0 : exp(-(0.5 * I.tau * (log(s0) - log(s1))) / I.eps);
  if (A.mode == ROW_SINK_U && blockIdx.x == 0 && threadIdx.x == 0) store_gauge(A, it, g, s0, s1);
  return g;
}

// Folded spectrum entry (E, O) of order m and row pair jp of item `it`: read
// from the spectrum, or, for an order that the preceding Legendre launch cut
// into parts, the sum of the parts' partial sums taken in part order.
template <typename T>
__device__ __forceinline__ void load_spec_pair(const RowArgs<T>& A, const cpx<T>* spec, int it, int m, int jp,
                                               cpx<T>& ge, cpx<T>& go) {
  if (A.cut) {
    const int2 c = A.cut[m];
    if (c.x > 1) {
      const int rel = it - A.item0, chunk = rel / A.cut_ib, i = rel - chunk * A.cut_ib;
      const cpx<T>* pb = static_cast<const cpx<T>*>(A.pbuf) + (size_t)chunk * A.npb * A.cut_ib * 2 * A.h +
                         (size_t)i * 2 * A.h + 2 * jp;
      ge = {(T)0, (T)0};
      go = {(T)0, (T)0};
      for (int p = 0; p < c.x; ++p) {
        const cpx<T>* q = pb + (size_t)(c.y + p) * A.cut_ib * 2 * A.h;
        ge = cadd(ge, q[0]);
        go = cadd(go, q[1]);
      }
      return;
    }
  }
  const cpx<T>* sp = spec + ((size_t)m * A.h + jp) * 2;
  ge = sp[0];
  go = sp[1];
}

// Bijection of [0, h): workgroup b runs on XCD b % 8; XCD x gets the
// contiguous row-pair range starting at x*(h/8) + min(x, h%8).
__device__ __forceinline__ int xcd_row_pair(int b, int h) {
  const int q = h >> 3, r = h & 7, x = b & 7;
  return x * q + min(x, r) + (b >> 3);
}

// Adjoint notes (balanced Alg. 1, reverse mode).  Forward iteration k:
//   A = K v_{k-1}, u-hat = p / A, B = K u-hat, v-hat = q / B, s = sum u-hat,
//   u_k = u-hat / s, v_k = s v-hat;  cost R = sum a (eps log u_T p + eps log v_T q).
// Only v_k feeds the next iteration, so the reverse sweep carries v-bar:
//   s-bar = sum v-bar (.) v-hat  (- sum u-bar_T (.) u-hat / s^2 at k = T)
//   q-bar += s v-bar v-hat / q,  B-bar = -s v-bar v-hat^2 / q
//   u-hat-bar = s-bar + K^T B-bar (+ u-bar_T / s at k = T)
//   p-bar += u-hat-bar u-hat / p,  A-bar = -u-hat-bar u-hat^2 / p,  v-bar_{k-1} = K^T A-bar
// with K^T x = a (.) K(x / a): the forward FFT skips the area weights and the
// inverse side multiplies by them.  u-bar_T = eps a p / u_T, v-bar_T = eps a q / v_T,
// and the cost contributes eps a log u_T to p-bar and eps a log v_T to q-bar.
//
// Unbalanced iteration k (lambda = tau/(tau+eps), eta = eps/tau):
//   u-hat = (p / K v_{k-1})^lambda, v-hat = (q / K u-hat)^lambda,
//   S_A = sum a p u-hat^-eta, S_B = sum a q v-hat^-eta, g = (S_A / S_B)^(-1/(2 eta)),
//   u_k = u-hat / g, v_k = g v-hat;  cost R = tau sum a (p (1 - u_T^-eta) + q (1 - v_T^-eta)).
// K v_{k-1} = p u-hat^(-1/lambda) and K u-hat = q v-hat^(-1/lambda) are recovered
// pointwise.  Reverse step k, given v-bar_k (at k = T: eps a q v_T^(-eta-1), and
// u-bar_T = eps a p u_T^(-eta-1)):
//   g-bar = sum v-bar v-hat (- sum u-bar_T u-hat / g^2 at k = T)
//   S_A-bar = -g-bar g / (2 eta S_A),  S_B-bar = g-bar g / (2 eta S_B)
//   v-hat-bar = g v-bar - eta S_B-bar a q v-hat^(-eta-1)
//   q-bar += S_B-bar a v-hat^-eta + lambda v-hat-bar v-hat / q,  B-bar = -lambda v-hat-bar v-hat^(1+1/lambda) / q
//   u-hat-bar = K^T B-bar - eta S_A-bar a p u-hat^(-eta-1) (+ u-bar_T / g at k = T)
//   p-bar += S_A-bar a u-hat^-eta + lambda u-hat-bar u-hat / p,  A-bar = -lambda u-hat-bar u-hat^(1+1/lambda) / p
//   v-bar_{k-1} = K^T A-bar;  the cost adds tau a (1 - u_T^-eta) to p-bar and tau a (1 - v_T^-eta) to q-bar.

// Kernel ratio of one half-iteration (min over all rows of K. / max), folded
// into the item's running minimum.  Called by one block per item.
template <typename T>
__device__ void kratio_fold(const RowArgs<T>& A, int it, int k, int slot, double* sh) {
  const double* R = A.red + ((size_t)(k & 1) * A.nitems_all + it) * (size_t)A.hs * RED_SLOTS;
  double mn = INFINITY, mx = -INFINITY;
  for (int q = threadIdx.x; q < A.h; q += blockDim.x) {
    mn = fmin(mn, R[(size_t)q * RED_SLOTS + slot]);
    mx = fmax(mx, R[(size_t)q * RED_SLOTS + slot + 1]);
  }
  mn = block_min(mn, sh);
  mx = block_max(mx, sh);
  if (threadIdx.x == 0) {
    const double r = (mx > 0.0 && isfinite(mn)) ? mn / mx : -INFINITY;
    A.kr[it] = fmin(A.kr[it], r);
  }
}

// Orders the lanes of a wave through LDS: its LDS operations complete in order, so
// only the compiler has to keep them in place.
__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Row (m, l = m) of the packed (m, l) triangle.
__device__ __forceinline__ long long tri_off(long long m, long long L) { return m * L - m * (m - 1) / 2; }

// 4 x 4 exchange of lane groups: afterwards register t holds, in lane group g,
// what lane group t held in register g (lane groups = 16-lane rows).
__device__ __forceinline__ void lanegroup_transpose4(unsigned& r0, unsigned& r1, unsigned& r2, unsigned& r3) {
  auto a = __builtin_amdgcn_permlane32_swap(r0, r2, false, false);
  auto b = __builtin_amdgcn_permlane32_swap(r1, r3, false, false);
  auto c = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
  auto d = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
  r0 = c[0];
  r1 = c[1];
  r2 = d[0];
  r3 = d[1];
}

}  // namespace shot
