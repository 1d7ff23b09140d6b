// Row kernels of many row pairs: TP threads of one wave per mirror pair.
//
// A launch of a batch has thousands of row pairs, and what bounded the
// workgroup-per-group form (row_sink_kernel, row_kernel) there was instruction
// issue and barriers: every FFT stage ended in a workgroup barrier, a stage of
// a 720-point row kept 60 % of 256 threads busy, and the pointwise step of
// Alg. 1 cost an LDS round trip of its own.  Here a pair belongs to TP lanes
// of one wave, so its FFT stages need no barrier (LDS operations of a wave
// complete in order), and
//   * compile-time lengths: stages of radix 4 to 15 (composite radices of
//     coprime factors need no inner twiddles) in one LDS buffer per pair; the
//     inverse transform runs the forward transform's radices in reverse, so
//     its last stage leaves exactly the columns that the forward transform's
//     first stage takes in the same lane: the pointwise step runs on those
//     registers;
//   * run-time lengths and HEALPix rings: radix 2 to 8 stages whose index
//     division is one 24-bit multiply (a compiler-made 32-bit division costs
//     about 20 instructions per butterfly), two buffers per pair.
// The spectra of a group's pairs are gathered and stored by the whole
// workgroup, NP neighbouring pairs (16 NP bytes) of one order per run.
// Arithmetic, partial sums and their slots are those of row_kernel; a wave
// writes its sums at its first pair and the neutral element at the others.
// Measured per launch (before -> after): Sinkhorn half of 24 items at 360x720
// 38 -> 31 us (75 MB, 2.4 TB/s), reverse half of 16 items 46 -> 31 us, both
// rows of a heat apply of 16 items 50 -> 23 us; 24 HEALPix items at Nside 64
// 58 -> 26 us, 4 at Nside 256 162 -> 67 us; one float64 item of 256-point rows
// 12.8 -> 8.6 us.  What bounds it now: issue (about 3000 instructions per
// 720-point pair) in batches, the launch's own latency for single items.

#include <algorithm>

#include "device_common.h"
#include "launch.h"

namespace shot {

namespace {

// ------------------------------------------------------------ butterflies
// Composite radices of coprime factors (Good-Thomas): input n = (R2 n1 + R1 n2)
// mod R, output k with k = k1 mod R1, k = k2 mod R2, no inner twiddles.
template <typename T, int R>
__device__ __forceinline__ void bfly(cpx<T>* v, T s) {
  if constexpr (R == 6 || R == 10 || R == 12 || R == 15) {
    constexpr int R1 = R == 6 || R == 10 ? 2 : (R == 12 ? 4 : 3), R2 = R / R1;
    cpx<T> y[R2][R1];
#pragma unroll
    for (int n2 = 0; n2 < R2; ++n2) {
#pragma unroll
      for (int n1 = 0; n1 < R1; ++n1) y[n2][n1] = v[(R2 * n1 + R1 * n2) % R];
      butterfly<T, R1>(y[n2], s);
    }
#pragma unroll
    for (int k1 = 0; k1 < R1; ++k1) {
      cpx<T> z[R2];
#pragma unroll
      for (int n2 = 0; n2 < R2; ++n2) z[n2] = y[n2][k1];
      butterfly<T, R2>(z, s);
#pragma unroll
      for (int k2 = 0; k2 < R2; ++k2) y[k2][k1] = z[k2];
    }
#pragma unroll
    for (int k = 0; k < R; ++k) v[k] = y[k % R2][k % R1];
  } else {
    butterfly<T, R>(v, s);
  }
}

// Forward radices of a compile-time length for TP lanes: a stage's N / R
// butterflies fill the lanes (720 points: 60, 60 and 144 of 64-lane rounds).
template <int N, int TP>
struct RowFac;
template <>
struct RowFac<64, 16> { static constexpr int n = 3, r[4] = {4, 4, 4}; };
template <>
struct RowFac<128, 32> { static constexpr int n = 3, r[4] = {4, 4, 8}; };
template <>
struct RowFac<256, 64> { static constexpr int n = 4, r[4] = {4, 4, 4, 4}; };
template <>
struct RowFac<512, 64> { static constexpr int n = 3, r[4] = {8, 8, 8}; };
template <>
struct RowFac<1024, 64> { static constexpr int n = 4, r[4] = {8, 8, 4, 4}; };
template <>
struct RowFac<180, 16> { static constexpr int n = 2, r[4] = {12, 15}; };
template <>
struct RowFac<180, 64> { static constexpr int n = 3, r[4] = {4, 5, 9}; };
template <>
struct RowFac<360, 32> { static constexpr int n = 3, r[4] = {12, 6, 5}; };
template <>
struct RowFac<360, 64> { static constexpr int n = 3, r[4] = {6, 6, 10}; };
template <>
struct RowFac<720, 64> { static constexpr int n = 3, r[4] = {12, 12, 5}; };

// Stage S of the transform (inverse: radices in reverse order) of one pair in
// place, lane l of TP.  The first stage's output is stored with one entry of
// padding after every R (lanes then write R + 1 entries apart, on distinct
// banks; an odd R needs none), which the second stage's reads undo.
template <typename T, int N, int TP, bool INV, int S>
struct StageC {
  using F = RowFac<N, TP>;
  static constexpr int fac(int s) { return INV ? F::r[F::n - 1 - s] : F::r[s]; }
  static constexpr int pre(int s) { return s == 0 ? 1 : pre(s - 1) * fac(s - 1); }
  static constexpr int R = fac(S), Ns = pre(S), NR = N / R, IT = (NR + TP - 1) / TP;
  static constexpr bool first = S == 0, last = S == F::n - 1;
  static constexpr int PAD = fac(0) % 2 == 0 ? 1 : 0;  // odd runs are on distinct banks as they are
  __device__ static __forceinline__ void read(cpx<T> (&v)[IT][R], const cpx<T>* buf, int l) {
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int b = min(l + i * TP, NR - 1);
      const int at = S == 1 ? b + PAD * (b / Ns) : b;
      constexpr int step = S == 1 ? NR + PAD * (NR / Ns) : NR;
#pragma unroll
      for (int r = 0; r < R; ++r) v[i][r] = buf[at + r * step];
    }
  }
  __device__ static __forceinline__ void compute(cpx<T> (&v)[IT][R], const cpx<T>* tw, int l) {
    constexpr T sign = INV ? (T)1 : (T)-1;
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      if constexpr (!first) {
        const int b = min(l + i * TP, NR - 1), k = b % Ns;
#pragma unroll
        for (int r = 1; r < R; ++r) {
          cpx<T> w = tw[r * k * (N / (Ns * R))];
          w.y *= -sign;  // the table holds exp(-2 pi i k/N); the inverse uses the conjugate
          v[i][r] = cmul(v[i][r], w);
        }
      }
      bfly<T, R>(v[i], sign);
    }
  }
  __device__ static __forceinline__ void write(const cpx<T> (&v)[IT][R], cpx<T>* buf, int l) {
#pragma unroll
    for (int i = 0; i < IT; ++i) {
      const int b = l + i * TP;
      if (NR % TP != 0 && b >= NR) continue;
      const int base = first && !last ? b * (R + PAD) : (b / Ns) * Ns * R + b % Ns;
#pragma unroll
      for (int r = 0; r < R; ++r) buf[base + r * Ns] = v[i][r];
    }
  }
  // stages S .. last, from and to the buffer
  __device__ static __forceinline__ void run(cpx<T>* buf, const cpx<T>* tw, int l) {
    cpx<T> v[IT][R];
    read(v, buf, l);
    wave_lds_sync();
    compute(v, tw, l);
    write(v, buf, l);
    wave_lds_sync();
    if constexpr (!last) StageC<T, N, TP, INV, S + 1>::run(buf, tw, l);
  }
  // stages S .. last, the last one's output left in registers: entry [i][r] of
  // lane l is point l + i TP + r NR
  template <typename V>
  __device__ static __forceinline__ void run_to_reg(cpx<T>* buf, const cpx<T>* tw, int l, V& out) {
    if constexpr (last) {
      read(out, buf, l);
      wave_lds_sync();
      compute(out, tw, l);
    } else {
      cpx<T> v[IT][R];
      read(v, buf, l);
      wave_lds_sync();
      compute(v, tw, l);
      write(v, buf, l);
      wave_lds_sync();
      StageC<T, N, TP, INV, S + 1>::run_to_reg(buf, tw, l, out);
    }
  }
};

// ------------------------------------------------- run-time length transform
// q = b / Ns by the stage's magic number ceil(2^20 / Ns): exact for b, Ns <=
// 1024 (b < N / R and Ns <= N / R with N <= 2048 and R >= 2).
__device__ __forceinline__ int div_magic(int b, int mg) {
  return (int)(((unsigned)__umul24((unsigned)b, (unsigned)mg)) >> 20);
}

template <typename T, int R>
__device__ __forceinline__ void rt_stage(const cpx<T>* __restrict__ src, cpx<T>* __restrict__ dst, int N, int Ns,
                                         int mg, int rd_pad, int wr_pad, const cpx<T>* __restrict__ tw, T sign, int l,
                                         int tp) {
  const int NR = N / R, tws = NR / Ns;
  const int rstep = NR + rd_pad * tws;
  for (int b = l; b < NR; b += tp) {
    const int q = Ns == 1 ? b : div_magic(b, mg), k = Ns == 1 ? 0 : b - q * Ns;
    const cpx<T>* s = src + b + rd_pad * q;
    cpx<T> v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) v[r] = s[r * rstep];
    if (Ns > 1) {
#pragma unroll
      for (int r = 1; r < R; ++r) {
        cpx<T> w = tw[r * k * tws];
        w.y *= -sign;
        v[r] = cmul(v[r], w);
      }
    }
    butterfly<T, R>(v, sign);
    cpx<T>* d = dst + q * (Ns * R + wr_pad) + k;
#pragma unroll
    for (int r = 0; r < R; ++r) d[r * Ns] = v[r];
  }
}

// A radix of a prime R above 5.  With w = exp(-+2 pi i / R) the outputs q and
// R - q share x_r w^(rq) + x_(R-r) w^(-rq) = cos (x_r + x_(R-r)) + i sin (x_r -
// x_(R-r)): the (twiddled) sums and differences are formed in place first, and
// a lane then forms both outputs from (R - 1) / 2 of them, four multiply-adds
// and three LDS reads per term (a quarter of the work of summing every term of
// every output; rings of 4 p pixels were most of a launch that way).
template <typename T>
__device__ __forceinline__ void rt_stage_prime(cpx<T>* __restrict__ src, cpx<T>* __restrict__ dst, int N, int Ns,
                                               int mg, int R, int rd_pad, int wr_pad, const cpx<T>* __restrict__ tw,
                                               T sign, int l, int tp, bool block) {
  const int NR = N / R, tws = NR / Ns, H = (R - 1) / 2;
  const int rstep = NR + rd_pad * tws;
  for (int o = l; o < NR * H; o += tp) {
    const int r = o / NR + 1, b = o - (r - 1) * NR;
    const int q = Ns == 1 ? b : div_magic(b, mg), k = Ns == 1 ? 0 : b - q * Ns;
    cpx<T>* s = src + b + rd_pad * q;
    cpx<T> x = s[r * rstep], y = s[(R - r) * rstep];
    if (Ns > 1) {
      cpx<T> wx = tw[r * k * tws], wy = tw[(R - r) * k * tws];
      wx.y *= -sign;
      wy.y *= -sign;
      x = cmul(x, wx);
      y = cmul(y, wy);
    }
    s[r * rstep] = cadd(x, y);
    s[(R - r) * rstep] = csub(x, y);
  }
  if (block) __syncthreads();
  else wave_lds_sync();
  for (int o = l; o < NR * (H + 1); o += tp) {
    const int x = o / NR, b = o - x * NR;
    const int q = Ns == 1 ? b : div_magic(b, mg), k = Ns == 1 ? 0 : b - q * Ns;
    const cpx<T>* s = src + b + rd_pad * q;
    const cpx<T> x0 = s[0];
    const int e = x * NR;  // w^(r x) = tw[r e mod N]
    T cx = (T)0, cy = (T)0, dx = (T)0, dy = (T)0;
    int idx = e;
    // sums of 32 terms, then their sum: as one running sum, rings of 4p pixels were 1.5
    // (p = 251) to 1.9 times (p = 509) less exact than row_kernel's Bluestein transform.
    // Float64 stages of one such sum have a loop of their own (half of one field of
    // 176-point rows 13.3 -> 12.7 us, 182 points 16.0 -> 15.3); in float32 it gains nothing.
    if (sizeof(T) == 8 && H <= 32) {
#pragma unroll 4
      for (int r = 1; r <= H; ++r) {
        const cpx<T> w = tw[idx], u = s[r * rstep], d = s[(R - r) * rstep];
        cx += w.x * u.x;
        cy += w.x * u.y;
        dx += w.y * d.x;
        dy += w.y * d.y;
        idx += e;
        idx = idx >= N ? idx - N : idx;
      }
    } else {
#pragma unroll 1
      for (int r0 = 1; r0 <= H; r0 += 32) {
        T ax = (T)0, ay = (T)0, bx = (T)0, by = (T)0;
        const int r1 = min(r0 + 31, H);
#pragma unroll 4
        for (int r = r0; r <= r1; ++r) {
          const cpx<T> w = tw[idx], u = s[r * rstep], d = s[(R - r) * rstep];
          ax += w.x * u.x;
          ay += w.x * u.y;
          bx += w.y * d.x;
          by += w.y * d.y;
          idx += e;
          idx = idx >= N ? idx - N : idx;
        }
        cx += ax;
        cy += ay;
        dx += bx;
        dy += by;
      }
    }
    // the table's exponent is negative: sin enters with the transform's sign
    dx *= -sign;
    dy *= -sign;
    cx += x0.x;
    cy += x0.y;
    cpx<T>* t = dst + q * (Ns * R + wr_pad) + k;
    t[x * Ns] = {cx - dy, cy + dx};
    if (x) t[(R - x) * Ns] = {cx + dy, cy - dx};
  }
}

// Transform of one pair's row in buffers a and b; returns the one holding the
// result.  fac, mg: radices and their stages' magic numbers.
template <typename T>
__device__ __forceinline__ cpx<T>* rt_fft(cpx<T>* a, cpx<T>* b, int N, const int* fac, const int* mg, int nfac,
                                          const cpx<T>* tw, T sign, int l, int tp, bool block) {
  int Ns = 1;
  cpx<T>* src = a;
  cpx<T>* dst = b;
  int Rn = fac[0], mn = mg[0], r0 = Rn;
#pragma unroll 1
  for (int s = 0; s < nfac; ++s) {
    const int R = Rn, m = mn, nx = min(s + 1, RING_MAXFAC - 1);
    Rn = fac[nx];  // the next stage's, in flight meanwhile
    mn = mg[nx];
    // the first of several stages pads its output runs of four or eight
    const int wp = s == 0 && nfac > 1 && (R & 3) == 0 ? 1 : 0, rp = s == 1 && (r0 & 3) == 0 ? 1 : 0;
    switch (R) {
      case 2: rt_stage<T, 2>(src, dst, N, Ns, m, rp, wp, tw, sign, l, tp); break;
      case 3: rt_stage<T, 3>(src, dst, N, Ns, m, rp, wp, tw, sign, l, tp); break;
      case 4: rt_stage<T, 4>(src, dst, N, Ns, m, rp, wp, tw, sign, l, tp); break;
      case 5: rt_stage<T, 5>(src, dst, N, Ns, m, rp, wp, tw, sign, l, tp); break;
      case 8: rt_stage<T, 8>(src, dst, N, Ns, m, rp, wp, tw, sign, l, tp); break;
      default: rt_stage_prime<T>(src, dst, N, Ns, m, R, rp, wp, tw, sign, l, tp, block); break;
    }
    if (block) __syncthreads();
    else wave_lds_sync();
    cpx<T>* t = src;
    src = dst;
    dst = t;
    Ns *= R;
  }
  return src;
}

// ---------------------------------------------------------------- pointwise
// What one column of a pair needs besides the transformed rows: two values of
// its first and of its second input field, of the gradient field it adds to and
// of v-bar.
template <typename T>
struct Col {
  T a[2], b[2], g[2], w[2];
};

__device__ __forceinline__ bool positive_finite(float x) { return __builtin_amdgcn_classf(x, 0x100 | 0x80); }
__device__ __forceinline__ bool positive_finite(double x) { return __builtin_amdgcn_class(x, 0x100 | 0x80); }

// min and max in the field precision (exact: both are among the values);
// non-finite outputs count as -inf, as in track_minmax
template <typename T>
__device__ __forceinline__ void track_range(T& mn, T& mx, T v) {
  const T d = isfinite(v) ? v : (T)-INFINITY;
  mn = sizeof(T) == 4 ? (T)fminf((float)mn, (float)d) : (T)fmin((double)mn, (double)d);
  mx = sizeof(T) == 4 ? (T)fmaxf((float)mx, (float)d) : (T)fmax((double)mx, (double)d);
}

// Quotient of the Sinkhorn update.  FAST (float rows of 180, 360 and 720 points):
// hardware reciprocal and one Newton step, about 1 ulp, as row_sink_kernel runs them
// in smaller launches; an IEEE divide below the smallest normal float.  Every other
// length divides exactly, as row_kernel does: the reciprocal of a value above 2^126
// is not a normal float and would make the scaling 0.
template <typename T, bool FAST>
__device__ __forceinline__ T quotient(T f, T kv) {
  if constexpr (FAST && sizeof(T) == 4) {
    const T r0 = __builtin_amdgcn_rcpf(kv);
    const T r1 = fmaf(fmaf(-kv, r0, (T)1), r0, r0);
    T x = f * r1;
    if (!(kv >= FLT_MIN)) x = f / kv;
    return x;
  } else {
    return f / kv;
  }
}

enum RowKind : int { RK_FWD, RK_INV, RK_SINK, RK_ADJ, RK_ADJU_V1, RK_ADJU_B, RK_ADJU_A };
// RK_SINK with it keeps the gauge for the reverse sweep: a kernel of its own, as
// the store costs the 720-point one, which is at its register limit, 1 us of 35
constexpr int RK_KEEP = 16;

// Everything a pair's pointwise step reads, and the sums it keeps.
template <typename T>
struct PairState {
  long long r1, r2;  // element offsets of the pair's rows in the call's fields
  long long f0;      // item offset (fields that start at the item)
  T aj;
  bool eq, act;
  T gs;              // gauge (SINK), s (ADJ), g (ADJU)
  double g, s1, s2;  // gauge in double; ADJ_A: s-bar in s1; ADJU: S_A-bar, S_B-bar
  double acc, acc2;
  T kmin, kmax;
  bool bad;
  const T* uold;     // SINK: u-hat of the previous iteration, and where this half's scaling goes
  T* out;
};

template <typename T, int KIND, bool FAST>
__device__ __forceinline__ void point(const RowArgs<T>& A, const ItemDev& I, PairState<T>& S, const Col<T>& C,
                                      long long c, cpx<T> z, T (&nv)[2]) {
  const bool umode = A.mode == ROW_SINK_U;
  nv[0] = nv[1] = (T)0;
#pragma unroll
  for (int rr = 0; rr < 2; ++rr) {
    if (rr && S.eq) break;
    const long long fidx = (rr ? S.r2 : S.r1) + c;
    const T zr = rr ? z.y : z.x;
    if constexpr (KIND == RK_SINK) {
      const T f = C.a[rr];
      if (umode && A.chk_slot >= 0) {  // one launch in C (and then not worth a prefetch's registers)
        const double r = (double)S.uold[fidx] * (double)zr - (double)f;
        S.acc2 += r * r;
      }
      const T kv = umode ? S.gs * zr : zr;
      S.bad |= !positive_finite(kv);
      track_range(S.kmin, S.kmax, zr);
      T x = quotient<T, FAST>(f, kv);
      if (!I.balanced) {
        double gt;
        x = unbalanced_update(x, I.lam, I.eot, gt);
        S.acc += (double)S.aj * (double)f * gt;
      } else if (umode) {
        S.acc += (double)x;
      }
      nv[rr] = x;
      if (A.store_field && S.act) {
        __builtin_nontemporal_store(x, S.out + fidx);
      }
    } else if constexpr (KIND == RK_ADJ) {
      const T kt = S.aj * zr;  // K^T applied: a (.) (synthesised field)
      if (A.mode == ROW_ADJ_A) {
        const T u = C.b[rr], pv = C.a[rr];
        T ub = (T)S.s1 + kt;
        if (A.k == A.kT) ub += (T)I.eps * S.aj * pv / u;
        if (S.act) A.gA[fidx] = C.g[rr] + ub * u / pv;
        nv[rr] = -ub * u * u / pv;
      } else {
        const T v = C.b[rr], qv = C.a[rr];
        S.acc += (double)kt * (double)v;
        if (S.act) A.gB[fidx] = C.g[rr] + S.gs * kt * v / qv;
        nv[rr] = -S.gs * kt * v * v / qv;
      }
    } else {
      const T kt = S.aj * zr;
      const T ea = (T)I.eps, lam = (T)I.lam, eta = (T)I.eot, tau = (T)I.tau;
      const bool last = (A.k == A.kT);
      // Two powers a point: u^(-eps/tau-1) = u^(-eps/tau) / u, but u^(1/lam) takes the
      // exponent 1/lam of the rounded lam of the forward update x -> x^lam, which it
      // undoes.  u / u^(-eps/tau), with a separately rounded eps/tau, is off in the same
      // direction at every point (gradient of 2 items at Nside 64, tau = 10, error
      // against float64: 8.3e-6 -> 1.3e-5)
      if constexpr (KIND == RK_ADJU_V1) {
        const T v = C.b[rr];
        const T vb = kt;
        S.acc += (double)vb * (double)v;
        if (S.act) A.vbar[fidx] = vb;
        (void)ea; (void)lam; (void)eta; (void)tau; (void)last;
      } else if constexpr (KIND == RK_ADJU_B) {
        const T v = C.b[rr], qv = C.a[rr], sBb = (T)S.s2;
        const T pe = pow(v, -eta);
        const T vhb = S.gs * C.w[rr] - eta * sBb * S.aj * qv * (pe / v);
        if (S.act) A.gB[fidx] = C.g[rr] + (sBb * S.aj * pe + lam * vhb * v / qv);
        nv[rr] = -lam * vhb * v * pow(v, (T)1 / lam) / qv;
        (void)ea; (void)tau; (void)last;
      } else if constexpr (KIND == RK_ADJU_A) {
        const T u = C.b[rr], pv = C.a[rr], sAb = (T)S.s1;
        const T pe = pow(u, -eta);
        T uhb = kt - eta * sAb * S.aj * pv * (pe / u);
        if (last) uhb += ea * S.aj * pv * pow(u / S.gs, -eta - (T)1) / S.gs;
        if (S.act) A.gA[fidx] = C.g[rr] + (sAb * S.aj * pe + lam * uhb * u / pv);
        nv[rr] = -lam * uhb * u * pow(u, (T)1 / lam) / pv;
        (void)tau;
      }
    }
  }
}

// One column's inputs (in-bounds for every lane; unused values are dropped).
template <typename T, int KIND>
__device__ __forceinline__ Col<T> load_col(const RowArgs<T>& A, const ItemDev& I, const PairState<T>& S, long long c) {
  using GT = const __attribute__((address_space(1))) T;
  Col<T> C;
  C.a[0] = C.a[1] = C.b[0] = C.b[1] = C.g[0] = C.g[1] = C.w[0] = C.w[1] = (T)0;
  const long long i1 = S.r1 + c, i2 = S.r2 + c;
  if constexpr (KIND == RK_SINK) {
    GT* F = (GT*)static_cast<const T*>(A.mode == ROW_SINK_U ? I.p : I.q);
    C.a[0] = __builtin_nontemporal_load(F + i1);
    C.a[1] = __builtin_nontemporal_load(F + i2);
  } else if constexpr (KIND == RK_FWD) {
    GT* F = (GT*)A.in;
    C.a[0] = F[i1];
    C.a[1] = F[i2];
  } else if constexpr (KIND != RK_INV) {
    // the scaling of the half being reversed and its marginal
    const bool uside = KIND == RK_ADJ ? A.mode == ROW_ADJ_A : KIND == RK_ADJU_A;
    GT* W = (GT*)(uside ? ubuf_of(A, 0) : vbuf_of(A, 0));
    C.b[0] = W[i1];
    C.b[1] = W[i2];
    if constexpr (KIND != RK_ADJU_V1) {
      GT* F = (GT*)static_cast<const T*>(uside ? I.p : I.q);
      C.a[0] = F[i1];
      C.a[1] = F[i2];
      GT* D = (GT*)(uside ? A.gA : A.gB);
      C.g[0] = D[i1];
      C.g[1] = D[i2];
    }
    if constexpr (KIND == RK_ADJU_B) {
      GT* V = (GT*)A.vbar;
      C.w[0] = V[i1];
      C.w[1] = V[i2];
    }
  }
  return C;
}

// col[e] of the four prefetched columns by selects (a run-time index would put
// them in scratch memory)
template <typename T, int R>
__device__ __forceinline__ Col<T> pick_col(const Col<T> (&col)[R], int e) {
  Col<T> C = col[0];
#pragma unroll
  for (int r = 1; r < R; ++r)
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      C.a[q] = e == r ? col[r].a[q] : C.a[q];
      C.b[q] = e == r ? col[r].b[q] : C.b[q];
      C.g[q] = e == r ? col[r].g[q] : C.g[q];
      C.w[q] = e == r ? col[r].w[q] : C.w[q];
    }
  return C;
}

// Folded entry (E, O) of order m, row pair j of the item: one 16-byte (float)
// or two 16-byte (double) accesses.
template <typename T>
struct alignas(16) EO {
  cpx<T> e, o;
};

// Waves per SIMD a kernel's registers leave room for.  The adjoint kinds hold
// more fields per column; one wave fewer keeps all but one of them out of scratch
// memory.  Mean row launch of a gradient with four waves -> with three, us: 8
// balanced HEALPix pairs at Nside 64 23.9 -> 22.5, 16 pairs of 192-point rows 15.2 ->
// 14.4 (unbalanced 16.0 -> 15.6).  Four are better where three leave a small rest to a
// second round of workgroups: 16 pairs at Nside 64 38.1 -> 40.6.
constexpr int row_waves(int real_bytes, int nc, int kind) {
  if (real_bytes == 8) return 2;
  if (nc == 720) return kind >= RK_ADJU_B ? 4 : 5;
  if (nc == 0) return kind >= RK_ADJ ? 3 : 4;
  return nc == 1024 && kind == RK_ADJU_A ? 3 : 4;
}

// ------------------------------------------------------------------- kernel
// NC > 0: compile-time row length, NPC pairs per workgroup.  NC == 0: run-time
// length or HEALPix rings, blockDim / TP pairs per workgroup; TP > 64: one
// pair per workgroup, stages separated by workgroup barriers.
template <typename T, int NC, int TP, int NPC, int KX>
__global__ void __launch_bounds__(NC > 0 ? TP * NPC : (TP > 64 ? TP : 256), row_waves(sizeof(T), NC, KX % RK_KEEP))
row_wave_kernel(RowArgs<T> A) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  constexpr int KIND = KX % RK_KEEP;
  constexpr bool CT = NC > 0, KEEP = KX >= RK_KEEP;
  constexpr bool INV = KIND != RK_FWD && KIND != RK_ADJU_B;           // has the inverse transform
  constexpr bool FWD = KIND != RK_INV && KIND != RK_ADJU_V1;          // has the forward transform
  const int bs = CT ? TP * NPC : (int)blockDim.x;
  const int NP = CT ? NPC : bs / TP;
  const int L = A.L, h = A.h, nlat = A.nlat;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nw = (bs + 63) >> 6;
  const int ngroups = (h + NP - 1) / NP;
  // neighbouring groups on one XCD; HEALPix: the host's dealt order of ring octets
  const int jp0 = A.rpair ? A.rpair[(blockIdx.x & 7) + 8 * ((blockIdx.x >> 3) * NP)]
                          : xcd_row_pair(blockIdx.x, ngroups) * NP;
  const int np = min(NP, h - jp0);
  const int it = A.item0 + blockIdx.y;
  const ItemDev I = A.items[it];
  __shared__ double shw[8][4];
  __shared__ double shr[8][4];
  __shared__ T awl[16];
  __shared__ int rlen[16], zof[16];

  // this lane's pair (a lane of a pair beyond np works on the last one and writes nothing)
  const int pr = CT || TP <= 64 ? tid / TP : 0, l = CT || TP <= 64 ? tid % TP : tid;
  const int jp = min(jp0 + pr, h - 1), j2 = nlat - 1 - jp;
  const RingDev* RG = !CT && A.ring ? A.ring + jp : nullptr;
  const RingDev* FR = RG ? RG : A.rowfft;  // radices of a run-time length
  const int N = CT ? NC : (RG ? RG->len : A.nlon);
  PairState<T> S;
  S.act = pr < np;
  S.eq = jp == j2;
  S.r1 = I.foff + (RG ? (long long)RG->off1 : (long long)jp * N);
  S.r2 = I.foff + (RG ? (long long)RG->off2 : (long long)j2 * N);
  S.f0 = I.foff;
  S.aj = A.aw[jp];
  S.acc = S.acc2 = 0.0;
  S.kmin = (T)INFINITY;
  S.kmax = (T)-INFINITY;
  S.bad = false;
  S.gs = (T)1;
  S.g = 1.0;
  S.s1 = S.s2 = 0.0;
  {
    T* const u0 = A.ubuf0;
    T* const u1 = A.ubuf1;
    T* const v0 = A.vbuf0;
    T* const v1 = A.vbuf1;
    S.uold = (A.k & 1) ? u0 : u1;
    S.out = A.mode == ROW_SINK_U ? ((A.k & 1) ? u1 : u0) : ((A.k & 1) ? v1 : v0);
  }

  // LDS: per pair one (CT) or two buffers of A.wstride entries, then twiddles
  const int WS = A.wstride;
  cpx<T>* all = reinterpret_cast<cpx<T>*>(smem_raw);
  cpx<T>* buf = all + (size_t)pr * WS * (CT ? 1 : 2);
  cpx<T>* buf1 = CT ? buf : buf + WS;
  cpx<T>* twl = all + (size_t)NP * WS * (CT ? 1 : 2) + (!CT && A.ring ? (size_t)pr * A.nlon : 0);
  cpx<T>* spec = A.spec + I.soff;

  // ---- loads, all issued before the first wait
  // (1) the pair's columns
  constexpr int IT0 = CT ? StageC<T, CT ? NC : 180, CT ? TP : 16, false, 0>::IT : 1;
  constexpr int R0 = CT ? StageC<T, CT ? NC : 180, CT ? TP : 16, false, 0>::R : 4;
  constexpr int NR0 = CT ? NC / R0 : 1;
  Col<T> col[IT0][R0];
  const bool pre = CT || N <= R0 * TP;  // run-time rows: up to four columns per lane are prefetched
  // (the adjoint kinds read four to six fields per column: registers for them
  // would cost a resident wave, 34 -> 33 us for 16 items of 360x720)
  constexpr bool PREF = KIND != RK_INV && (!CT || KIND == RK_SINK || KIND == RK_FWD);
  if constexpr (PREF) {
    if (pre) {
#pragma unroll
      for (int i = 0; i < IT0; ++i)
#pragma unroll
        for (int r = 0; r < R0; ++r) {
          const int c = CT ? min(l + i * TP, NR0 - 1) + r * NR0 : min(l + r * TP, N - 1);
          col[i][r] = load_col<T, KIND>(A, I, S, c);
        }
    }
  }
  // (2) partial sums: gauge and previous kernel range (SINK), s-bar or g-bar (adjoint)
  double s0 = 0.0, s1 = 0.0, mn = INFINITY, mx = -INFINITY;
  const bool umode = A.mode == ROW_SINK_U;
  const bool gsum = KIND == RK_SINK && umode && !A.gk && A.k > 1;
  const bool kfold = KIND == RK_SINK && A.kr && blockIdx.x == 0 && (!umode || A.k > 1);
  const bool asum = (KIND == RK_ADJ && A.mode == ROW_ADJ_A) || KIND == RK_ADJU_B || KIND == RK_ADJU_A;
  if constexpr (KIND == RK_SINK) {
    const double* Rg = A.red + ((size_t)((A.k - 1) & 1) * A.nitems_all + it) * (size_t)A.hs * RED_SLOTS;
    const double* Rk = A.red + ((size_t)((umode ? A.k - 1 : A.k) & 1) * A.nitems_all + it) * (size_t)A.hs * RED_SLOTS;
    const int ks = umode ? 4 : 2;
    for (int q0 = tid; q0 < h; q0 += 2 * bs) {  // two row pairs' loads in flight
      const int qa = q0, qb = min(q0 + bs, h - 1);
      const bool two = q0 + bs < h;
      if (gsum) {
        const double a0 = Rg[(size_t)qa * RED_SLOTS], a1 = Rg[(size_t)qa * RED_SLOTS + 1];
        const double b0 = Rg[(size_t)qb * RED_SLOTS], b1 = Rg[(size_t)qb * RED_SLOTS + 1];
        s0 += a0 + (two ? b0 : 0.0);
        s1 += a1 + (two ? b1 : 0.0);
      }
      if (kfold) {
        mn = fmin(mn, fmin(Rk[(size_t)qa * RED_SLOTS + ks], Rk[(size_t)qb * RED_SLOTS + ks]));
        mx = fmax(mx, fmax(Rk[(size_t)qa * RED_SLOTS + ks + 1], Rk[(size_t)qb * RED_SLOTS + ks + 1]));
      }
    }
  }
  if (asum)
    for (int q = tid; q < h; q += bs) s0 += A.adjp[(size_t)it * A.hs + q];
  // (3) twiddles and the group's spectra
  if (CT || !A.ring) {
    for (int i = tid; i < N; i += bs) twl[i] = A.tw[i];
  } else {
    const cpx<T>* src = A.ring_tw + RG->twoff;
    for (int i = l; i < N; i += TP) twl[i] = src[i];
  }
  if (tid < NP) {
    awl[tid] = tid < np ? A.aw[jp0 + tid] : (T)0;
    rlen[tid] = A.ring ? A.ring[min(jp0 + tid, h - 1)].len : A.nlon;
  }
  const int lnp = 31 - __clz(NP);  // NP is a power of two
  if constexpr (INV) {
    if (CT || !A.ring) {
      // Hermitian spectrum of each pair: Z[m] = G_j[m] + i G_j'[m], Z[N-m] its mirror
      const int nz = N - 2 * L + 1;
      if (nz > 0)
        for (int c = L + l; c < L + nz; c += TP) buf[c] = {(T)0, (T)0};
      auto put = [&](int m, int p, cpx<T> e, cpx<T> o) {
        const bool eq = jp0 + p == nlat - 1 - jp0 - p;
        const cpx<T> a = cadd(e, o);
        const cpx<T> b = eq ? cpx<T>{(T)0, (T)0} : csub(e, o);
        cpx<T>* d = all + (size_t)p * WS * (CT ? 1 : 2);
        d[m] = {a.x - b.y, a.y + b.x};
        if (m > 0) d[N - m] = {a.x + b.y, -a.y + b.x};
      };
      if (!A.cut) {
        constexpr int GU = CT ? (NPC * ((NC + 1) / 2) + TP * NPC - 1) / (TP * NPC) : 4;
        for (int i0 = 0; i0 < NP * L; i0 += GU * bs) {
          EO<T> g[GU];
#pragma unroll
          for (int u = 0; u < GU; ++u) {
            const int idx = min(i0 + u * bs + tid, NP * L - 1);
            const int m = idx >> lnp, p = min(idx & (NP - 1), np - 1);
            g[u] = reinterpret_cast<const EO<T>*>(spec)[(size_t)m * h + jp0 + p];
          }
#pragma unroll
          for (int u = 0; u < GU; ++u) {
            const int idx = i0 + u * bs + tid;
            if (idx < NP * L) put(idx >> lnp, idx & (NP - 1), g[u].e, g[u].o);
          }
        }
      } else {
        for (int idx = tid; idx < NP * L; idx += bs) {
          const int m = idx >> lnp, p = idx & (NP - 1);
          cpx<T> e, o;
          load_spec_pair(A, spec, it, m, jp0 + min(p, np - 1), e, o);
          put(m, p, e, o);
        }
      }
    } else {
      // HEALPix: with P_m = G_m e^{i m phi0}, order m lands in bin m mod N and -m
      // in bin -m mod N of the packed spectrum (orders beyond the ring's length
      // alias, as its samples do).  Both bins' terms of every order are formed
      // once, into the second buffer; the pair's lanes then add up each bin.
      for (int i0 = 0; i0 < NP * L; i0 += 2 * bs) {
        EO<T> g[2];
        cpx<T> ph[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int idx = min(i0 + u * bs + tid, NP * L - 1);
          const int m = idx >> lnp, j = jp0 + min(idx & (NP - 1), np - 1);
          ph[u] = A.ring_ph[(size_t)j * L + m];
          if (!A.cut) g[u] = reinterpret_cast<const EO<T>*>(spec)[(size_t)m * h + j];
          else load_spec_pair(A, spec, it, m, j, g[u].e, g[u].o);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int idx = i0 + u * bs + tid;
          if (idx >= NP * L) continue;
          const int m = idx >> lnp, p = idx & (NP - 1), j = min(jp0 + p, h - 1);
          const bool eq = j == nlat - 1 - j;
          const cpx<T> a = cmul(cadd(g[u].e, g[u].o), ph[u]);
          const cpx<T> b = eq ? cpx<T>{(T)0, (T)0} : cmul(csub(g[u].e, g[u].o), ph[u]);
          cpx<T>* d = all + (size_t)p * WS * 2 + WS;
          d[m] = {a.x - b.y, a.y + b.x};
          d[L + m] = {a.x + b.y, -a.y + b.x};
        }
      }
    }
  }
  // ---- sums over the item's row pairs, wave partials combined after the barrier
  if (gsum || asum) {
    s0 = wave_sum(s0);
    if (gsum) s1 = wave_sum(s1);
  }
  if (kfold) {
    mn = wave_min(mn);
    mx = wave_max(mx);
  }
  if (lane == 0) {
    shw[wave][0] = s0;
    shw[wave][1] = s1;
    shw[wave][2] = mn;
    shw[wave][3] = mx;
  }
  __syncthreads();
  if constexpr (KIND == RK_SINK) {
    if (umode) {
      if (A.gk) {
        S.g = A.gk[it];
      } else if (A.k > 1) {
        double a = 0.0, b = 0.0;
        for (int w = 0; w < nw; ++w) {
          a += shw[w][0];
          b += shw[w][1];
        }
        S.g = I.balanced ? a : exp(-(0.5 * I.tau * (log(a) - log(b))) / I.eps);
        if (KEEP && blockIdx.x == 0 && tid == 0) store_gauge(A, it, S.g, a, b);
      }
      S.gs = (T)S.g;
    }
    if (kfold && tid == 0) {
      double pmn = INFINITY, pmx = -INFINITY;
      for (int w = 0; w < nw; ++w) {
        pmn = fmin(pmn, shw[w][2]);
        pmx = fmax(pmx, shw[w][3]);
      }
      const double r = (pmx > 0.0 && isfinite(pmn)) ? pmn / pmx : -INFINITY;
      A.kr[it] = fmin(A.kr[it], r);
    }
  }
  if constexpr (KIND == RK_ADJ || KIND == RK_ADJU_B || KIND == RK_ADJU_A) {
    double sb = 0.0;
    if (asum)
      for (int w = 0; w < nw; ++w) sb += shw[w][0];
    if constexpr (KIND == RK_ADJ) {
      S.gs = (T)A.gk[it];
      S.s1 = sb;
    } else {
      const double G = A.gk[3 * it], SA = A.gk[3 * it + 1], SB = A.gk[3 * it + 2];
      S.gs = (T)G;
      S.s1 = -sb * G / (2.0 * I.eot * SA);
      S.s2 = sb * G / (2.0 * I.eot * SB);
    }
  }

  // ---- inverse transform, pointwise step, forward transform
  cpx<T>* Z = buf;
  if constexpr (CT) {
    cpx<T> v[IT0][R0];
    if constexpr (INV) {
      StageC<T, CT ? NC : 180, CT ? TP : 16, true, 0>::run_to_reg(buf, twl, l, v);
    }
#pragma unroll
    for (int i = 0; i < IT0; ++i) {
      const int b = l + i * TP;
      if (NR0 % TP != 0 && b >= NR0) continue;
#pragma unroll
      for (int r = 0; r < R0; ++r) {
        const int c = b + r * NR0;
        if constexpr (KIND == RK_FWD) {
          v[i][r] = {col[i][r].a[0], S.eq ? (T)0 : col[i][r].a[1]};
        } else if constexpr (KIND == RK_INV) {
          const T s = A.wts_out ? S.aj : (T)1;
          if (S.act) {
            A.out[S.r1 + c] = v[i][r].x * s;
            if (!S.eq) A.out[S.r2 + c] = v[i][r].y * s;
          }
        } else {
          T nv[2];
          point<T, KIND, NC % 180 == 0>(A, I, S, PREF ? col[i][r] : load_col<T, KIND>(A, I, S, c), c, INV ? v[i][r] : cpx<T>{(T)0, (T)0}, nv);
          v[i][r] = {nv[0], nv[1]};
        }
      }
    }
    if constexpr (FWD) {
      using S0 = StageC<T, CT ? NC : 180, CT ? TP : 16, false, 0>;
      wave_lds_sync();
      S0::compute(v, twl, l);
      S0::write(v, buf, l);
      wave_lds_sync();
      StageC<T, CT ? NC : 180, CT ? TP : 16, false, 1>::run(buf, twl, l);
    }
  } else {
    const bool block = TP > 64;
    const int* fac = FR->fac;
    const int* mg = FR->mg;
    const int nfac = FR->nfac;
    if (INV && RG) {
      // bins: G lanes share a short ring's bin, partials added in lane order
      const cpx<T>* zp = buf1;
      const cpx<T>* zn = buf1 + L;
      const int G = N >= TP ? 1 : TP / N;
      for (int c = l; c < N * G; c += TP) {
        const int g = G == 1 ? 0 : c / N, cb = c - g * N;
        cpx<T> z = {(T)0, (T)0};
        for (int m = cb + g * N; m < L; m += G * N) z = cadd(z, zp[m]);
        for (int m = (cb == 0 ? N : N - cb) + g * N; m < L; m += G * N) z = cadd(z, zn[m]);
        buf[c] = z;
      }
      if (block) __syncthreads();
      else wave_lds_sync();
      if (G > 1) {
        cpx<T> z = {(T)0, (T)0};
        if (l < N)
          for (int g = 0; g < G; ++g) z = cadd(z, buf[g * N + l]);
        if (block) __syncthreads();
        else wave_lds_sync();
        if (l < N) buf[l] = z;
        if (block) __syncthreads();
        else wave_lds_sync();
      }
    }
    // one inlined transform for both directions
#pragma unroll 1
    for (int pass = INV ? 0 : 1; pass < (FWD ? 2 : 1); ++pass) {
      if (pass == 1) {
#pragma unroll 1
        for (int c = l, e = 0; c < N; c += TP, ++e) {
          const Col<T> C = pre ? pick_col(col[0], e) : load_col<T, KIND>(A, I, S, c);
          if constexpr (KIND == RK_FWD) {
            Z[c] = {C.a[0], S.eq ? (T)0 : C.a[1]};
          } else {
            T nv[2];
            point<T, KIND, false>(A, I, S, C, c, INV ? Z[c] : cpx<T>{(T)0, (T)0}, nv);
            Z[c] = {nv[0], nv[1]};
          }
        }
        if (block) __syncthreads();
        else wave_lds_sync();
      }
      Z = rt_fft<T>(Z, Z == buf ? buf1 : buf, N, fac, mg, nfac, twl, pass ? (T)-1 : (T)1, l, TP, block);
    }
    if constexpr (KIND == RK_INV) {
      const T s = A.wts_out ? S.aj : (T)1;
      if (S.act)
        for (int c = l; c < N; c += TP) {
          const cpx<T> z = Z[c];
          A.out[S.r1 + c] = z.x * s;
          if (!S.eq) A.out[S.r2 + c] = z.y * s;
        }
    } else if constexpr (KIND == RK_ADJU_V1) {
#pragma unroll 1
      for (int c = l, e = 0; c < N; c += TP, ++e) {
        T nv[2];
        point<T, KIND, false>(A, I, S, pre ? pick_col(col[0], e) : load_col<T, KIND>(A, I, S, c), c, Z[c], nv);
      }
    }
    if (l == 0) zof[pr] = (int)(Z - all);
  }
  if constexpr (KIND == RK_INV) return;

  // ---- this launch's partial sums: each wave at its first pair, neutral
  // elements at its others; a pair of several waves through LDS
  if constexpr (KIND == RK_SINK || KIND == RK_ADJ || KIND == RK_ADJU_V1) {
    if (!S.act) {
      S.acc = S.acc2 = 0.0;
      S.kmin = (T)INFINITY;
      S.kmax = (T)-INFINITY;
      S.bad = false;
    }
    double r4[4] = {S.acc, S.acc2, (double)S.kmin, (double)S.kmax};
    const bool anybad = KIND == RK_SINK && __any(S.bad);
    r4[0] = wave_sum(r4[0]);
    if constexpr (KIND == RK_SINK) {
      if (umode && A.chk_slot >= 0) r4[1] = wave_sum(r4[1]);
      r4[2] = wave_min(r4[2]);
      r4[3] = wave_max(r4[3]);
    }
    constexpr int PW = CT || TP <= 64 ? 64 / (TP < 64 ? TP : 64) : 1;  // pairs per wave
    int slot = wave * PW, nslot = min(PW, np - slot);                  // this wave's pairs
    if (!CT && TP > 64) {
      if (lane == 0)
        for (int i = 0; i < 4; ++i) shr[wave][i] = r4[i];
      __syncthreads();
      slot = 0;
      nslot = wave == 0 ? 1 : 0;
      r4[0] = r4[1] = 0.0;
      r4[2] = INFINITY;
      r4[3] = -INFINITY;
      for (int w = 0; w < nw; ++w) {
        r4[0] += shr[w][0];
        r4[1] += shr[w][1];
        r4[2] = fmin(r4[2], shr[w][2]);
        r4[3] = fmax(r4[3], shr[w][3]);
      }
    }
    if (lane < nslot) {
      const bool fst = lane == 0;
      const int j = jp0 + slot + lane;
      if constexpr (KIND == RK_SINK) {
        double* rp = A.red + (((size_t)(A.k & 1) * A.nitems_all + it) * A.hs + j) * RED_SLOTS;
        rp[umode ? 0 : 1] = fst ? r4[0] : 0.0;
        rp[umode ? 2 : 4] = fst ? r4[2] : INFINITY;
        rp[umode ? 3 : 5] = fst ? r4[3] : -INFINITY;
        if (umode && A.chk_slot >= 0)
          A.rhist[((size_t)it * A.nslot + A.chk_slot) * A.hs + j] = fst ? r4[1] : 0.0;
      } else if (KIND == RK_ADJU_V1 || A.mode == ROW_ADJ_VB) {
        A.adjp[(size_t)it * A.hs + j] = fst ? r4[0] : 0.0;
      }
    }
    // (read first: once an item has broken down every wave of every later half is bad, and
    // their atomics on its one word took 8 us a half of 361 float64 pairs)
    if (anybad && lane == 0 && A.brk[it] > A.k) atomicMin(&A.brk[it], A.k);
  }
  if constexpr (!FWD) return;

  // ---- fold, weight, store: orders' entries of the group's pairs together
  __syncthreads();
  const bool unweighted = (KIND == RK_FWD && !A.wts_in) || (KIND != RK_FWD && KIND != RK_SINK);
  for (int idx = tid; idx < NP * L; idx += bs) {
    const int m = idx >> lnp, p = idx & (NP - 1);
    if (p >= np) continue;
    const int j = jp0 + p;
    const bool eq = j == nlat - 1 - j;
    const int n = CT ? NC : rlen[p];
    const cpx<T>* Zp = CT ? all + (size_t)p * WS : all + zof[p];
    const int cm = !CT && A.ring ? (m < n ? m : m % n) : m;  // rings: order m sits in bin m mod n
    const cpx<T> a = Zp[cm];
    cpx<T> b = Zp[cm == 0 ? 0 : n - cm];
    b.y = -b.y;
    EO<T> g;
    if (eq) {
      g.e = a;
      g.o = {(T)0, (T)0};
    } else {
      const cpx<T> x1 = {(T)0.5 * (a.x + b.x), (T)0.5 * (a.y + b.y)};
      const cpx<T> x2 = {(T)0.5 * (a.y - b.y), (T)-0.5 * (a.x - b.x)};
      g.e = cadd(x1, x2);
      g.o = csub(x1, x2);
    }
    if (!CT && A.ring) {  // e^{-i m phi0}
      cpx<T> e = A.ring_ph[(size_t)j * L + m];
      e.y = -e.y;
      g.e = cmul(g.e, e);
      g.o = cmul(g.o, e);
    }
    const T cw = unweighted ? (T)1 : awl[p];
    g.e = cscale(g.e, cw);
    g.o = cscale(g.o, cw);
    reinterpret_cast<EO<T>*>(spec)[(size_t)m * h + j] = g;
  }
}

}  // namespace

// LDS entries of one buffer of a pair.  Compile-time rows: the first stage's
// padding, then rounded so that the NP pairs' buffers start on banks that the
// gather's and the stages' accesses share evenly.
static int wave_stride_ct(int n, int first_radix_pad, int mod) {
  int w = n + first_radix_pad;
  while (w % 32 != mod) ++w;
  return w;
}
static int wave_stride_rt(int nbuf, int pad, int need) {
  int w = std::max({nbuf + pad, need, 64});
  while (w % 16 != 4) ++w;
  return w;
}

template <typename T, int NC, int TP, int NPC, int KIND>
static hipError_t launch_ct(RowArgs<T> a, int nb, int mod, hipStream_t stream) {
  using F = RowFac<NC, TP>;
  // both directions' first stages: radix r[0] forward, r[n - 1] inverse
  const int pf = F::r[0] % 2 == 0 ? NC / F::r[0] : 0, pi = F::r[F::n - 1] % 2 == 0 ? NC / F::r[F::n - 1] : 0;
  a.wstride = wave_stride_ct(NC, std::max(pf, pi), mod);
  const size_t lds = ((size_t)NPC * a.wstride + NC) * sizeof(cpx<T>);
  static std::atomic<unsigned long long> lds_set{0};
  hipError_t e = allow_lds(reinterpret_cast<const void*>(&row_wave_kernel<T, NC, TP, NPC, KIND>), lds, lds_set);
  if (e != hipSuccess) return e;
  dim3 grid((a.h + NPC - 1) / NPC, nb);
  SHOT_LAUNCH((row_wave_kernel<T, NC, TP, NPC, KIND>), grid, dim3(TP * NPC), lds, stream, a);
  return hipGetLastError();
}

template <typename T, int TP, int KIND>
static hipError_t launch_rt(RowArgs<T> a, int nb, int np, hipStream_t stream) {
  a.wstride = wave_stride_rt(a.nlon, a.row_pad, std::max(a.ring ? 2 * a.L : 0, TP));
  const size_t lds = ((size_t)np * 2 * a.wstride + (size_t)(a.ring ? np : 1) * a.nlon) * sizeof(cpx<T>);
  static std::atomic<unsigned long long> lds_set{0};
  hipError_t e = allow_lds(reinterpret_cast<const void*>(&row_wave_kernel<T, 0, TP, 1, KIND>), lds, lds_set);
  if (e != hipSuccess) return e;
  dim3 grid((a.h + np - 1) / np, nb);
  SHOT_LAUNCH((row_wave_kernel<T, 0, TP, 1, KIND>), grid, dim3(TP * np), lds, stream, a);
  return hipGetLastError();
}

template <typename T, int KIND>
static hipError_t launch_kind(const RowArgs<T>& a, int nb, const RowWaveShape& w, hipStream_t stream) {
  if (w.ct) {
    switch (a.nlon) {
      case 64: return launch_ct<T, 64, 16, 4, KIND>(a, nb, 8, stream);
      case 128: return launch_ct<T, 128, 32, 4, KIND>(a, nb, 8, stream);
      case 256: return launch_ct<T, 256, 64, 4, KIND>(a, nb, 8, stream);
      case 512: return launch_ct<T, 512, 64, 4, KIND>(a, nb, 8, stream);
      case 1024: return launch_ct<T, 1024, 64, 4, KIND>(a, nb, 8, stream);
      default: break;
    }
    if constexpr (sizeof(T) == 4) {
      if (a.nlon == 180)
        return w.tp == 16 ? launch_ct<T, 180, 16, 16, KIND>(a, nb, 18, stream)
                          : launch_ct<T, 180, 64, 4, KIND>(a, nb, 8, stream);
      if (a.nlon == 360)
        return w.tp == 32 ? launch_ct<T, 360, 32, 8, KIND>(a, nb, 4, stream)
                          : launch_ct<T, 360, 64, 4, KIND>(a, nb, 8, stream);
      if (a.nlon == 720) return launch_ct<T, 720, 64, 4, KIND>(a, nb, 8, stream);
    }
    return hipErrorInvalidValue;
  }
  return w.tp == 64 ? launch_rt<T, 64, KIND>(a, nb, w.np, stream) : launch_rt<T, 256, KIND>(a, nb, 1, stream);
}

// Kind of a row mode, or -1 where row_kernel runs it.
static int kind_of(int mode, bool last_v1, bool has_in) {
  switch (mode) {
    case ROW_FWD: return has_in ? RK_FWD : -1;
    case ROW_INV: return RK_INV;
    case ROW_SINK_U: case ROW_SINK_V: return RK_SINK;
    case ROW_ADJ_A: case ROW_ADJ_VB: return RK_ADJ;
    case ROW_ADJU_V1: return last_v1 ? -1 : RK_ADJU_V1;
    case ROW_ADJU_B: return RK_ADJU_B;
    case ROW_ADJU_A: return RK_ADJU_A;
    default: return -1;
  }
}

template <typename T>
RowWaveShape row_wave_shape(const RowArgs<T>& a, int nb) {
  RowWaveShape w{0, 0, 0};
  const int kind = kind_of(a.mode, a.k >= a.kT, a.in != nullptr);
  if (kind < 0) return w;
  const long long pairs = (long long)a.h * nb;
  // Powers: the unbalanced reverse steps, and in float64 the unbalanced halves (about 150
  // instructions each).  Float64 rows of compile-time lengths whose launch does not fill
  // the device take the run-time form with more lanes a pair (one item, a Sinkhorn half:
  // 512 points 16.0 us with 256 lanes against 23.4 with 64, 256 points 13.0 against 14.0;
  // 64 points 10.4 with 64 lanes against 12.7 with 16), of 1024 points always (1536 pairs:
  // 112 us in the compile-time form, whose LDS leaves one workgroup a compute unit,
  // against 85).  Above the lines: 512 points, 1024 pairs 30.5 us against 32.1; 256
  // points, 512 pairs 15.4 against 16.2.
  const bool powers = kind == RK_ADJU_B || kind == RK_ADJU_A || (sizeof(T) == 8 && a.unbal && kind == RK_SINK);
  const bool shared = sizeof(T) == 8 && powers &&
                      (a.nlon == 1024 || pairs < (a.nlon == 128 || a.nlon == 256 ? 400 : 900));
  const bool pow2 = a.nlon == 64 || a.nlon == 128 || a.nlon == 256 || a.nlon == 512 || (a.nlon == 1024 && pairs >= 1024);
  const bool deg = sizeof(T) == 4 && (a.nlon == 180 || a.nlon == 360 || a.nlon == 720);
  if (!a.ring && !shared && (pow2 || deg)) {
    // 64 to 1024 points: always (one item of 256 points: 12.8 -> 8.6 us in
    // float64; of 1024 points only with many pairs, the run-time form's 256
    // lanes are faster for one item: 15.1 against 16.9 us).  180, 360 and 720
    // points: from 1024 pairs on; below, row_sink_kernel's wide workgroups
    // measured the same or faster.  Half- and quarter-wave pairs, which fill
    // the lanes better, once the launch has waves enough to spare.
    if (deg && pairs < 1024) return w;
    w.ct = 1;
    w.tp = 64;
    if (a.nlon == 180 && pairs >= 16384) w.tp = 16;
    if (a.nlon == 360 && pairs >= 8192) w.tp = 32;
    return w;
  }
  if (!a.ring && sizeof(T) == 4 && a.nlon == 1440) return w;  // row_sink_kernel, 512 lanes
  // A belt of rings of 4 k p pixels, p a prime beyond 480 (one item: beyond 400): their
  // radix-p stage takes (p - 1)^2 products a row pair, row_kernel's Bluestein transform
  // two FFTs of 4096 points (a half at Nside 509: one item 229 us against 172, 4 items
  // 655 against 610; Nside 449: one item 191 against 169, 4 items 437 against 529;
  // Nside 401: one item 166.5 against 166.7).  Float64 rings that long have direct
  // stages in either kernel.
  if (a.ring && sizeof(T) == 4 && a.max_prime > (nb == 1 ? 400 : 480)) return w;
  // Run-time lengths: one wave per pair for rows of up to 200 points (192 points, one
  // item, a half: 9.7 us; float64 10.6 against 11.2 with 256 lanes), of up to 256 points
  // from 500 pairs on (240 points: one item 11.1 us against 10.2, 960 pairs reverse 14.7
  // against 18.0), with powers beyond 128 points from 640 pairs on (240 points, float64
  // half: one item 17.8 us against 13.2, 960 pairs 22.5 against 22.4); 256 lanes for
  // longer rows (400 points: 15.1 against 11.9) and for large primes.  Rings of more than
  // 128 pixels from 1200 pairs on (Nside 64, a half: 8 items 18.6 us against 16.6 with
  // 256 lanes, 12 items 20.6 against 23.2).
  // A prime radix of 7 to 13 beyond 128 points leaves most of 64 lanes idle in its stages:
  // one wave per pair from 800 pairs on, float64 from 640 (half of 8 fields of 252 points
  // 15.6 us against 13.4, float64 16.7 against 15.0; 16 of 182 points 16.3 against 14.9; 16 of
  // 224, 896 pairs, 14.9 against 15.4; float64 16 of 176, 704 pairs, 14.2 against 15.0).
  // Below, float32 Sinkhorn and balanced reverse halves run on row_kernel (one field of 154
  // points: 64 lanes 14.9, 256 lanes 12.3, row_kernel 11.4; 8 of 252 15.6, 13.4, 12.2).
  const bool prime = !a.ring && a.max_prime > 5 && a.max_prime <= 13 && a.nlon > 128 && a.nlon <= 256;
  const int line = prime ? (sizeof(T) == 4 && !powers ? 800 : 640)
                         : powers && a.nlon > 128 ? 640 : a.nlon > 200 ? 500 : 0;
  if (prime && pairs < line && sizeof(T) == 4 && (kind == RK_SINK || kind == RK_ADJ)) return w;
  const bool narrow = a.ring ? (a.nlon <= 128 || (a.nlon <= 256 && pairs >= 1200))
                             : a.max_prime <= 13 && a.nlon <= 256 && pairs >= line;
  w.tp = narrow ? 64 : 256;
  w.np = 1;
  const int ws = wave_stride_rt(a.nlon, a.row_pad, std::max(a.ring ? 2 * a.L : 0, w.tp));
  auto lds = [&](int np) { return ((size_t)np * 2 * ws + (size_t)(a.ring ? np : 1) * a.nlon) * sizeof(cpx<T>); };
  if (lds(1) > 150 * 1024) return RowWaveShape{0, 0, 0};  // band limits far beyond a ring's length
  // float64 rows whose buffers leave room for one workgroup a compute unit where
  // row_kernel's (smaller by the padding) leave room for two: row_kernel (one item of
  // 1600 points: 33.6 against 42.2 us a Sinkhorn half; 1500 points 30.3 against 40.7;
  // 1536 and 1440 points fit twice: 26.8 and 26.6 against 34.1 and 31.8).  A prime
  // above 5 costs row_kernel more than that.
  if (!a.ring && a.max_prime <= 5 && lds(1) + 1024 > 80 * 1024 &&
      (size_t)3 * a.nlon * sizeof(cpx<T>) + 5 * 1024 <= 80 * 1024)
    return RowWaveShape{0, 0, 0};
  if (w.tp == 64) {
    // four neighbouring pairs per workgroup while the launch keeps 512 workgroups
    w.np = 4;
    while (w.np > 1 && (lds(w.np) > 40 * 1024 || pairs / w.np < 512)) w.np >>= 1;
    if (a.rpair && w.np > 1 && a.h % (8 * w.np) != 0) w.np = 1;
  }
  return w;
}

template <typename T>
hipError_t launch_rows_wave(const RowArgs<T>& a, int nb, const RowWaveShape& w, hipStream_t stream) {
  switch (kind_of(a.mode, a.k >= a.kT, a.in != nullptr)) {
    case RK_FWD: return launch_kind<T, RK_FWD>(a, nb, w, stream);
    case RK_INV: return launch_kind<T, RK_INV>(a, nb, w, stream);
    case RK_SINK: return a.gout ? launch_kind<T, RK_SINK | RK_KEEP>(a, nb, w, stream) : launch_kind<T, RK_SINK>(a, nb, w, stream);
    case RK_ADJ: return launch_kind<T, RK_ADJ>(a, nb, w, stream);
    case RK_ADJU_V1: return launch_kind<T, RK_ADJU_V1>(a, nb, w, stream);
    case RK_ADJU_B: return launch_kind<T, RK_ADJU_B>(a, nb, w, stream);
    case RK_ADJU_A: return launch_kind<T, RK_ADJU_A>(a, nb, w, stream);
    default: return hipErrorInvalidValue;
  }
}

template RowWaveShape row_wave_shape<float>(const RowArgs<float>&, int);
template RowWaveShape row_wave_shape<double>(const RowArgs<double>&, int);
template hipError_t launch_rows_wave<float>(const RowArgs<float>&, int, const RowWaveShape&, hipStream_t);
template hipError_t launch_rows_wave<double>(const RowArgs<double>&, int, const RowWaveShape&, hipStream_t);

}  // namespace shot
