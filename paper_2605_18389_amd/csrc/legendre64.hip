// Matrix-core Legendre kernel of float64 tables.
//
// One workgroup per order m and chunk of 8 items (16 real columns).  Its waves
// are (64 latitudes, parity) pairs: a wave keeps its latitudes' spectra of one
// parity and their synthesis accumulators in registers (about 150, three waves
// per SIMD) and takes the order's rows of that parity 16 at a time, lane =
// latitude, coalesced 512-byte row reads, the next block's rows loaded while
// this one is contracted.  The table is read once for both transforms:
//   analysis   D[r][n] = sum_j P[r][j] Y[j][n]     K = the wave's 64 latitudes
//   combine    b[r][n] = h_l sum over the waves of D (fixed order), in LDS
//   synthesis  G[j][n] = sum_r P[r][j] b[r][n]     K = the block's 16 rows
// on v_mfma_f64_16x16x4_f64: A[i][k] in lane i + 16 k, B[k][j] in lane j + 16 k,
// D[i][j] in lane j + 16 (i mod 4), element i / 4.  Everything is float64.
// The vector-unit form it replaces (legendre_table_kernel) took one row per
// wave and pass, latitudes in LDS, the table read twice.  Heat apply, before ->
// after: 8 items at 33x64 46 -> 5.9 us, 12 at 180x360 307 -> 25, 16 at 360x720
// 542 -> 85, one at 721x1440 936 -> 222 us (750 MB of table, 3.4 TB/s).
// Bound: the table stream for few items (8 bytes per entry against 16 columns of
// matrix work); beyond about 8 items at L = 360 the float64 matrix rate.

#include "device_common.h"
#include "launch.h"

namespace shot {

namespace {

typedef double f64x4_t __attribute__((ext_vector_type(4)));

constexpr int T64_PLD = 68;  // tile row pitch (doubles)
constexpr int T64_DLD = 20;  // partials and b: row pitch per column

struct T64Layout {
  size_t o_p, o_d, o_b, total;
};
__host__ __device__ inline T64Layout t64_layout(int nc) {
  T64Layout q;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += (bytes + 15) / 16 * 16; return o; };
  q.o_p = take(sizeof(double) * 2 * nc * 16 * T64_PLD);
  q.o_d = take(sizeof(double) * 2 * nc * 16 * T64_DLD);
  q.o_b = take(sizeof(double) * 2 * 16 * T64_DLD);
  q.total = off;
  return q;
}

__device__ __forceinline__ void lanegroup_transpose4d(double* r) {
  unsigned lo[4], hi[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const unsigned long long u = (unsigned long long)__double_as_longlong(r[e]);
    lo[e] = (unsigned)u;
    hi[e] = (unsigned)(u >> 32);
  }
  lanegroup_transpose4(lo[0], lo[1], lo[2], lo[3]);
  lanegroup_transpose4(hi[0], hi[1], hi[2], hi[3]);
#pragma unroll
  for (int e = 0; e < 4; ++e)
    r[e] = __longlong_as_double((long long)((unsigned long long)lo[e] | ((unsigned long long)hi[e] << 32)));
}

template <int MODE, int BT>  // BT: 768 threads (168 registers) up to 384 latitude pairs, 1024 up to 448
__global__ void __launch_bounds__(BT) legendre_t64_kernel(LegArgs<double> A) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int L = A.L, h = A.h, hpad = A.hpad;
  const int nw = blockDim.x >> 6, nc = nw >> 1;  // waves; latitude chunks
  const T64Layout Q = t64_layout(nc);
  // an order's item chunks follow each other on one XCD (workgroups are dealt
  // round-robin to eight), longest orders first
  const int nch = gridDim.y, lin = blockIdx.x + gridDim.x * blockIdx.y;
  const int L8 = L & ~7;
  const int m = lin < L8 * nch ? 8 * (lin / (8 * nch)) + (lin & 7) : L8 + (lin - L8 * nch) / nch;
  const int chunk = lin < L8 * nch ? (lin >> 3) % nch : (lin - L8 * nch) % nch;
  const int c0 = 8 * chunk, nit = min(8, A.nb - c0);
  const int nr = L - m, nblk = (nr + 31) / 32;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int par = wave & 1, wc = wave >> 1;
  const int li = lane & 15, lg = lane >> 4;
  double* Pt = reinterpret_cast<double*>(smem_raw + Q.o_p) + (size_t)wave * 16 * T64_PLD;
  double* Dp = reinterpret_cast<double*>(smem_raw + Q.o_d);  // [wave][column][row]
  double* Bs = reinterpret_cast<double*>(smem_raw + Q.o_b);  // [parity][column][row]
  const long long toff = tri_off(m, L);
  const int j = 64 * wc + lane;
  const double* tabp = static_cast<const double*>(A.tab) + (size_t)toff * hpad + min(j, hpad - 1);
  double vn[16];
  auto load_rows = [&](int blk) {
#pragma unroll
    for (int k = 0; k < 16; ++k) vn[k] = tabp[(size_t)min(32 * blk + 2 * k + par, nr - 1) * hpad];
  };
  load_rows(0);
  // this lane's column (item li / 2, real or imaginary part) at latitudes 4 s + lg
  const int il = li >> 1;
  double yb[16];
  if constexpr (MODE != 2) {
    const double* sp = reinterpret_cast<const double*>(A.spec + A.items[A.item0 + c0 + min(il, nit - 1)].soff +
                                                       (size_t)m * h * 2 + par) + (li & 1);
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      const int jj = 64 * wc + 4 * s + lg;
      yb[s] = il < nit && jj < h ? sp[(size_t)4 * jj] : 0.0;
    }
  }
  // coefficients of this lane's column (synthesis alone)
  const double* cin = nullptr;
  if (MODE == 2 && il < nit)
    cin = reinterpret_cast<const double*>(A.coeff + A.items[A.item0 + c0 + il].coff + toff) + (li & 1);
  double bn[4];
  auto load_coeff = [&](int blk) {
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int r = 32 * blk + 2 * (4 * s + lg) + par;
      bn[s] = cin && r < nr ? cin[(size_t)2 * r] : 0.0;
    }
  };
  if constexpr (MODE == 2) load_coeff(0);
  f64x4_t G[4];
#pragma unroll
  for (int jt = 0; jt < 4; ++jt) G[jt] = f64x4_t{0.0, 0.0, 0.0, 0.0};

  for (int blk = 0; blk < nblk; ++blk) {
    double v[16], bc[4];
#pragma unroll
    for (int k = 0; k < 16; ++k) {
      v[k] = j < h ? vn[k] : 0.0;
      if (MODE != 2) Pt[k * T64_PLD + lane] = v[k];
    }
    if constexpr (MODE == 2) {
#pragma unroll
      for (int s = 0; s < 4; ++s) bc[s] = bn[s];
    }
    if (blk + 1 < nblk) {
      load_rows(blk + 1);
      if constexpr (MODE == 2) load_coeff(blk + 1);
    }
    if constexpr (MODE != 2) {
      wave_lds_sync();
      f64x4_t acc = f64x4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
      for (int s = 0; s < 16; ++s)
        acc = __builtin_amdgcn_mfma_f64_16x16x4f64(Pt[li * T64_PLD + 4 * s + lg], yb[s], acc, 0, 0, 0);
      double* d = Dp + ((size_t)wave * 16 + li) * T64_DLD + lg;
#pragma unroll
      for (int e = 0; e < 4; ++e) d[4 * e] = acc[e];
      __syncthreads();
      // b of both parities: one (column, row) per thread and round
      for (int idx = tid; idx < 512; idx += blockDim.x) {
        const int row = idx & 15, n = (idx >> 4) & 15, pp = idx >> 8;
        const int r = 32 * blk + 2 * row + pp;
        const double* dp = Dp + ((size_t)pp * 16 + n) * T64_DLD + row;
        double sum = 0.0;
        for (int w = 0; w < nc; ++w) sum += dp[(size_t)w * 2 * 16 * T64_DLD];
        const bool ok = r < nr && (n >> 1) < nit;
        const int item = A.item0 + c0 + min(n >> 1, nit - 1);
        if constexpr (MODE == 0) {
          const double hv = A.hl[(size_t)item * A.hl_stride + m + min(r, nr - 1)];
          Bs[((size_t)pp * 16 + n) * T64_DLD + row] = ok ? sum * hv : 0.0;
        } else if (ok) {
          reinterpret_cast<double*>(A.coeff + A.items[item].coff + toff + r)[n & 1] = sum;
        }
      }
      __syncthreads();
      if constexpr (MODE == 1) continue;
      const double* b = Bs + ((size_t)par * 16 + li) * T64_DLD + lg;
#pragma unroll
      for (int s = 0; s < 4; ++s) bc[s] = b[4 * s];
    }
    // k step s: rows 4 s + lane group
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      double a[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] = v[4 * s + e];
      lanegroup_transpose4d(a);
#pragma unroll
      for (int jt = 0; jt < 4; ++jt) G[jt] = __builtin_amdgcn_mfma_f64_16x16x4f64(a[jt], bc[s], G[jt], 0, 0, 0);
    }
  }
  if constexpr (MODE == 1) return;
  // G[j][n]: latitude 64 wc + 16 jt + 4 e + lg, this lane's column
  if (il < nit) {
    double* dst = reinterpret_cast<double*>(A.spec + A.items[A.item0 + c0 + il].soff + (size_t)m * h * 2 + par) + (li & 1);
#pragma unroll
    for (int jt = 0; jt < 4; ++jt)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int jj = 64 * wc + 16 * jt + 4 * e + lg;
        if (jj < h) dst[(size_t)4 * jj] = G[jt][e];
      }
  }
}

template <int MODE, int BT>
hipError_t launch_mode(const LegArgs<double>& a, hipStream_t stream) {
  const int nc = (a.h + 63) / 64;
  const size_t lds = t64_layout(nc).total;
  static std::atomic<unsigned long long> lds_set{0};
  hipError_t e = allow_lds(reinterpret_cast<const void*>(&legendre_t64_kernel<MODE, BT>), lds, lds_set);
  if (e != hipSuccess) return e;
  dim3 grid(a.L, (a.nb + 7) / 8);
  SHOT_LAUNCH((legendre_t64_kernel<MODE, BT>), grid, dim3(128 * nc), lds, stream, a);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Recurrence-fed form: a batch of a recurrence plan, float32 or float64.
//
// The split into workgroups and waves is that of the table kernel; the rows
// come from the rescaled recurrence R_{r+1} = c_{r+1} x R_r + R_{r-1}, run by
// each wave for its latitudes over all rows, 32 a block (both parity waves run
// it: 64 of a block's 2350 float64 cycles).  Float64 vector and matrix
// instructions share one unit (measured: 64 cycles a matrix instruction and 4.7
// a fused multiply-add, additive also over waves), so what can overlap is
// latency: the next block's rows are computed between this block's analysis
// instructions, a dependent chain, and its look-ahead loads fly meanwhile.  One
// barrier a block: waves exchange partial sums in D's own layout (which is also
// B's: rows 4 s + lane group of this lane's column) through two buffers.
// Everything is float64; the row-split kernel, which this replaces for batches,
// reduced its analysis sums across lanes in the field's precision.  Its cost was
// that reduction (32 values through 64 lanes for every 8 rows of 2 items) and
// the recurrence once per 2 items and pass.  Heat apply, row-split -> this:
// float32 16 and 24 items at Nside 64 16.7 -> 12.7 and 22.9 -> 15.9 us, 24 items
// at 180x360 33.2 -> 21.1, 24 at 256x512 57 -> 35, 8 at 721x1440 319 -> 192;
// float64 24 items at 256x512 71 -> 35.
// Bound: the float64 unit once several workgroups meet on a compute unit (24
// items at 256x512: 20 us of it), before that one order's chain of blocks
// (1.9 us each).  At 129 to 192 and 257 to 320 latitude pairs, 6 or 10 waves
// load the four SIMDs unevenly.
// ---------------------------------------------------------------------------

constexpr int R64_PLD = 66;  // tile row pitch (doubles)
// LDS position of tile row i: rows 4 s + k, k < 4, apart by 8 and 4 positions, so
// that neither the row-wise nor the column-wise operand reads meet in a bank
__device__ __forceinline__ constexpr int r64_pos(int i) { return 8 * (i & 1) + 4 * ((i >> 1) & 1) + (i >> 2); }

// Spectra of 8 items, 4 values a latitude, staged over the tiles and partials;
// the pitch puts four items' columns into different banks.
template <typename T>
__host__ __device__ constexpr int r64_stage(int h) { return (4 * h + 63) / 64 * 64 + (sizeof(T) == 4 ? 16 : 8); }

struct R64Layout {
  size_t o_p, o_d, o_c, o_g, total;
};
__host__ __device__ inline R64Layout r64_layout(int L, int nc) {
  R64Layout q;
  size_t off = 0;
  auto take = [&](size_t bytes) { size_t o = off; off += (bytes + 15) / 16 * 16; return o; };
  const int npl0 = (L + 31) / 32 * 32 + 4, npl = npl0 > 128 * nc ? npl0 : 128 * nc;
  q.o_p = take(sizeof(double) * 2 * nc * 16 * R64_PLD);
  q.o_d = take(sizeof(double) * 2 * 2 * nc * 256);
  q.o_c = take(sizeof(double) * npl);
  q.o_g = take(sizeof(double) * npl);
  q.total = off;
  return q;
}

template <typename T, int MODE, int BT>
__global__ void __launch_bounds__(BT, 3) legendre_r64_kernel(LegArgs<T> A) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  const int L = A.L, h = A.h;
  const int nw = blockDim.x >> 6, nc = nw >> 1;  // waves; latitude chunks
  const R64Layout Q = r64_layout(L, nc);
  const int nch = gridDim.y, lin = blockIdx.x + gridDim.x * blockIdx.y;
  const int L8 = L & ~7;
  const int m = lin < L8 * nch ? 8 * (lin / (8 * nch)) + (lin & 7) : L8 + (lin - L8 * nch) / nch;
  const int chunk = lin < L8 * nch ? (lin >> 3) % nch : (lin - L8 * nch) % nch;
  const int c0 = 8 * chunk, nit = min(8, A.nb - c0);
  const int nr = L - m, nblk = (nr + 31) / 32;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int par = wave & 1, wc = wave >> 1;
  const int li = lane & 15, lg = lane >> 4, il = li >> 1;
  const int pli = r64_pos(li), plg = r64_pos(lg);  // tile rows li and lg
  double* Pt = reinterpret_cast<double*>(smem_raw + Q.o_p) + (size_t)wave * 16 * R64_PLD;
  double2* Dp = reinterpret_cast<double2*>(smem_raw + Q.o_d);  // [buffer][wave][2][lane]
  double* cf = reinterpret_cast<double*>(smem_raw + Q.o_c);
  double* gm = reinterpret_cast<double*>(smem_raw + Q.o_g);
  const long long toff = tri_off(m, L);
  const int j = 64 * wc + lane, jc = min(j, h - 1);
  // loads of the prologue at clamped addresses, issued before the first use.  The
  // spectra (E and O of a latitude in one 16- or 32-byte entry) pass through LDS:
  // thread (item mod 2, latitude) here, lane (column, latitude mod 4) below.
  const int half = wave >= nc ? 1 : 0, ql = tid - 64 * nc * half, qc = min(ql, h - 1);
  const int sp = r64_stage<T>(h);  // stage pitch per item
  T* stage = reinterpret_cast<T*>(smem_raw + Q.o_p);
  typedef T v4_t __attribute__((ext_vector_type(4)));
  v4_t* spec4 = reinterpret_cast<v4_t*>(A.spec + A.soff0) + ((size_t)c0 * L + m) * h;
  v4_t sv[4];
  if constexpr (MODE != 2) {
#pragma unroll
    for (int k = 0; k < 4; ++k) sv[k] = spec4[(size_t)min(2 * k + half, nit - 1) * L * h + qc];
  }
  const size_t co = MODE == 0 ? 0 : A.items[A.item0 + c0 + min(il, nit - 1)].coff;
  const double seed = A.rseed[(size_t)m * h + jc], xn = A.xs[jc];
  const double c_ = A.rcoef[toff + min(tid, nr - 1)], g_ = A.rgam[toff + min(tid, nr - 1)];
  cf[tid] = tid < nr ? c_ : 0.0;
  gm[tid] = tid < nr ? g_ : 0.0;
  for (int q = tid + blockDim.x; q < 32 * nblk + 4; q += blockDim.x) {
    const int r = min(q, nr - 1);
    const double c = A.rcoef[toff + r], g = A.rgam[toff + r];
    cf[q] = q < nr ? c : 0.0;
    gm[q] = q < nr ? g : 0.0;
  }
  T yb[16];
  if constexpr (MODE != 2) {
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (ql < h) {
        const v4_t z = {(T)0, (T)0, (T)0, (T)0};
        *reinterpret_cast<v4_t*>(stage + (2 * k + half) * sp + 4 * ql) = 2 * k + half < nit ? sv[k] : z;
      }
  }
  const T* cin = MODE == 2 ? reinterpret_cast<const T*>(A.coeff + co + toff) + (li & 1) : nullptr;
  T* cout = MODE == 1 ? reinterpret_cast<T*>(A.coeff + co + toff) + (li & 1) : nullptr;
  const T* hl = A.hl + (size_t)(A.item0 + c0 + min(il, nit - 1)) * A.hl_stride + m;
  f64x4_t G[4];
#pragma unroll
  for (int jt = 0; jt < 4; ++jt) G[jt] = f64x4_t{0.0, 0.0, 0.0, 0.0};
  __syncthreads();
  if constexpr (MODE != 2) {
#pragma unroll
    for (int s = 0; s < 16; ++s) {
      const int jj = 64 * wc + 4 * s + lg;
      const T y = stage[il * sp + 4 * min(jj, h - 1) + 2 * par + (li & 1)];
      yb[s] = jj < h ? y : (T)0;
    }
    __syncthreads();  // the tiles take the stage's place
  }
  const double xj = j < h ? xn : 0.0;
  double R1 = j < h ? seed : 0.0, R2 = 0.0;
  if (par) {
    const double rn = cf[1] * xj * R1;
    R2 = R1;
    R1 = rn;
  }
  // quarter q of a block's rows (four of this wave's parity); coefficients cc
  double v[16];
  auto coefs = [&](double* cc, int blk, int q) {
#pragma unroll
    for (int k = 0; k < 8; ++k) cc[k] = cf[32 * blk + 8 * q + k + par + 1];
  };
  auto advance = [&](const double* cc) {  // by two rows
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      const double rn = fma(cc[u] * xj, R1, R2);
      R2 = R1;
      R1 = rn;
    }
  };
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    double cc[8];
    coefs(cc, 0, q);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[4 * q + e] = R1;
      advance(cc + 2 * e);
    }
  }
  T hn[4];
  auto load_b = [&](int blk) {  // multipliers (heat) or coefficients (synthesis) of a block's rows
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int r = 32 * blk + 2 * (4 * s + lg) + par;
      if (MODE == 0) hn[s] = hl[min(r, nr - 1)];
      if (MODE == 2) hn[s] = cin[(size_t)2 * min(r, nr - 1)];
    }
  };
  load_b(0);
  for (int blk = 0; blk < nblk; ++blk) {
    double bc[4];
    T hv[4];
#pragma unroll
    for (int s = 0; s < 4; ++s) hv[s] = hn[s];
    const int next = min(blk + 1, nblk - 1);  // (the last block's look-ahead is not used)
    load_b(next);
#pragma unroll
    for (int k = 0; k < 16; ++k) Pt[r64_pos(k) * R64_PLD + lane] = v[k];
    wave_lds_sync();
    double pa[2][4];
    f64x4_t acc = f64x4_t{0.0, 0.0, 0.0, 0.0};
    auto frag = [&](double* p, int q) {
      if (MODE == 2) return;
#pragma unroll
      for (int e = 0; e < 4; ++e) p[e] = Pt[pli * R64_PLD + 16 * q + 4 * e + lg];
    };
    frag(pa[0], 0);
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      double cc[8];
      coefs(cc, next, q);
      if (q < 3) frag(pa[(q + 1) & 1], q + 1);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (MODE != 2) acc = __builtin_amdgcn_mfma_f64_16x16x4f64(pa[q & 1][e], (double)yb[4 * q + e], acc, 0, 0, 0);
        v[4 * q + e] = R1;
        advance(cc + 2 * e);
      }
      asm volatile("" : "+v"(R1), "+v"(R2));  // here, in the matrix instructions' shadow, not where v is used
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (MODE != 2) {
      // a lane holds the rows and column of D that it needs of b
      double2* buf = Dp + (size_t)(blk & 1) * nw * 128 + lane;
      buf[128 * wave] = make_double2(acc[0], acc[1]);
      buf[128 * wave + 64] = make_double2(acc[2], acc[3]);
      __syncthreads();
#pragma unroll
      for (int s = 0; s < 4; ++s) bc[s] = 0.0;
#pragma unroll 1
      for (int w = par; w < nw; w += 2) {
        const double2 d0 = buf[128 * w], d1 = buf[128 * w + 64];
        bc[0] += d0.x;
        bc[1] += d0.y;
        bc[2] += d1.x;
        bc[3] += d1.y;
      }
    }
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int r = 32 * blk + 2 * (4 * s + lg) + par;
      const double g = gm[r];
      if constexpr (MODE == 0) bc[s] *= g * g * (double)hv[s];
      if constexpr (MODE == 1) {
        if (wc == 0 && il < nit && r < nr) cout[(size_t)2 * r] = (T)(bc[s] * g);
      }
      if constexpr (MODE == 2) bc[s] = (double)hv[s] * g;
    }
    if constexpr (MODE != 1) {
#pragma unroll
      for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int jt = 0; jt < 4; ++jt)
          G[jt] = __builtin_amdgcn_mfma_f64_16x16x4f64(Pt[(s + plg) * R64_PLD + 16 * jt + li], bc[s], G[jt], 0, 0, 0);
    }
  }
  if constexpr (MODE == 1) return;
  __syncthreads();
#pragma unroll
  for (int jt = 0; jt < 4; ++jt)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int jj = 64 * wc + 16 * jt + 4 * e + lg;
      if (jj < h) stage[il * sp + 4 * jj + 2 * par + (li & 1)] = (T)G[jt][e];
    }
  __syncthreads();
  if (ql < h)
#pragma unroll
    for (int k = 0; k < 4; ++k)
      if (2 * k + half < nit)
        spec4[(size_t)(2 * k + half) * L * h + ql] = *reinterpret_cast<v4_t*>(stage + (2 * k + half) * sp + 4 * ql);
}

template <typename T, int MODE, int BT>
hipError_t launch_r64_mode(const LegArgs<T>& a, hipStream_t stream) {
  const int nc = (a.h + 63) / 64;
  const size_t lds = r64_layout(a.L, nc).total;
  static std::atomic<unsigned long long> lds_set{0};
  hipError_t e = allow_lds(reinterpret_cast<const void*>(&legendre_r64_kernel<T, MODE, BT>), lds, lds_set);
  if (e != hipSuccess) return e;
  dim3 grid(a.L, (a.nb + 7) / 8);
  SHOT_LAUNCH((legendre_r64_kernel<T, MODE, BT>), grid, dim3(128 * nc), lds, stream, a);
  return hipGetLastError();
}

template <typename T, int BT>
hipError_t launch_r64_bt(const LegArgs<T>& a, hipStream_t stream) {
  switch (a.mode) {
    case 0: return launch_r64_mode<T, 0, BT>(a, stream);
    case 1: return launch_r64_mode<T, 1, BT>(a, stream);
    default: return launch_r64_mode<T, 2, BT>(a, stream);
  }
}

}  // namespace

bool t64_fits(int h) { return t64_layout((h + 63) / 64).total <= 160 * 1024; }  // h <= 448

hipError_t launch_legendre_t64(const LegArgs<double>& a, hipStream_t stream) {
  if (!t64_fits(a.h)) return hipErrorInvalidValue;
  const bool wide = a.h > 384;
  switch (a.mode) {
    case 0: return wide ? launch_mode<0, 1024>(a, stream) : launch_mode<0, 768>(a, stream);
    case 1: return wide ? launch_mode<1, 1024>(a, stream) : launch_mode<1, 768>(a, stream);
    default: return wide ? launch_mode<2, 1024>(a, stream) : launch_mode<2, 768>(a, stream);
  }
}

bool r64_fits(int L, int h) { return h <= 384 && r64_layout(L, (h + 63) / 64).total <= 160 * 1024; }

template <typename T>
hipError_t launch_legendre_r64(const LegArgs<T>& a, hipStream_t stream) {
  if (!r64_fits(a.L, a.h)) return hipErrorInvalidValue;
  if (a.h <= 128) return launch_r64_bt<T, 256>(a, stream);
  return launch_r64_bt<T, 768>(a, stream);
}
template hipError_t launch_legendre_r64<float>(const LegArgs<float>&, hipStream_t);
template hipError_t launch_legendre_r64<double>(const LegArgs<double>&, hipStream_t);

}  // namespace shot
