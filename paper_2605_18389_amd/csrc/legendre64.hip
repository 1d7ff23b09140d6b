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

#include <hip/hip_ext.h>

#include "device_common.h"

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

template <int MODE, int BT>  // BT: 768 threads (168 registers) up to 384 latitude pairs, 1024 beyond
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
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
      __builtin_amdgcn_wave_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
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
  if (lds > 65536) {
    static size_t enabled = 65536;
    if (lds > enabled) {
      hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(&legendre_t64_kernel<MODE, BT>),
                                         hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
      if (e != hipSuccess) return e;
      enabled = lds;
    }
  }
  dim3 grid(a.L, (a.nb + 7) / 8);
  hipEvent_t e0, e1;
  if (take_launch_events(&e0, &e1))
    hipExtLaunchKernelGGL((legendre_t64_kernel<MODE, BT>), grid, dim3(128 * nc), lds, stream, e0, e1, 0, a);
  else
    hipLaunchKernelGGL((legendre_t64_kernel<MODE, BT>), grid, dim3(128 * nc), lds, stream, a);
  return hipGetLastError();
}

}  // namespace

bool t64_fits(int h) { return h <= 512 && t64_layout((h + 63) / 64).total <= 160 * 1024; }

hipError_t launch_legendre_t64(const LegArgs<double>& a, hipStream_t stream) {
  if (!t64_fits(a.h)) return hipErrorInvalidValue;
  const bool wide = a.h > 384;
  switch (a.mode) {
    case 0: return wide ? launch_mode<0, 1024>(a, stream) : launch_mode<0, 768>(a, stream);
    case 1: return wide ? launch_mode<1, 1024>(a, stream) : launch_mode<1, 768>(a, stream);
    default: return wide ? launch_mode<2, 1024>(a, stream) : launch_mode<2, 768>(a, stream);
  }
}

}  // namespace shot
