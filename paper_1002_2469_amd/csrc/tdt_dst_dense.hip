// tdt_dst_dense.hip -- sine transforms as matrix products, for interval counts
// n <= 512 with a prime factor above 13 (17, 51, 301, ...), along rows and
// along columns.
//
// S_m = sum_i f_i sin(pi i m / n): with s_i = f_i + f_{n-i} and d_i = f_i -
// f_{n-i} the odd m need the s_i (i <= n/2) only and the even m the d_i (i <
// n/2), two products of half the size on the fp64 matrix instructions
// (16 x 16 x 4).  A workgroup keeps 16 CT sequences whole in LDS, folded in
// place, so the transform may be in place and the 3D iterate's two transforms
// and factor are one pass over HBM; its eight wavefronts share the 16-row
// tiles of the matrix, whose entries come from L2 in the order of the lanes.
//
// Bound by the matrix units from n of about 150 on (n flops per entry; the rows
// of 300^3 points, n = 301: 8.1 GFLOP in 216 us, 38 TFLOP/s), by HBM below
// (50 x 100000 points, 80 MB, 44 us), by launches when small.  Before, a
// library FFT between fold, split and prefix-sum kernels, transposes around
// the 2D line solves and the iterated 3D half-steps: 2D 50 x 1000 points 42 ->
// 20 us, 250 x 20000 360 -> 140, 508 x 60000 2263 -> 1088; 3D 40 x 50 x 59 602 ->
// 28, 100^3 781 -> 55, 300^3 6926 -> 1286.  Above 512 the matrix outgrows both the
// work saved and the LDS.  Where there are at least two workgroups per compute
// unit, 32 sequences share each load of the matrix (CT = 2); below, 16 (more
// workgroups), and a few rows' tiles are dealt to several workgroups (508 x 500
// points 97 -> 35 us).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cmath>
#include <vector>

#include "tdt_dst.h"
#include "tdt_internal.h"

namespace tdt {
namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));
constexpr int kDenseNT = 512;

// Tiles of 16 coefficients and steps of 4 entries of the odd and even halves.
__host__ __device__ inline int dense_tiles(int n, int even) { return ((even ? (n - 1) / 2 : n / 2) + 15) / 16; }
__host__ __device__ inline int dense_steps(int n, int even) { return ((even ? (n - 1) / 2 : n / 2) + 3) / 4; }

// The products of one wavefront: tiles w, w + step, ... (the odd half's first).
// get(k, h): entry k (1-based position in the folded sequence) of the lane's
// sequence h; TABLE_A: the matrix is the left operand (columns of an array),
// else the right one (rows).
template <int TPW, int CT, bool TABLE_A, class Get>
__device__ __forceinline__ void dense_products(const double* __restrict__ tab, int n, int w,
                                               int step, int lane, const Get& get,
                                               f64x4 (&acc)[TPW][CT]) {
  const int to = dense_tiles(n, 0), te = dense_tiles(n, 1);
  const int ko = dense_steps(n, 0), ke = dense_steps(n, 1);
  const int kq = lane / 16;
#pragma unroll
  for (int q = 0; q < TPW; ++q) {
#pragma unroll
    for (int h = 0; h < CT; ++h) acc[q][h] = f64x4{0.0, 0.0, 0.0, 0.0};
    const int tile = w + step * q;   // uniform in the wavefront
    if (tile >= to + te) continue;
    const bool even = tile >= to;
    const int ks = even ? ke : ko;
    const double* tb = tab + (even ? (int64_t)to * ko + (int64_t)(tile - to) * ke
                                   : (int64_t)tile * ko) * 64 + lane;
    // s_i at position i, d_i at n - i; steps past the last entry meet zeros of
    // the matrix (and positions inside the sequence, n >= 17)
    const int p0 = even ? n - 1 - kq : 1 + kq, dp = even ? -4 : 4;
    if constexpr (TPW == 1) {
#pragma unroll 8
      for (int s = 0; s < ks; ++s) {
        const double a = tb[s * 64];
#pragma unroll
        for (int h = 0; h < CT; ++h) {
          const double b = get(p0 + dp * s, h);
          acc[q][h] = TABLE_A ? __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, acc[q][h], 0, 0, 0)
                              : __builtin_amdgcn_mfma_f64_16x16x4f64(b, a, acc[q][h], 0, 0, 0);
        }
      }
      continue;
    }
    // Eight steps' matrix entries are requested while the eight before are
    // used: with one or two workgroups per compute unit their latency was the
    // bound (300^3 rows 455 -> 216 us).  Short sequences (TPW = 1) have more
    // workgroups, and lose some to the registers (100^3 solve 60 -> 68 us).
    constexpr int U = 8;
    double a[U], an[U];
#pragma unroll
    for (int u = 0; u < U; ++u) a[u] = tb[min(u, ks - 1) * 64];
    for (int s0 = 0; s0 < ks; s0 += U) {
#pragma unroll
      for (int u = 0; u < U; ++u) an[u] = tb[min(s0 + U + u, ks - 1) * 64];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (s0 + u >= ks) break;
        const int pos = p0 + dp * (s0 + u);
#pragma unroll
        for (int h = 0; h < CT; ++h) {
          const double b = get(pos, h);
          acc[q][h] = TABLE_A ? __builtin_amdgcn_mfma_f64_16x16x4f64(a[u], b, acc[q][h], 0, 0, 0)
                              : __builtin_amdgcn_mfma_f64_16x16x4f64(b, a[u], acc[q][h], 0, 0, 0);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) a[u] = an[u];
    }
  }
}

// The coefficient of entry e (0 .. 15) of tile `tile`.
__device__ __forceinline__ int dense_coef(int n, int tile, int e) {
  const int to = dense_tiles(n, 0);
  return tile < to ? 2 * (16 * tile + e) + 1 : 2 * (16 * (tile - to) + e) + 2;
}

// Columns: see launch_dst_columns (rz here [n - 1][ldz], modes last).
template <int NMAX, int CT, bool FACTOR>
__global__ __launch_bounds__(kDenseNT, 2) void k_dst_dense_columns(const double* __restrict__ tab,
                                                                int n, DstColumns A) {
  constexpr int C = 16 * CT, TPW = (NMAX + 127) / 128, RS = kDenseNT / C;
  __shared__ double buf[NMAX * C];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  // position p of column c; odd positions of 32 columns swap their halves
  // (a wavefront reads 16 columns of 4 positions)
  auto at = [&](int p, int c) -> double& {
    return buf[(p - 1) * C + (CT == 2 ? c ^ ((p & 1) * 16) : c)];
  };
  const uint32_t groups = (uint32_t)((A.M + C - 1) / C);
  const int64_t bt = blockIdx.x / groups;
  const int64_t c0 = (int64_t)(blockIdx.x - (uint32_t)bt * groups) * C;
  const int hc = t % C, hr = t / C;
  const bool la = c0 + hc < A.M;
  {
    const double* f = A.in + bt * A.ldb + (la ? c0 + hc : 0) - A.ld;
    constexpr int U = 4;
    for (int i0 = 1 + hr; i0 <= n / 2; i0 += U * RS) {
      double a[U], b[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + u * RS;
        a[u] = b[u] = 0.0;
        if (la && i <= n / 2) {
          a[u] = f[i * A.ld];
          b[u] = f[(n - i) * A.ld];
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int i = i0 + u * RS;
        if (i <= n / 2) {
          if (2 * i < n) at(n - i, hc) = a[u] - b[u];
          at(i, hc) = 2 * i < n ? a[u] + b[u] : a[u];
        }
      }
    }
  }
  __syncthreads();
  f64x4 acc[TPW][CT];
  auto get = [&](int p, int h) { return at(p, 16 * h + (lane & 15)); };
  dense_products<TPW, CT, true>(tab, n, w, 8, lane, get, acc);
  // the lane's entries: coefficient row 4 v + lane / 16 of a tile, column
  // 16 h + lane % 16
  if constexpr (FACTOR) {
    __syncthreads();   // the folded sequences are read
#pragma unroll
    for (int h = 0; h < CT; ++h) {
      const int cl = 16 * h + (lane & 15);
      const int64_t c = c0 + cl < A.M ? c0 + cl : 0;
      const double y = A.ry[c * A.ldy + bt], d = A.ly[bt] + A.mu[c];
#pragma unroll
      for (int q = 0; q < TPW; ++q)
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int m = dense_coef(n, w + 8 * q, 4 * v + lane / 16);
          if (m < n)
            at(m, cl) = acc[q][h][v] *
                        (A.norm * (1.0 - y * A.rz[(m - 1) * A.ldz + c]) / (A.lz[m - 1] + d));
        }
    }
    __syncthreads();
    for (int i = 1 + hr; 2 * i < n; i += RS) {
      const double a = at(i, hc), b = at(n - i, hc);
      at(i, hc) = a + b;
      at(n - i, hc) = a - b;
    }
    __syncthreads();
    dense_products<TPW, CT, true>(tab, n, w, 8, lane, get, acc);
  }
#pragma unroll
  for (int h = 0; h < CT; ++h) {
    const int64_t c = c0 + 16 * h + (lane & 15);
    if (c >= A.M) continue;
    double* o = A.out + bt * A.ldb + c - A.ld;
#pragma unroll
    for (int q = 0; q < TPW; ++q)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int m = dense_coef(n, w + 8 * q, 4 * v + lane / 16);
        if (m < n) o[m * A.ld] = acc[q][h][v];
      }
  }
}

// Rows, 16 CT per workgroup, the tiles dealt to `parts` workgroups (few rows:
// in and out are different arrays).  A pitch of twice an odd number: 16 rows
// of 2 positions without bank conflicts.
template <int NMAX, int CT>
__global__ __launch_bounds__(kDenseNT, 2) void k_dst_dense_rows(const double* __restrict__ tab, int n,
                                                             const double* __restrict__ in,
                                                             double* __restrict__ out, int64_t rows,
                                                             int64_t ldi, int64_t ldo, double scale,
                                                             int parts) {
  constexpr int R = 16 * CT, TPW = (NMAX + 127) / 128, PITCH = NMAX == 320 ? 318 : NMAX + 2;
  __shared__ double buf[R * PITCH];
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  const int64_t r0 = (int64_t)(blockIdx.x / parts) * R;
  const int w0 = w + 8 * (int)(blockIdx.x % parts);
  for (int i = 1 + lane; i <= n / 2; i += 64) {
    double a[R / 8], b[R / 8];
#pragma unroll
    for (int u = 0; u < R / 8; ++u) {
      const int64_t r = r0 + w + 8 * u;
      a[u] = b[u] = 0.0;
      if (r < rows) {
        const double* f = in + r * ldi - 1;
        a[u] = f[i];
        b[u] = f[n - i];
      }
    }
#pragma unroll
    for (int u = 0; u < R / 8; ++u) {
      double* z = buf + (w + 8 * u) * PITCH - 1;
      if (2 * i < n) z[n - i] = a[u] - b[u];
      z[i] = 2 * i < n ? a[u] + b[u] : a[u];
    }
  }
  __syncthreads();
  f64x4 acc[TPW][CT];
  dense_products<TPW, CT, false>(
      tab, n, w0, 8 * parts, lane,
      [&](int p, int h) { return buf[(16 * h + (lane & 15)) * PITCH + p - 1]; }, acc);
  // the lane's entries: row 16 h + 4 v + lane / 16, coefficient lane % 16
#pragma unroll
  for (int q = 0; q < TPW; ++q) {
    const int m = dense_coef(n, w0 + 8 * parts * q, lane & 15);
    if (m >= n) continue;
#pragma unroll
    for (int h = 0; h < CT; ++h)
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t r = r0 + 16 * h + 4 * v + lane / 16;
        if (r < rows) out[r * ldo + m - 1] = scale * acc[q][h][v];
      }
  }
}

template <int NMAX, int CT>
void dense_rows(const DstPlan& p, const double* in, double* out, int64_t rows, int64_t ldi,
                int64_t ldo, double scale, hipStream_t st) {
  const int64_t g = (rows + 16 * CT - 1) / (16 * CT);
  const int tiles = dense_tiles(p.n, 0) + dense_tiles(p.n, 1);
  int parts = 1;
  while (g * 2 * parts <= device_cus() && 8 * parts < tiles) parts *= 2;
  hipLaunchKernelGGL((k_dst_dense_rows<NMAX, CT>), dim3((unsigned)(g * parts)), dim3(kDenseNT), 0,
                     st, p.tw, p.n, in, out, rows, ldi, ldo, scale, parts);
}

template <int NMAX, int CT>
void dense_columns(const DstPlan& p, const DstColumns& a, hipStream_t st) {
  const int64_t g = (a.M + 16 * CT - 1) / (16 * CT) * a.nb;
  if (a.ry)
    hipLaunchKernelGGL((k_dst_dense_columns<NMAX, CT, true>), dim3((unsigned)g), dim3(kDenseNT), 0,
                       st, p.tw, p.n, a);
  else
    hipLaunchKernelGGL((k_dst_dense_columns<NMAX, CT, false>), dim3((unsigned)g), dim3(kDenseNT),
                       0, st, p.tw, p.n, a);
}

}  // namespace

void dst_dense_table(int64_t n, std::vector<double>& tab) {
  const long double pi = 3.141592653589793238462643383279502884L;
  std::vector<double> sn((size_t)(2 * n));   // sin(pi q / n)
  for (int64_t q = 0; q < 2 * n; ++q)
    sn[(size_t)q] = (double)std::sin(pi * (long double)q / (long double)n);
  tab.clear();
  for (int even = 0; even < 2; ++even) {
    const int K = even ? (int)(n - 1) / 2 : (int)n / 2;
    const int steps = dense_steps((int)n, even);
    for (int t = 0; t < dense_tiles((int)n, even); ++t)
      for (int s = 0; s < steps; ++s)
        for (int l = 0; l < 64; ++l) {
          const int64_t m = 2 * (16 * t + l % 16) + 1 + even, i = 4 * s + l / 16 + 1;
          tab.push_back(m < n && i <= K ? sn[(size_t)(i * m % (2 * n))] : 0.0);
        }
  }
}

hipError_t launch_dst_dense_rows(const DstPlan& p, const double* in, double* out, int64_t rows,
                                 int64_t ldi, int64_t ldo, double scale, hipStream_t st) {
  if (p.n < 17 || p.n > kDstDenseMax || rows < 1 || (rows + 15) / 16 > 0x7fffffff)
    return hipErrorInvalidValue;
  const bool two = (rows + 31) / 32 >= 2 * (int64_t)device_cus();
#define TDT_DENSE(N)                                                        \
  if (two) dense_rows<N, 2>(p, in, out, rows, ldi, ldo, scale, st);         \
  else dense_rows<N, 1>(p, in, out, rows, ldi, ldo, scale, st)
  if (p.n <= 128) { TDT_DENSE(128); }
  else if (p.n <= 256) { TDT_DENSE(256); }
  else if (p.n < 320) { TDT_DENSE(320); }   // two workgroups' LDS per compute unit
  else { TDT_DENSE(512); }
#undef TDT_DENSE
  return hipGetLastError();
}

hipError_t launch_dst_dense_columns(const DstPlan& p, const DstColumns& a, hipStream_t st) {
  if (p.n < 17 || p.n > kDstDenseMax || a.M < 1 || a.nb < 1 ||
      (a.M + 15) / 16 * a.nb > 0x7fffffff)
    return hipErrorInvalidValue;
  const bool two = (a.M + 31) / 32 * a.nb >= 2 * (int64_t)device_cus();
#define TDT_DENSE(N)                        \
  if (two) dense_columns<N, 2>(p, a, st);   \
  else dense_columns<N, 1>(p, a, st)
  if (p.n <= 128) { TDT_DENSE(128); }
  else if (p.n <= 256) { TDT_DENSE(256); }
  else if (p.n < 320) { TDT_DENSE(320); }   // two workgroups' LDS per compute unit
  else { TDT_DENSE(512); }
#undef TDT_DENSE
  return hipGetLastError();
}

}  // namespace tdt
