// tdt_dst.h -- sine transforms of rows and of columns: lengths whose interval
// count has small prime factors (tdt_dst.hip) or is at most kDstDenseMax
// (tdt_dst_dense.hip).
#pragma once
#include <stdint.h>
#include <vector>
#include <hip/hip_runtime.h>

namespace tdt {

// The transform of length n - 1 (n intervals): S_m = sum_{j=1}^{n-1} f_j
// sin(pi j m / n).  n = product of the radices below, 2 <= n <= kDstAnyMax
// (rows) or kDstColMax (columns), or any n <= kDstDenseMax.
constexpr int64_t kDstAnyMax = 8192;
constexpr int64_t kDstColMax = 1024;
constexpr int64_t kDstDenseMax = 512;
constexpr int kDstPasses = 10;
struct DstPlan {
  int n, np;                    // np = 0: dense, tw the matrix (dst_dense_table)
  int radix[kDstPasses];
  int ns[kDstPasses], nb[kDstPasses], step[kDstPasses];   // Ns, n / R, n / (R Ns)
  uint32_t magic[kDstPasses];   // floor(2^31 / Ns) + 1, Ns the product of the radices before
  const double* sn;             // sin(pi j / n), j < n (device)
  const double* tw;             // e^{-2 pi i q / n}, q < n, complex (device)
};
// n intervals have the factors 2, 3, 5, 7, 11 and 13 only (and fit), or are
// few enough for the matrix.
bool dst_any_supported(int64_t n, int64_t max_n);
// The radices, and the tables in long double on the host, uploaded into one
// allocation *mem that the caller frees.
hipError_t dst_plan_make(int64_t n, DstPlan& p, double** mem);
// out[r][m-1] = scale S_m of in[r][.], rows ldi / ldo apart.
hipError_t launch_dst_any_rows(const DstPlan& p, const double* in, double* out, int64_t rows,
                               int64_t ldi, int64_t ldo, double scale, hipStream_t st);
// Columns: column c < M of batch b has entry i at b ldb + i ld + c; ld and ldb
// even, 16-byte aligned arrays, columns in pairs (M odd: the entry after the
// last column of every row exists; the dense form asks for none of this).  out may be in.  Without ry: out =
// S.  With ry: the transform, times the factor of the ADI iterate, transformed
// again (the inverse up to the factor's scale):
//   norm (1 - ry[c][b] rz[c][m]) / (ly[b] + lz[m] + mu[c])   (dense: rz[m][c]).
struct DstColumns {
  const double* in;
  double* out;
  int64_t M, ld, nb, ldb;
  const double *ry, *rz;        // [M][ldy], [M][ldz] (dense: [n - 1][ldz]), or null
  const double *ly, *lz, *mu;
  int64_t ldy, ldz;
  double norm;
};
hipError_t launch_dst_columns(const DstPlan& p, const DstColumns& a, hipStream_t st);
// out[c][l] (modes_last: out[l][c]) = prod_{j < count[c]} (w[c][j] - x) / (w[c][j] + x), x = lam[l] +
// mu[c] / 2: an ADI cycle's error factor in one direction (w: [M][jmax]).
hipError_t launch_adi_factors(const double* w, const int* count, int jmax, const double* lam,
                              const double* mu, int64_t L, int64_t M, bool modes_last,
                              double* out, hipStream_t st);
// The dense form: its matrix in the order of the lanes, and the launches that
// the two above dispatch to.
void dst_dense_table(int64_t n, std::vector<double>& tab);
hipError_t launch_dst_dense_rows(const DstPlan& p, const double* in, double* out, int64_t rows,
                                 int64_t ldi, int64_t ldo, double scale, hipStream_t st);
hipError_t launch_dst_dense_columns(const DstPlan& p, const DstColumns& a, hipStream_t st);

}  // namespace tdt
