// tdt_dst.hip -- fused sine transforms for interval counts with small prime
// factors, along rows and along columns (a slow axis) of an array.
//
// Two real sequences share one complex FFT: z = A + i B, both folded as in
// the power-of-two transform (y_0 = 0, y_j = sin(pi j / n)(f_j + f_{n-j}) +
// (f_j - f_{n-j}) / 2; Makhoul, IEEE Trans. ASSP 28, 1980), so that any n, odd
// or even, takes one FFT of length n for two rows.  The FFT is a mixed-radix
// Stockham autosort in LDS (radices 8, 4, 2, 3, 5, 7, 11, 13; Govindaraju et
// al., SC 2008), in place: every pass reads its inputs into registers before
// any thread writes.  From Z the two transforms are Y^A_k = (Z_k + conj
// Z_{n-k}) / 2, Y^B_k = (Z_k - conj Z_{n-k}) / 2i, S_2k = -Im Y_k, and the odd
// coefficients are the prefix sums of Re Y_k.  One pass over HBM, where a
// library FFT between separate fold, split and prefix-sum kernels takes four:
// the 2D solve of 999 x 1499 points 86 -> 42 us, of 4094 x 4000 1434 -> 257 us (with the
// in-place line solves it allows).
//
// Bound by HBM on large arrays (columns of 511 entries: 445 us for 2.15 GB,
// 4.8 TB/s), by the passes' barriers on small ones.  68 to 124 VGPRs: the
// addresses of one pass are hidden from the next (opaque), without which the
// compiler kept them all (250 VGPRs, spills).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <cmath>
#include <vector>

#include "tdt_dst.h"
#include "tdt_internal.h"

namespace tdt {
namespace {

__device__ __forceinline__ double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ double2 csub(double2 a, double2 b) { return make_double2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ double2 cmul(double2 a, double2 b) {
  return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// cos and sin of 2 pi m / R, m = 1 .. (R-1)/2
template <int R> struct Trig;
template <> struct Trig<3> {
  static constexpr double c[1] = {-0.5}, s[1] = {0.86602540378443864676};
};
template <> struct Trig<5> {
  static constexpr double c[2] = {0.3090169943749474241, -0.8090169943749474241};
  static constexpr double s[2] = {0.95105651629515357212, 0.58778525229247312917};
};
template <> struct Trig<7> {
  static constexpr double c[3] = {0.62348980185873353053, -0.22252093395631440429,
                                  -0.90096886790241912624};
  static constexpr double s[3] = {0.78183148246802980871, 0.97492791218182360702,
                                  0.43388373911755812048};
};
template <> struct Trig<11> {
  static constexpr double c[5] = {0.84125353283118116886, 0.41541501300188642553,
                                  -0.14231483827328514044, -0.65486073394528506406,
                                  -0.95949297361449738989};
  static constexpr double s[5] = {0.54064081745559758211, 0.90963199535451837141,
                                  0.98982144188093273238, 0.75574957435425828377,
                                  0.28173255684142969771};
};
template <> struct Trig<13> {
  static constexpr double c[6] = {0.8854560256532098959,   0.56806474673115580251,
                                  0.12053668025532305335,  -0.35460488704253562597,
                                  -0.74851074817110109863, -0.97094181742605202716};
  static constexpr double s[6] = {0.46472317204376854566, 0.82298386589365639458,
                                  0.9927088740980539928,  0.93501624268541482344,
                                  0.66312265824079520238, 0.23931566428755776715};
};

// An index hidden from the optimiser: the addresses derived from it are formed
// where they are used instead of being kept live from one pass to the next.
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// Orders the LDS accesses of a sequence's T threads: a barrier where they span
// wavefronts; inside one wavefront its LDS operations complete in order, and
// only the compiler has to keep them so.
template <int T>
__device__ __forceinline__ void seq_sync() {
  if constexpr (T > 64) {
    __syncthreads();
  } else {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
  }
}

// R-point DFT in place, X_k = sum_r v_r e^{-2 pi i r k / R}
__device__ __forceinline__ void dft4(double2& x0, double2& x1, double2& x2, double2& x3) {
  const double2 s0 = cadd(x0, x2), d0 = csub(x0, x2), s1 = cadd(x1, x3), d1 = csub(x1, x3);
  x0 = cadd(s0, s1);
  x1 = make_double2(d0.x + d1.y, d0.y - d1.x);
  x2 = csub(s0, s1);
  x3 = make_double2(d0.x - d1.y, d0.y + d1.x);
}
template <int R>
__device__ __forceinline__ void dft(double2 (&v)[R]) {
  if constexpr (R == 2) {
    const double2 a = v[0];
    v[0] = cadd(a, v[1]);
    v[1] = csub(a, v[1]);
  } else if constexpr (R == 4) {
    dft4(v[0], v[1], v[2], v[3]);
  } else if constexpr (R == 8) {
    dft4(v[0], v[2], v[4], v[6]);
    dft4(v[1], v[3], v[5], v[7]);
    constexpr double h = 0.70710678118654752440;
    const double2 o0 = v[1];
    const double2 o1 = make_double2(h * (v[3].x + v[3].y), h * (v[3].y - v[3].x));
    const double2 o2 = make_double2(v[5].y, -v[5].x);
    const double2 o3 = make_double2(h * (v[7].y - v[7].x), -h * (v[7].x + v[7].y));
    const double2 e0 = v[0], e1 = v[2], e2 = v[4], e3 = v[6];
    v[0] = cadd(e0, o0);
    v[4] = csub(e0, o0);
    v[1] = cadd(e1, o1);
    v[5] = csub(e1, o1);
    v[2] = cadd(e2, o2);
    v[6] = csub(e2, o2);
    v[3] = cadd(e3, o3);
    v[7] = csub(e3, o3);
  } else {
    // odd prime: sums and differences of v_r and v_{R-r}
    constexpr int H = (R - 1) / 2;
    double2 s[H], d[H];
#pragma unroll
    for (int r = 0; r < H; ++r) {
      s[r] = cadd(v[r + 1], v[R - 1 - r]);
      d[r] = csub(v[r + 1], v[R - 1 - r]);
    }
    const double2 x0 = v[0];
#pragma unroll
    for (int r = 0; r < H; ++r) v[0] = cadd(v[0], s[r]);
#pragma unroll
    for (int k = 1; k <= H; ++k) {
      double2 a = x0, b = make_double2(0.0, 0.0);
#pragma unroll
      for (int r = 1; r <= H; ++r) {
        const int m = r * k % R;
        const double c = Trig<R>::c[(m <= H ? m : R - m) - 1];
        const double sg = m <= H ? Trig<R>::s[m - 1] : -Trig<R>::s[R - m - 1];
        a.x += c * s[r - 1].x;
        a.y += c * s[r - 1].y;
        b.x += sg * d[r - 1].x;
        b.y += sg * d[r - 1].y;
      }
      // X_k = a - i b, X_{R-k} = a + i b
      v[k] = make_double2(a.x + b.y, a.y - b.x);
      v[R - k] = make_double2(a.x - b.y, a.y + b.x);
    }
  }
}

// A sequence in LDS: one entry of padding after every 8 (strides 1, 8 and 64
// without bank conflicts).  at(base, off), off a multiple of 8 known to the
// compiler: a constant distance from at(base), no address of its own.
struct Seq {
  double2* p;
  __device__ __forceinline__ double2& operator()(int i) const { return p[i + (i >> 3)]; }
  __device__ __forceinline__ double2& at(int base, int off) const {
    return p[base + (base >> 3) + off / 8 * 9];
  }
};

// One Stockham pass of radix R: butterfly b = q Ns + k takes the entries
// b + r n/R, times W^{k r}, W = e^{-2 pi i / (Ns R)}, and writes q Ns R + k + r Ns.
// T threads, n <= 8 T: a thread has at most ceil(8 / R) butterflies.  N = 8 T:
// n = N and Ns = NS, powers of two, so that every distance is a constant;
// N = 0: pass `p` of the plan, Ns the product of the radices before.
template <int R, int T, int N, int NS>
__device__ __forceinline__ void fft_pass(const Seq& at, int j, const DstPlan& P, int p) {
  constexpr int MB = (8 + R - 1) / R;
  const auto* tw = reinterpret_cast<const double2*>(P.tw);
  const int nb = N ? N / R : P.nb[p], Ns = N ? NS : P.ns[p], step = N ? N / R / NS : P.step[p];
  j = opaque(j);
  __builtin_assume(j >= 0 && j < T);
  double2 v[MB][R];
  int base[MB];
#pragma unroll
  for (int m = 0; m < MB; ++m) {
    const int b = j + T * m;
    const int q = N ? b / NS : (int)__umulhi(2u * (uint32_t)b, P.magic[p]), k = b - q * Ns;
    base[m] = N || b < nb ? q * Ns * R + k : -1;
    if (N || b < nb) {
      double2 w = make_double2(1.0, 0.0);
      if (Ns > 1) w = tw[k * step];
#pragma unroll
      for (int r = 0; r < R; ++r) v[m][r] = N ? at.at(b, r * nb) : at(b + r * nb);
      if (Ns > 1) {
        // W^{k r}: one table entry, its even powers by squares
        const double2 w2 = cmul(w, w);
        double2 po = w, pe = w2;
#pragma unroll
        for (int r = 1; r < R; r += 2) {
          v[m][r] = cmul(v[m][r], po);
          if (r + 1 < R) v[m][r + 1] = cmul(v[m][r + 1], pe);
          if (r + 2 < R) po = cmul(po, w2);
          if (r + 3 < R) pe = cmul(pe, w2);
        }
      }
      dft<R>(v[m]);
    }
  }
  seq_sync<T>();   // every thread has read the pass's inputs
#pragma unroll
  for (int m = 0; m < MB; ++m)
    if (N || base[m] >= 0) {
#pragma unroll
      for (int r = 0; r < R; ++r) {
        if constexpr (N == 0) at(base[m] + r * Ns) = v[m][r];
        else if constexpr (NS == 1) at.p[base[m] / 8 * 9 + r] = v[m][r];   // (R = 8)
        else at.at(base[m], r * NS) = v[m][r];
      }
    }
  seq_sync<T>();
}

template <int T, int N, int NS = 1>
__device__ __forceinline__ void fft(const Seq& at, int j, const DstPlan& P) {
  if constexpr (N > 0) {
    static_assert(N == 8 * T && N >= 64, "the first radix is 8");
    if constexpr (NS < N) {
      constexpr int R = N / NS >= 8 ? 8 : N / NS;
      fft_pass<R, T, N, NS>(at, j, P, 0);
      fft<T, N, NS * R>(at, j, P);
    }
  } else {
    for (int p = 0; p < P.np; ++p) {
      const int R = P.radix[p];
      if (R == 8) fft_pass<8, T, 0, 0>(at, j, P, p);
      else if (R == 4) fft_pass<4, T, 0, 0>(at, j, P, p);
      else if (R == 2) fft_pass<2, T, 0, 0>(at, j, P, p);
      else if (R == 3) fft_pass<3, T, 0, 0>(at, j, P, p);
      else if (R == 5) fft_pass<5, T, 0, 0>(at, j, P, p);
      else if (R == 7) fft_pass<7, T, 0, 0>(at, j, P, p);
      else if (R == 11) fft_pass<11, T, 0, 0>(at, j, P, p);
      else fft_pass<13, T, 0, 0>(at, j, P, p);
    }
  }
}

// The transforms of the pair from its spectrum: entry m (1 <= m < n) becomes
// (S^A_m, S^B_m).  wt: the wavefronts' totals of the pair.  Ends synchronised.
template <int T, int N>
__device__ __forceinline__ void split_scan(const Seq& at, int j, int n, double2* wt) {
  constexpr int EP = 4;                          // ceil(K1 / T) <= 4
  constexpr int JW = T < 64 ? T : 64;            // threads of a sequence per wavefront
  // (entry n / 2 of an even n belongs to no coefficient below n)
  const int K1 = N ? N / 2 : (n + 1) / 2, ep = N ? EP : (K1 + T - 1) / T;
  if (N) n = N;
  j = opaque(j);
  __builtin_assume(j >= 0 && j < T);
  double2 v[EP], im[EP];
#pragma unroll
  for (int e = 0; e < EP; ++e) {
    const int k = j * ep + e;
    v[e] = im[e] = make_double2(0.0, 0.0);
    if (N || (e < ep && k < K1)) {
      const double2 a = at(k), b = at(k == 0 ? 0 : n - k);
      const double h = k == 0 ? 0.25 : 0.5;   // Re Y_0 counts half
      v[e] = make_double2(h * (a.x + b.x), h * (a.y + b.y));
      im[e] = make_double2(0.5 * (a.y - b.y), 0.5 * (b.x - a.x));
    }
  }
#pragma unroll
  for (int e = 1; e < EP; ++e) v[e] = cadd(v[e], v[e - 1]);
  double2 x = v[EP - 1];
  const int jl = j % JW;
#pragma unroll
  for (int d = 1; d < JW; d <<= 1) {
    const double yx = __shfl_up(x.x, d, 64), yy = __shfl_up(x.y, d, 64);
    if (jl >= d) {
      x.x += yx;
      x.y += yy;
    }
  }
  double2 off = csub(x, v[EP - 1]);
  if constexpr (T > JW) {
    if (jl == JW - 1) wt[j / JW] = x;
    __syncthreads();   // (the spectrum is read, too)
    double2 c = make_double2(0.0, 0.0);
    for (int q = 0; q < j / JW; ++q) c = cadd(c, wt[q]);
    off = cadd(off, c);
  } else {
    seq_sync<T>();     // the spectrum is read
  }
#pragma unroll
  for (int e = 0; e < EP; ++e) {
    const int k = j * ep + e;
    if (N || (e < ep && k < K1)) {
      if (k >= 1) at(2 * k) = make_double2(-im[e].x, -im[e].y);
      if (N || 2 * k + 1 < n) at(2 * k + 1) = cadd(off, v[e]);
    }
  }
  seq_sync<T>();
}

template <int T>
struct RowShape {
  static constexpr int NT = T >= 128 ? T : 128;
  static constexpr int PR = NT / T;               // pairs of rows per workgroup
  static constexpr int NW = T > 64 ? T / 64 : 1;  // wavefronts per pair
  static constexpr int PITCH = 9 * T + 1;         // one entry of padding after every 8
};

// The folded pair into LDS: f(base, off) the pair's entry base + off of the
// transform (off constant); a thread takes entries jj and n - jj.
template <int T, int N, class Get>
__device__ __forceinline__ void fold_pair(const Seq& at, int j, int n, const double* sn,
                                          const Get& f) {
  if (N) n = N;
  j = opaque(j);
  __builtin_assume(j >= 0 && j < T);
  const int hi = 5 * T - 1 - j;   // N = 8 T: n - jj = hi + T (3 - i)
  double2 a[4], b[4];
  double s[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int jj = 1 + j + T * i;
    a[i] = b[i] = make_double2(0.0, 0.0);
    s[i] = 0.0;
    if (N || 2 * jj <= n) {
      s[i] = sn[jj];
      a[i] = f(1 + j, T * i);
      b[i] = N ? f(hi, T * (3 - i)) : f(n - jj, 0);
    }
  }
  if (j == 0) at(0) = make_double2(0.0, 0.0);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int jj = 1 + j + T * i;
    if (N || 2 * jj <= n) {
      const double2 u = cadd(a[i], b[i]), d = csub(a[i], b[i]);
      at.at(1 + j, T * i) = make_double2(s[i] * u.x + 0.5 * d.x, s[i] * u.y + 0.5 * d.y);
      (N ? at.at(hi, T * (3 - i)) : at(n - jj)) =
          make_double2(s[i] * u.x - 0.5 * d.x, s[i] * u.y - 0.5 * d.y);
    }
  }
}

// Rows in pairs, T threads per pair, n <= 8 T.
template <int T>
__global__ __launch_bounds__(RowShape<T>::NT, 4) void k_dst_any_rows(
    DstPlan P, const double* __restrict__ in, double* __restrict__ out, int64_t rows, int64_t ldi,
    int64_t ldo, double scale) {
  using S = RowShape<T>;
  __shared__ double2 buf[S::PR][S::PITCH];
  __shared__ double2 wt[S::PR][S::NW];
  const int t = threadIdx.x, pr = t / T, j = t % T, n = P.n;
  const Seq at{buf[pr]};
  const int64_t r = 2 * ((int64_t)blockIdx.x * S::PR + pr);
  const bool la = r < rows, lb = r + 1 < rows;
  {
    const double* fa = in + (la ? r : 0) * ldi - 1;
    const double* fb = in + (lb ? r + 1 : 0) * ldi - 1;
    fold_pair<T, 0>(at, j, n, P.sn, [&](int i, int o) {
      return make_double2(la ? fa[i + o] : 0.0, lb ? fb[i + o] : 0.0);
    });
  }
  seq_sync<T>();
  fft<T, 0>(at, j, P);
  split_scan<T, 0>(at, j, n, wt[pr]);
  double* oa = out + (la ? r : 0) * ldo - 1;
  double* ob = out + (lb ? r + 1 : 0) * ldo - 1;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int m = 1 + j + T * i;
    if (m < n) {
      const double2 v = at.at(1 + j, T * i);
      if (la) oa[m] = scale * v.x;
      if (lb) ob[m] = scale * v.y;
    }
  }
}

// Sixteen adjacent columns (eight pairs, 128 bytes of every row) per
// workgroup, T threads per pair.  HBM is accessed with the pairs side by side
// (every eight lanes 128 contiguous bytes of a row), the transforms run with a
// pair's threads side by side: T <= 64 then needs no barrier between the two
// accesses.  With FACTOR (two transforms and the factor between them) the
// vector ALUs were the bound, half of their work the addresses: 3130
// instructions per wavefront at n = 512, 87 % of the kernel's cycles.  With
// N = n = 8 T, where every distance is a constant, 1380: 1012 -> 733 us for the
// z axis of 511^3 (the plain transform of y 490 -> 445); eight columns per
// workgroup, or the columns in chunks that stay in the last cache, gave nothing more.
constexpr int kPairs = 8;
template <int T, bool FACTOR, int N>
__global__ __launch_bounds__(kPairs * T, 4) void k_dst_columns(DstPlan P, DstColumns A) {
  __shared__ double2 buf[kPairs][9 * T + 1];
  __shared__ double2 wt[kPairs][T > 64 ? T / 64 : 1];
  const int t = threadIdx.x, n = N ? N : P.n;
  const uint32_t groups = (uint32_t)((A.M + 2 * kPairs - 1) / (2 * kPairs));
  const int64_t bt = blockIdx.x / groups;
  const int64_t c0 = (int64_t)(blockIdx.x - (uint32_t)bt * groups) * (2 * kPairs);
  const int hp = t % kPairs, hj = t / kPairs;   // pair and thread in HBM's order
  const int64_t c = c0 + 2 * hp;
  const bool la = c < A.M, lb = c + 1 < A.M;
  const int64_t base = bt * A.ldb + (la ? c : 0) - A.ld;
  {
    const double* f = A.in + base;
    fold_pair<T, N>(Seq{buf[hp]}, hj, n, P.sn, [&](int i, int o) {
      double2 v = make_double2(0.0, 0.0);
      if (la) v = *reinterpret_cast<const double2*>(f + (i * A.ld + o * A.ld));
      if (!lb) v.y = 0.0;
      return v;
    });
  }
  __syncthreads();
  {
    const int pr = t / T, j = t % T;
    const Seq at{buf[pr]};
    fft<T, N>(at, j, P);
    split_scan<T, N>(at, j, n, wt[pr]);
    if constexpr (FACTOR) {
      const int64_t ca = c0 + 2 * pr < A.M ? c0 + 2 * pr : 0, cb = ca + 1 < A.M ? ca + 1 : ca;
      const double ya = A.ry[ca * A.ldy + bt], yb = A.ry[cb * A.ldy + bt];
      const double da = A.ly[bt] + A.mu[ca], db = A.ly[bt] + A.mu[cb];
      const double* rza = A.rz + ca * A.ldz - 1;
      const double* rzb = A.rz + cb * A.ldz - 1;
      const double* lz = A.lz - 1;
      // (a thread reads and rewrites its own entries jj and n - jj only)
      fold_pair<T, N>(at, j, n, P.sn, [&](int i, int o) {
        double2 v = at.at(i, o);
        v.x *= A.norm * (1.0 - ya * rza[i + o]) / (lz[i + o] + da);
        v.y *= A.norm * (1.0 - yb * rzb[i + o]) / (lz[i + o] + db);
        return v;
      });
      seq_sync<T>();
      fft<T, N>(at, j, P);
      split_scan<T, N>(at, j, n, wt[pr]);
    }
  }
  if constexpr (T <= 64) __syncthreads();
  const Seq at{buf[hp]};
  double* o = A.out + base + (1 + hj) * A.ld;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const int m = 1 + hj + T * i;
    if (m < n && la) {
      const double2 v = at.at(1 + hj, T * i);
      if (lb) *reinterpret_cast<double2*>(o + T * i * A.ld) = v;
      else o[T * i * A.ld] = v.x;
    }
  }
}

__global__ __launch_bounds__(256) void k_adi_factors(const double* __restrict__ w,
                                                     const int* __restrict__ count, int jmax,
                                                     const double* __restrict__ lam,
                                                     const double* __restrict__ mu, int64_t L,
                                                     int64_t M, bool modes_last,
                                                     double* __restrict__ out) {
  const int64_t id = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (id >= L * M) return;
  const int64_t c = id / L, l = id - c * L;
  const double x = lam[l] + 0.5 * mu[c];
  double r = 1.0;
  for (int j = 0; j < count[c]; ++j) {
    const double wj = w[c * jmax + j];
    r *= (wj - x) / (wj + x);
  }
  out[modes_last ? l * M + c : id] = r;
}

// Threads per pair: the least power of two with n <= 8 T, at least 8.
int threads_for(int64_t n) {
  int t = 8;
  while (8 * (int64_t)t < n) t *= 2;
  return t;
}

// Rows: two or four times as many where that still is at most twelve
// wavefronts per compute unit.  A few rows are bound by a thread's chain of
// LDS passes (one pass over 99 x 2000 points 10.5 -> 8.9 us, 499 x 500 11.6 ->
// 9.4, 999 x 700 15.0 -> 13.1); with more wavefronts the lanes without a
// butterfly cost more than the shorter chain gives (999 x 3000 22.9 and 22.8
// us, 999 x 6000 32.9 -> 35.6, 239 x 20000 28.9 -> 30.7).
int row_threads(int64_t n, int64_t pairs) {
  int t = threads_for(n);
  const int most = std::min(t <= 32 ? 4 * t : 2 * t, 1024);
  while (t < most && pairs * 2 * t <= (int64_t)12 * 64 * device_cus()) t *= 2;
  return t;
}

}  // namespace

namespace {
bool small_factors(int64_t n) {
  for (int f : {2, 3, 5, 7, 11, 13})
    while (n % f == 0) n /= f;
  return n == 1;
}
}  // namespace

bool dst_any_supported(int64_t n, int64_t max_n) {
  return n >= 2 && n <= max_n && (n <= kDstDenseMax || small_factors(n));
}

hipError_t dst_plan_make(int64_t n, DstPlan& p, double** mem) {
  *mem = nullptr;
  p = DstPlan{};
  p.n = (int)n;
  if (!small_factors(n)) {
    if (n > kDstDenseMax) return hipErrorInvalidValue;
    std::vector<double> tab;
    dst_dense_table(n, tab);
    hipError_t e = hipMalloc(reinterpret_cast<void**>(mem), tab.size() * sizeof(double));
    if (e != hipSuccess) {
      *mem = nullptr;
      return e;
    }
    p.tw = *mem;
    return hipMemcpy(*mem, tab.data(), tab.size() * sizeof(double), hipMemcpyHostToDevice);
  }
  // the large radices first: their first pass has no twiddles
  int64_t rest = n, ns = 1;
  for (int f : {8, 4, 2, 13, 11, 7, 5, 3})
    while (rest % f == 0) {
      if (p.np == kDstPasses) return hipErrorInvalidValue;
      p.radix[p.np] = f;
      p.magic[p.np] = (uint32_t)(((uint64_t)1 << 31) / (uint64_t)ns) + 1u;
      p.ns[p.np] = (int)ns;
      p.nb[p.np] = (int)(n / f);
      p.step[p.np] = (int)(n / f / ns);
      ++p.np;
      ns *= f;
      rest /= f;
    }
  if (rest != 1) return hipErrorInvalidValue;
  const long double pi = 3.141592653589793238462643383279502884L;
  std::vector<double> tab((size_t)(3 * n + 1));
  const size_t sn0 = (size_t)(2 * n);
  for (int64_t q = 0; q < n; ++q) {
    const long double a = -2.0L * pi * (long double)q / (long double)n;
    tab[(size_t)(2 * q)] = (double)std::cos(a);
    tab[(size_t)(2 * q + 1)] = (double)std::sin(a);
    tab[sn0 + (size_t)q] = (double)std::sin(pi * (long double)q / (long double)n);
  }
  hipError_t e = hipMalloc(reinterpret_cast<void**>(mem), tab.size() * sizeof(double));
  if (e != hipSuccess) {
    *mem = nullptr;
    return e;
  }
  p.tw = *mem;
  p.sn = *mem + sn0;
  return hipMemcpy(*mem, tab.data(), tab.size() * sizeof(double), hipMemcpyHostToDevice);
}

hipError_t launch_dst_any_rows(const DstPlan& p, const double* in, double* out, int64_t rows,
                               int64_t ldi, int64_t ldo, double scale, hipStream_t st) {
  if (p.np == 0) return launch_dst_dense_rows(p, in, out, rows, ldi, ldo, scale, st);
  switch (row_threads(p.n, (rows + 1) / 2)) {
#define TDT_ROWS(T)                                                                         \
  case T: {                                                                                 \
    const int64_t g = ((rows + 1) / 2 + RowShape<T>::PR - 1) / RowShape<T>::PR;             \
    if (g > 0x7fffffff) return hipErrorInvalidValue;                                        \
    hipLaunchKernelGGL(k_dst_any_rows<T>, dim3((unsigned)g), dim3(RowShape<T>::NT), 0, st,  \
                       p, in, out, rows, ldi, ldo, scale);                                  \
    break;                                                                                  \
  }
    TDT_ROWS(8) TDT_ROWS(16) TDT_ROWS(32) TDT_ROWS(64)
    TDT_ROWS(128) TDT_ROWS(256) TDT_ROWS(512) TDT_ROWS(1024)
#undef TDT_ROWS
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_dst_columns(const DstPlan& p, const DstColumns& a, hipStream_t st) {
  if (p.np == 0) return launch_dst_dense_columns(p, a, st);
  if (a.M < 1 || a.nb < 1 || (a.ld & 1) || (a.ldb & 1)) return hipErrorInvalidValue;
  const int64_t g = (a.M + 2 * kPairs - 1) / (2 * kPairs) * a.nb;
  if (g > 0x7fffffff) return hipErrorInvalidValue;
  const dim3 grid((unsigned)g);
  switch (threads_for(p.n)) {
#define TDT_COL(T, F, N)                                                                  \
  hipLaunchKernelGGL((k_dst_columns<T, F, N>), grid, dim3(kPairs * T), 0, st, p, a)
#define TDT_COLS(T)                                                                       \
  case T:                                                                                 \
    if (p.n == 8 * T) {                                                                   \
      if (a.ry) TDT_COL(T, true, 8 * T);                                                  \
      else TDT_COL(T, false, 8 * T);                                                      \
    } else {                                                                              \
      if (a.ry) TDT_COL(T, true, 0);                                                      \
      else TDT_COL(T, false, 0);                                                          \
    }                                                                                     \
    break;
    TDT_COLS(8) TDT_COLS(16) TDT_COLS(32) TDT_COLS(64) TDT_COLS(128)
#undef TDT_COLS
#undef TDT_COL
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_adi_factors(const double* w, const int* count, int jmax, const double* lam,
                              const double* mu, int64_t L, int64_t M, bool modes_last,
                              double* out, hipStream_t st) {
  const int64_t g = (L * M + 255) / 256;
  if (g < 1 || g > 0x7fffffff) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_adi_factors, dim3((unsigned)g), dim3(256), 0, st, w, count, jmax, lam, mu,
                     L, M, modes_last, out);
  return hipGetLastError();
}

}  // namespace tdt
