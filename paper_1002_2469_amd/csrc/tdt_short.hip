// tdt_short.hip -- systems of a few blocks: several of them per workgroup.
//
// A system of n rows fills nb = ceil(n / 16) lanes of 16 rows.  A tile kernel
// gives it a whole workgroup, so that most lanes of a short system idle (16 of
// 512 for the 65025 lines of 255 rows of a 255^3 grid, which took 911 us for
// 265 MB in double; here 51 us, 5.2 TB/s).
// Here the lanes of a workgroup are dealt out to consecutive systems, nb
// each, and the steps of the method run on all of them at once: the local
// sweeps as in a tile, the affine recurrences of eq. (15) as the same scans,
// cut where a system begins or ends (a system's first block takes nothing
// from the left and its last nothing from the right, so a value of another
// system never enters, whatever it is), and the correction.  The corner rows
// of a quasi-Toeplitz system (eq. (21)) are the one-row segments at the two
// ends of its own chain of blocks: no first pass and no interface launch
// (double and refined plans; in refined ones that chain runs in double before
// the float solves, as the interface pass does for tiles).
//
// The rows of the workgroup's systems are one contiguous run, loaded and
// stored coalesced; LDS holds the run with 16 bytes of padding after every
// 16 rows, so that lanes 16 rows apart fall on different banks.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tdt_device.h"
#include "tdt_internal.h"

namespace tdt {
namespace {

constexpr int kB = kShortB;

template <typename Tio>
struct ShortArgs {
  const Tio* __restrict__ F;
  Tio* __restrict__ X;
  const Tio* __restrict__ Xfwd;       // adjoint: forward solution
  const SysDesc* __restrict__ sys;
  const double* __restrict__ vec64;
  const float* __restrict__ vec32;
  const double* __restrict__ tab64;   // [ncidx][kTabN tabnt]: beta_{m-1}, then
  const float* __restrict__ tab32;    //   1/(1 - phi_f beta_{m-1}) of tabnt positions each
  const double* __restrict__ qtab64;  // quasi-Toeplitz: [ncidx][2 qnt + kQTabN], the chain with
                                      //   its corner rows
  const int* __restrict__ items;      // varlen: one system per workgroup; null for a series
  int64_t nitems;                     // workgroups' worth of systems
  int64_t M;                          // series: right-hand sides
  int tabnt, qnt;
  int G;                              // systems per workgroup
  double* __restrict__ gpart;
  int* __restrict__ iters;
  int max_iter;
  double refine_tol;
};

// What a lane knows of its block: its position in its system (blk blocks
// before it, rb after it), its rows, and the block's coefficients.
template <typename Tc>
struct Block {
  int blk, rb, len;
  bool first, last;
  Tc pf, pl, cf, bp, iD;
};

// The scans of eq. (15) of tile_solve, cut at the systems' ends: a map or a
// value enters a lane only from lanes of its own system.  On return A, g (C,
// h) compose the lane's system inside the wavefront, and cin (ein) is the
// value entering it there from the wavefronts before (after).
template <int NW, typename Tc>
__device__ __forceinline__ void cut_scan_fwd(const Block<Tc>& b, Tc& A, Tc& g, Tc (*fw)[2],
                                             Tc& cin) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#define TDT_STEP(D)                                        \
  {                                                        \
    Tc As = dpp<kDppRowShr + D>(Tc(1), A);                 \
    Tc gs = dpp<kDppRowShr + D>(Tc(0), g);                 \
    As = b.blk >= D ? As : Tc(1);                          \
    gs = b.blk >= D ? gs : Tc(0);                          \
    g = A * gs + g;                                        \
    A = A * As;                                            \
  }
  TDT_STEP(1) TDT_STEP(2) TDT_STEP(4) TDT_STEP(8)
#undef TDT_STEP
  const int row = lane >> 4;
  const Tc A0 = readlane(A, 15), g0 = readlane(g, 15);
  const Tc A1 = readlane(A, 31), g1 = readlane(g, 31);
  const Tc A2 = readlane(A, 47), g2 = readlane(g, 47);
  const bool x1 = __builtin_amdgcn_readlane(b.blk, 31) >= 16;
  const bool x2 = __builtin_amdgcn_readlane(b.blk, 47) >= 16;
  const Tc cA1 = A0, cg1 = g0;
  const Tc cA2 = x1 ? A1 * cA1 : A1, cg2 = x1 ? A1 * cg1 + g1 : g1;
  const Tc cA3 = x2 ? A2 * cA2 : A2, cg3 = x2 ? A2 * cg2 + g2 : g2;
  Tc cA = row == 1 ? cA1 : (row == 2 ? cA2 : cA3);
  Tc cg = row == 1 ? cg1 : (row == 2 ? cg2 : cg3);
  const bool in = row > 0 && b.blk > (lane & 15);
  cA = in ? cA : Tc(1);
  cg = in ? cg : Tc(0);
  g = A * cg + g;
  A = A * cA;
  cin = Tc(0);
  if constexpr (NW > 1) {
    // the wavefronts' totals; ext: the system at the wavefront's last lane
    // began before the wavefront
    __shared__ int ext[NW];
    if (lane == 63) {
      fw[w][0] = A;
      fw[w][1] = g;
      ext[w] = b.blk > 63;
    }
    __syncthreads();
    for (int k = 0; k < w; ++k) cin = ext[k] ? fw[k][0] * cin + fw[k][1] : fw[k][1];
    cin = b.blk > lane ? cin : Tc(0);
  }
}

template <int NW, typename Tc>
__device__ __forceinline__ void cut_scan_bwd(const Block<Tc>& b, Tc& C, Tc& h, Tc (*bw)[2],
                                             Tc& ein) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#define TDT_STEP(D)                                        \
  {                                                        \
    Tc Cs = dpp<kDppRowShl + D>(Tc(1), C);                 \
    Tc hs = dpp<kDppRowShl + D>(Tc(0), h);                 \
    Cs = b.rb >= D ? Cs : Tc(1);                           \
    hs = b.rb >= D ? hs : Tc(0);                           \
    h = C * hs + h;                                        \
    C = C * Cs;                                            \
  }
  TDT_STEP(1) TDT_STEP(2) TDT_STEP(4) TDT_STEP(8)
#undef TDT_STEP
  const int row = lane >> 4;
  const Tc C1 = readlane(C, 16), h1 = readlane(h, 16);
  const Tc C2 = readlane(C, 32), h2 = readlane(h, 32);
  const Tc C3 = readlane(C, 48), h3 = readlane(h, 48);
  const bool x1 = __builtin_amdgcn_readlane(b.rb, 16) >= 16;
  const bool x2 = __builtin_amdgcn_readlane(b.rb, 32) >= 16;
  const Tc eC2 = C3, eh2 = h3;
  const Tc eC1 = x2 ? C2 * eC2 : C2, eh1 = x2 ? C2 * eh2 + h2 : h2;
  const Tc eC0 = x1 ? C1 * eC1 : C1, eh0 = x1 ? C1 * eh1 + h1 : h1;
  Tc eC = row == 2 ? eC2 : (row == 1 ? eC1 : eC0);
  Tc eh = row == 2 ? eh2 : (row == 1 ? eh1 : eh0);
  const bool in = row < 3 && b.rb > 15 - (lane & 15);
  eC = in ? eC : Tc(1);
  eh = in ? eh : Tc(0);
  h = C * eh + h;
  C = C * eC;
  ein = Tc(0);
  if constexpr (NW > 1) {
    __shared__ int ext[NW];
    if (lane == 0) {
      bw[w][0] = C;
      bw[w][1] = h;
      ext[w] = b.rb > 63;
    }
    __syncthreads();
    for (int k = NW - 1; k > w; --k) ein = ext[k] ? bw[k][0] * ein + bw[k][1] : bw[k][1];
    ein = b.rb > 63 - lane ? ein : Tc(0);
  }
}

// Solves the workgroup's systems for the right-hand side rows in q (0 past
// len).  What lies outside a system, in its first and last lane:
//   kOpen   nothing
//   kGiven  the values fl and fr
//   kChain  its corner rows (quasi-Toeplitz), fl and fr their right-hand
//           sides; out: the corner unknowns.  kEnds: these alone, q not solved.
enum { kOpen, kGiven, kChain, kEnds };
template <int NW, typename Tc, int OUT>
__device__ __forceinline__ void short_solve(Tc (&q)[kB], const Block<Tc>& b,
                                            const Consts<Tc>& K, const SysDesc& S, Tc qs5,
                                            Tc& fl, Tc& fr, Tc (*fw)[2], Tc (*bw)[2]) {
  constexpr bool CHAIN = OUT == kChain || OUT == kEnds;
  const int lane = threadIdx.x & 63;
  const bool wave_tail = __ballot(b.len > 0 && b.len < kB) != 0;
  const cptr<Tc> iu = fresh(K.iu), aiu = fresh(K.aiu);
#pragma unroll
  for (int i = 0; i < kB; ++i) q[i] *= iu[i];
  if (!wave_tail) {
#pragma unroll
    for (int i = 1; i < kB; ++i) q[i] -= aiu[i] * q[i - 1];
  } else {
#pragma unroll
    for (int i = 1; i < kB; ++i) {
      const Tc d = q[i] - aiu[i] * q[i - 1];
      q[i] = i < b.len ? d : Tc(0);
    }
  }
  const cptr<Tc> cpb = fresh(K.cp);
#pragma unroll
  for (int i = kB - 2; i >= 0; --i) q[i] -= cpb[i] * q[i + 1];
  const Tc yf = q[0];
  Tc yl = q[kB - 1];
  if (CHAIN && wave_tail) {
#pragma unroll
    for (int i = 0; i + 1 < kB; ++i)
      if (i == b.len - 1) yl = q[i];
  }
  // the interface recurrences (see tile_solve), each system's own
  const Tc alpha_in = OUT != kOpen && b.first ? (CHAIN ? fl * (Tc)S.qc[0] : fl) : Tc(0);
  const Tc A0 = b.pl * b.iD;
  Tc A = A0;
  Tc g = yl + A0 * b.bp * yf;
  if (OUT != kOpen && b.first) g += A0 * alpha_in;
  Tc cin, ein;
  cut_scan_fwd<NW>(b, A, g, fw, cin);
  const Tc alpha = A * cin + g;
  Tc alpha_prev = __shfl_up(alpha, 1, 64);
  if (lane == 0) alpha_prev = cin;
  if (b.first) alpha_prev = alpha_in;
  // the unknown right of the system: its last corner row, a value, or nothing
  const Tc u_right = OUT != kOpen && b.last
                         ? (CHAIN ? (fr * (Tc)S.qc[2] + (Tc)S.qc[3] * alpha) * qs5 : fr)
                         : Tc(0);
  const Tc C0 = b.cf * b.iD;
  Tc C = C0;
  Tc h = (yf + b.pf * alpha_prev) * b.iD;
  if (OUT != kOpen && b.last) h += C0 * u_right;
  cut_scan_bwd<NW>(b, C, h, bw, ein);
  const Tc u = C * ein + h;
  Tc u_next = __shfl_down(u, 1, 64);
  if (lane == 63) u_next = ein;
  const Tc xl = alpha_prev + b.bp * u;            // last unknown of the previous block
  const Tc xr = b.last ? u_right : u_next;        // first unknown of the next block
  if (CHAIN) {
    fl = xl;
    fr = xr;
  }
  if constexpr (OUT == kEnds) return;
  if (b.len == kB) {
    const cptr<Tc> phi = fresh(K.phi), chi = fresh(K.chi);
#pragma unroll
    for (int i = 0; i < kB; ++i) q[i] += xl * phi[i] + xr * chi[i];
  } else if (b.len > 0) {
    // last block: re-swept with its outside values folded into its first and
    // last right-hand side rows
    Tc delta = -K.a * xl * K.iu[0];
#pragma unroll
    for (int i = 0; i < kB; ++i) {
      const Tc ynext = i + 1 < kB ? q[i + 1] : Tc(0);
      Tc dp = q[i] + K.cp[i] * ynext + delta;
      if (OUT != kOpen && i == b.len - 1) dp -= K.cp[i] * xr;
      q[i] = i < b.len ? dp : Tc(0);
      if (i + 1 < kB) delta = -K.aiu[i + 1] * delta;
    }
#pragma unroll
    for (int i = kB - 2; i >= 0; --i) q[i] -= K.cp[i] * q[i + 1];
  }
}

// The largest of v (non-negative) over the lanes of each system; every lane
// of the system receives it.  Two barriers.
__device__ __forceinline__ float system_max(float v, int s, int* smax) {
  smax[threadIdx.x] = 0;
  __syncthreads();
  atomicMax(&smax[s], __float_as_int(fmaxf(v, 0.0f)));
  __syncthreads();
  return __int_as_float(smax[s]);
}

// Bound by HBM like the tile kernels (16 bytes per unknown, 24 in the
// adjoint); one run per workgroup, latency hidden by the other workgroups.
// Series of 2^24 unknowns in double, forward, before and now: 100 rows 2297
// and 51 us, 1000 rows 258 and 51, 2000 rows 131 and 52, 3000 rows 97 and 56
// (a copy of these bytes takes 52); the adjoint with its reduction 255 rows
// 1858 and 114 us, 2000 rows 256 and 110.  The adjoint requests four rows of
// the forward solution ahead of the stores: eight spilled.
template <int NT, typename Tio, typename Tc, bool REFINE, bool BWD, bool QUASI>
__global__ __launch_bounds__(NT, kMinWavesPerSimd) void k_short(ShortArgs<Tio> A) {
  constexpr int NW = NT / 64;
  constexpr int PAD = 16 / (int)sizeof(Tio);
  constexpr int ROWS = NT * kB;
  using SH = Shape<kB, NT, kMinWavesPerSimd>;
  // (a block's 16 rows are read whole: up to 16 past the run's last)
  __shared__ __align__(16) Tio lds[(ROWS + kB) / kB * (kB + PAD)];
  __shared__ Tc fw[NW][2], bw[NW][2];
  __shared__ double red[NW][kGradN];
  __shared__ int smax[REFINE ? NT : 1];
  __shared__ double edge[REFINE ? NW : 1][2];
  // refined quasi-Toeplitz systems: the double chain's exchange
  __shared__ double fwd[REFINE && QUASI ? NW : 1][2], bwd[REFINE && QUASI ? NW : 1][2];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  int it_max = 0;
  float est_max = 0.0f;
  for (int64_t k = blockIdx.x; k < A.nitems; k += gridDim.x) {
    const int sid = A.items ? as_const(A.items)[k] : 0;
    const SysDesc S = load_sys(A.sys, sid);
    const int n = (int)S.n, N = QUASI ? n + 2 : n;
    const int nb = (n + kB - 1) / kB;
    const int64_t m0 = A.items ? 0 : k * A.G;
    const int G = A.items ? 1 : (int)(A.M - m0 < A.G ? A.M - m0 : A.G);
    const int64_t base = S.off - (QUASI ? 1 : 0) + m0 * N;
    const int rows = G * N;
    const __amdgpu_buffer_rsrc_t src = make_rsrc(A.F + base, (int64_t)rows * sizeof(Tio));
    const int vs = opaque(tid * (int)sizeof(Tio));
    Tio v[kB];
#pragma unroll
    for (int j = 0; j < kB; ++j) v[j] = buf_load<Tio>(src, vs + j * NT * (int)sizeof(Tio));
    // this lane's block: system sl of the run, block blk of it
    const int sl = A.items ? tid / nb : (int)(((uint32_t)tid * ((1u << 20) / (uint32_t)nb + 1u)) >> 20);
    Block<Tc> b;
    b.blk = tid - sl * nb;
    b.rb = nb - 1 - b.blk;
    const bool live = sl < G;
    b.first = b.blk == 0;
    b.last = b.rb == 0;
    b.len = live ? (n - b.blk * kB < kB ? n - b.blk * kB : kB) : 0;
    const Consts<Tc> K = make_consts<SH, Tc>(S, A.vec64, A.vec32);
    const double* qt = nullptr;
    double qs5 = 0.0;
    if constexpr (QUASI) {
      qt = A.qtab64 + (int64_t)S.cidx * (kTabN * A.qnt + kQTabN);
      qs5 = as_const(qt)[kTabN * A.qnt + kQTabClose];
    }
    if constexpr (QUASI && !REFINE) {
      b.bp = qt[b.blk];
      b.iD = qt[A.qnt + b.blk];
    } else {
      const Tc* tb;
      if constexpr (sizeof(Tc) == 8) tb = A.tab64 + (int64_t)S.cidx * kTabN * A.tabnt;
      else tb = A.tab32 + (int64_t)S.cidx * kTabN * A.tabnt;
      const int ti = S.tfix > 0 && b.blk > S.tfix ? S.tfix : b.blk;
      b.bp = tb[ti];
      b.iD = tb[A.tabnt + ti];
    }
    b.pf = K.pf;
    b.pl = K.pl;
    b.cf = K.cf;
    if (b.last && n % kB != 0) {
      b.pf = K.tail_pf;
      b.pl = K.tail_pl;
      b.cf = K.tail_cf;
      b.iD = Tc(1) / (Tc(1) - b.pf * b.bp);
    }
    __syncthreads();   // the previous run is done with LDS
    {
      Tio* lw = lds + tid + (tid / kB) * PAD;
#pragma unroll
      for (int j = 0; j < kB; ++j) lw[j * (NT / kB) * (kB + PAD)] = v[j];
    }
    __syncthreads();
    // the lane's rows e0 .. e0 + 15 of the run; past row wrap the address
    // skips one more stretch of padding
    const int e0 = live ? sl * N + (QUASI ? 1 : 0) + b.blk * kB : 0;
    Tio* p0 = lds + e0 + (e0 / kB) * PAD;
    const int wrap = kB - (e0 % kB);
    auto at = [&](int i) -> Tio& { return p0[i + (i >= wrap ? PAD : 0)]; };
    auto flat = [&](int e) -> Tio& { return lds[e + (e / kB) * PAD]; };
    const int ecl = live ? sl * N : 0, ecr = live ? sl * N + N - 1 : 0;   // corner rows
    Tc fl = Tc(0), fr = Tc(0);
    constexpr int OUT = !QUASI ? kOpen : (REFINE ? kGiven : kChain);
    if constexpr (!REFINE) {
      Tc q[kB];
#pragma unroll
      for (int i = 0; i < kB; ++i) {
        const Tc f = (Tc)at(i);
        q[i] = i < b.len ? f : Tc(0);
      }
      if (QUASI) {
        if (b.first) fl = (Tc)flat(ecl);
        if (b.last) fr = (Tc)flat(ecr);
      }
      short_solve<NW, Tc, OUT>(q, b, K, S, (Tc)qs5, fl, fr, fw, bw);
#pragma unroll
      for (int i = 0; i < kB; ++i)
        if (i < b.len) at(i) = (Tio)q[i];
    } else {
      // iterative refinement as in the tile kernels, each system by its own
      // stopping test (a system that has met it keeps its iterate); the corner
      // unknowns come from the double chain first and stay.  (Refined with the
      // inner rows instead, by one float chain, they were off by 2e-15 to
      // 2e-14 of the largest unknown where the double chain leaves 1e-16; 65793
      // systems of 255 rows 82 and 88 us, the adjoint 168 and 166.)
      const double a = S.a, bb = S.b, c = S.c;
      double x[kB], xcl = 0.0, xcr = 0.0;
      float vloc = 0.0f;
      if constexpr (QUASI) {
        const Consts<double> K64 = make_consts<SH, double>(S, A.vec64, A.vec32);
        Block<double> d;
        d.blk = b.blk;
        d.rb = b.rb;
        d.len = b.len;
        d.first = b.first;
        d.last = b.last;
        d.bp = qt[b.blk];
        d.iD = qt[A.qnt + b.blk];
        d.pf = K64.pf;
        d.pl = K64.pl;
        d.cf = K64.cf;
        if (b.last && n % kB != 0) {
          d.pf = K64.tail_pf;
          d.pl = K64.tail_pl;
          d.cf = K64.tail_cf;
        }
        double q[kB];
#pragma unroll
        for (int i = 0; i < kB; ++i) {
          const double f = (double)at(i);
          q[i] = i < b.len ? f : 0.0;
        }
        if (b.first) xcl = (double)flat(ecl);
        if (b.last) xcr = (double)flat(ecr);
        short_solve<NW, double, kEnds>(q, d, K64, S, qs5, xcl, xcr, fwd, bwd);
        fl = (Tc)xcl;
        fr = (Tc)xcr;
      }
      {
        Tc q[kB];
#pragma unroll
        for (int i = 0; i < kB; ++i) {
          const Tc f = (Tc)at(i);
          q[i] = i < b.len ? f : Tc(0);
        }
        short_solve<NW, Tc, OUT>(q, b, K, S, Tc(0), fl, fr, fw, bw);
#pragma unroll
        for (int i = 0; i < kB; ++i) {
          x[i] = (double)q[i];
          vloc = fmaxf(vloc, fabsf((float)q[i]));
        }
        fl = fr = Tc(0);   // the corrections have nothing outside
      }
      const float xmax = system_max(vloc, sl, smax);
      float dprev = xmax, est = 1.0f;   // est: remaining relative error (1: no update ran)
      bool done = !live;
      int it = 1, my_it = 1;
      while (it < A.max_iter) {
        double xm = __shfl_up(x[kB - 1], 1, 64);
        double xp = __shfl_down(x[0], 1, 64);
        if constexpr (NW > 1) {
          if (lane == 0) edge[w][0] = x[0];
          if (lane == 63) edge[w][1] = x[kB - 1];
          __syncthreads();
          if (lane == 0 && w > 0) xm = edge[w - 1][1];
          if (lane == 63 && w + 1 < NW) xp = edge[w + 1][0];
        }
        if (b.first) xm = xcl;
        if (b.last) xp = xcr;
        Tc q[kB];
#pragma unroll
        for (int i = 0; i < kB; ++i) {
          const double left = i == 0 ? xm : x[i - 1];
          double right = i + 1 < kB ? x[i + 1] : xp;
          if (QUASI && i == b.len - 1) right = xp;
          double r = fma(-bb, x[i], (double)at(i));
          r = fma(-a, left, r);
          r = fma(-c, right, r);
          q[i] = i < b.len ? (Tc)r : Tc(0);
        }
        short_solve<NW, Tc, OUT>(q, b, K, S, Tc(0), fl, fr, fw, bw);
        vloc = 0.0f;
        if (!done) {
#pragma unroll
          for (int i = 0; i < kB; ++i) {
            x[i] += (double)q[i];
            vloc = fmaxf(vloc, fabsf((float)q[i]));
          }
        }
        ++it;
        const float dmax = system_max(vloc, sl, smax);
        if (!done) {
          const float rho = dmax / dprev;
          dprev = dmax;
          my_it = it;
          est = dmax == 0.0f ? 0.0f
                             : (xmax > 0.0f ? (rho > 0.9f ? dmax : dmax * rho) / xmax : 1.0f);
          done = dmax == 0.0f || (double)dmax * rho <= A.refine_tol * xmax || rho > 0.9f;
        }
        if (__syncthreads_and(done)) break;
      }
      if (live) {
        it_max = my_it > it_max ? my_it : it_max;
        est_max = fmaxf(est_max, est);
      }
#pragma unroll
      for (int i = 0; i < kB; ++i)
        if (i < b.len) at(i) = (Tio)x[i];
      if (QUASI && live && b.first) flat(ecl) = (Tio)xcl;
      if (QUASI && live && b.last) flat(ecr) = (Tio)xcr;
    }
    if (!REFINE && QUASI && live) {
      if (b.first) flat(ecl) = (Tio)fl;
      if (b.last) flat(ecr) = (Tio)fr;
    }
    __syncthreads();
    // the run, coalesced: store j of lane tid writes row j NT + tid - mis, so
    // that every wavefront covers whole 128-byte lines where the run starts
    // inside one (as store_tile)
    const __amdgpu_buffer_rsrc_t xf =
        make_rsrc(BWD ? A.Xfwd + base : A.X + base, BWD ? (int64_t)rows * sizeof(Tio) : 0);
    Tio xpre[BWD ? 4 : 1];
    if constexpr (BWD) {
#pragma unroll
      for (int j = 0; j < 4; ++j) xpre[j] = buf_load<Tio>(xf, vs + j * NT * (int)sizeof(Tio));
    }
    constexpr int kLine = 128 / (int)sizeof(Tio);
    const int mis = __builtin_amdgcn_readfirstlane(
        (int)((reinterpret_cast<uintptr_t>(A.X + base) / sizeof(Tio)) & (kLine - 1)));
    const Tio* lr = lds + opaque(tid + (tid / kB) * PAD);
    constexpr int lstride = (NT / kB) * (kB + PAD);
    if (mis == 0) {
      const __amdgpu_buffer_rsrc_t dst = make_rsrc(A.X + base, (int64_t)rows * sizeof(Tio));
#pragma unroll
      for (int j = 0; j < kB; ++j)
        buf_store<Tio, kStoreAux>(dst, vs + j * NT * (int)sizeof(Tio), lr[j * lstride]);
    } else {
      constexpr int kDrop = 1 << 30;
      const __amdgpu_buffer_rsrc_t dst =
          make_rsrc(A.X + base - mis, (int64_t)(rows + mis) * sizeof(Tio));
      int u = tid - mis, jo = 0;
      if (u < 0) {
        u += NT;
        jo = -1;
      }
      const Tio* lu = lds + opaque(u + (u / kB) * PAD);
#pragma unroll
      for (int j = 0; j <= kB; ++j) {
        const int jj = j + jo;
        const bool ok = jj >= 0 && jj < kB && jj * NT + u < rows;
        const Tio val = lu[(jj < 0 ? 0 : (jj < kB ? jj : kB - 1)) * lstride];
        buf_store<Tio, kStoreAux>(dst, ok ? vs + j * NT * (int)sizeof(Tio) : kDrop, val);
      }
    }
    if constexpr (BWD) {
      // t-gradient partial sums of the run; products across two systems' rows
      // are left out.  row r of its system: e - (e / N) N, by a 31-bit
      // reciprocal (exact: e N < 2^31 here)
      const uint32_t rn = (uint32_t)((1u << 31) / (uint32_t)N) + 1u;
      double s0 = 0.0, s1 = 0.0, sm1 = 0.0, sp = 0.0, sc = 0.0;
#pragma unroll 4
      for (int j = 0; j < kB; ++j) {
        const int e = j * NT + tid;
        const int xo = vs + j * NT * (int)sizeof(Tio);
        const Tio xt = j < 4 ? xpre[j < 4 ? j : 0] : buf_load<Tio>(xf, xo);
        Tio xn = __shfl_down(xt, 1, 64);   // element e + 1
        Tio xq = __shfl_up(xt, 1, 64);     // element e - 1
        if (lane == 63) xn = buf_load<Tio>(xf, xo + (int)sizeof(Tio));
        if (lane == 0) xq = buf_load<Tio>(xf, xo - (int)sizeof(Tio));
        const int r = e - (int)__umulhi(2u * (uint32_t)e, rn) * N;
        const double gv = e < rows ? (double)lr[j * lstride] : 0.0;
        const double d = e < rows ? gv * (double)xt : 0.0;
        s0 += d;
        s1 += e < rows && r + 1 < N ? gv * (double)xn : 0.0;
        sm1 += e < rows && r > 0 ? gv * (double)xq : 0.0;
        if (QUASI) {
          sp += r == 0 ? d : 0.0;
          sc += r == N - 1 ? d : 0.0;
        }
      }
#pragma unroll
      for (int d = 32; d >= 1; d >>= 1) {
        s0 += __shfl_xor(s0, d, 64);
        s1 += __shfl_xor(s1, d, 64);
        sm1 += __shfl_xor(sm1, d, 64);
        if (QUASI) {
          sp += __shfl_xor(sp, d, 64);
          sc += __shfl_xor(sc, d, 64);
        }
      }
      double* gp = A.gpart + (QUASI ? kGradN : 3) * (A.items ? (int64_t)S.fslot0 : k);
      if constexpr (NW > 1) {
        if (lane == 0) {
          red[w][0] = sm1;
          red[w][1] = s0;
          red[w][2] = s1;
          red[w][3] = sp;
          red[w][4] = sc;
        }
        __syncthreads();
        sm1 = s0 = s1 = sp = sc = 0.0;
        for (int q = 0; q < NW; ++q) {
          sm1 += red[q][0];
          s0 += red[q][1];
          s1 += red[q][2];
          sp += red[q][3];
          sc += red[q][4];
        }
      }
      if (tid == 0) {
        gp[0] = -sm1;
        gp[1] = -s0;
        gp[2] = -s1;
        if (QUASI) {
          gp[3] = -sp;
          gp[4] = -sc;
          if (A.items)   // the system's corner slots: their terms are above
            for (int q = kGradN; q < 3 * kGradN; ++q) gp[q] = 0.0;
        }
      }
    }
  }
  if constexpr (REFINE) {
    // the workgroup's record: the largest over its lanes' systems
    __syncthreads();
    smax[tid] = 0;
    __syncthreads();
    atomicMax(&smax[0], it_max);
    atomicMax(&smax[1], __float_as_int(est_max));
    __syncthreads();
    publish_refine_record(A.iters, smax[0], __int_as_float(smax[1]));
  }
}

template <int NT, typename Tio, typename Tc, bool REFINE, bool BWD, bool QUASI>
hipError_t go(const LaunchSet& L, const ShortArgs<Tio>& A, hipStream_t st) {
  // with a cap of persistent workgroups per CU (counted in workgroups of the
  // plan's shape) as many lanes loop over the runs
  int64_t grid = A.nitems;
  if (L.wg_per_cu > 0) {
    const int64_t cap = (int64_t)device_cus() * L.wg_per_cu * (kShapes[L.shape].NT / NT);
    grid = grid < cap ? grid : cap;
  }
  hipLaunchKernelGGL((k_short<NT, Tio, Tc, REFINE, BWD, QUASI>), dim3((unsigned)grid), dim3(NT),
                     0, st, A);
  return hipGetLastError();
}

template <typename Tio, typename Tc, bool REFINE, bool BWD, bool QUASI>
hipError_t by_width(int nt, const LaunchSet& L, const ShortArgs<Tio>& A, hipStream_t st) {
  switch (nt) {
    case 64: return go<64, Tio, Tc, REFINE, BWD, QUASI>(L, A, st);
    case 128: return go<128, Tio, Tc, REFINE, BWD, QUASI>(L, A, st);
    case 256: return go<256, Tio, Tc, REFINE, BWD, QUASI>(L, A, st);
    case 512: return go<512, Tio, Tc, REFINE, BWD, QUASI>(L, A, st);
  }
  return hipErrorInvalidValue;
}

template <typename Tio, typename Tc, bool REFINE>
hipError_t run_short(const LaunchSet& L, const void* F, void* X, const void* Xfwd, bool bwd,
                     hipStream_t st) {
  const int nt = L.n_short > 0 ? kShortItemNT : L.short_nt;
  ShortArgs<Tio> A{};
  A.F = static_cast<const Tio*>(F);
  A.X = static_cast<Tio*>(X);
  A.Xfwd = static_cast<const Tio*>(Xfwd);
  A.sys = L.sys;
  A.vec64 = L.vec64;
  A.vec32 = L.vec32;
  A.tabnt = kShapes[L.shape].NT;
  A.tab64 = L.tab64;
  A.tab32 = L.tab32;
  A.qtab64 = L.qtab64;
  A.qnt = L.qnt;
  A.items = L.n_short > 0 ? L.short_items : nullptr;
  A.nitems = L.n_short > 0 ? L.n_short : L.short_runs;
  A.M = L.short_M;
  A.G = L.short_g;
  A.gpart = L.gpart;
  A.iters = L.iters;
  A.max_iter = L.max_iter;
  A.refine_tol = L.refine_tol;
  if constexpr (sizeof(Tio) == 8) {
    if (L.quasi)
      return bwd ? by_width<Tio, Tc, REFINE, true, true>(nt, L, A, st)
                 : by_width<Tio, Tc, REFINE, false, true>(nt, L, A, st);
  }
  if (L.quasi) return hipErrorInvalidValue;   // (float plans: mark_short)
  return bwd ? by_width<Tio, Tc, REFINE, true, false>(nt, L, A, st)
             : by_width<Tio, Tc, REFINE, false, false>(nt, L, A, st);
}

}  // namespace

hipError_t launch_short(int dtype, bool bwd, const LaunchSet& L, const void* F, void* X,
                        const void* Xfwd, hipStream_t st) {
  switch (dtype) {
    case 0: return run_short<double, double, false>(L, F, X, Xfwd, bwd, st);
    case 1: return run_short<float, float, false>(L, F, X, Xfwd, bwd, st);
    default: return run_short<double, float, true>(L, F, X, Xfwd, bwd, st);
  }
}

}  // namespace tdt
