// tdt_device.h -- device helpers shared by the kernels of Toeplitz systems
// (tdt_kernels.hip, tdt_short.hip): work shapes, constant-address-space and
// buffer accesses, cross-lane moves, the affine scans of eq. (15) inside a
// wavefront, and a system's constants in compute precision.
#pragma once
#include <stdint.h>
#include <hip/hip_runtime.h>

#include "tdt_internal.h"

namespace tdt {

// Compile-time work shape of the tile kernels: B rows per lane, NT lanes per
// workgroup (NW wavefronts), tiles of L = B*NT rows, occupancy target WAVES.
template <int B_, int NT_, int WAVES_>
struct Shape {
  static constexpr int B = B_;
  static constexpr int NT = NT_;
  static constexpr int NW = NT_ / 64;
  static constexpr int L = B_ * NT_;
  static constexpr int WAVES = WAVES_;
};
// The names the shape-generic code uses for its shape's sizes.
#define TDT_SHAPE(SH)                          \
  [[maybe_unused]] constexpr int kB = SH::B;   \
  [[maybe_unused]] constexpr int kNT = SH::NT; \
  [[maybe_unused]] constexpr int kNW = SH::NW; \
  [[maybe_unused]] constexpr int kTile = SH::L;

// Read-only per-plan data (block vectors, system descriptors, work lists) is
// read through the constant address space: with a wave-uniform address the
// compiler then uses scalar loads into SGPRs, which the sweeps take as
// operands, instead of vector loads into VGPRs.
template <typename T>
using cptr = const __attribute__((address_space(4))) T*;
template <typename T>
__device__ __forceinline__ cptr<T> as_const(const T* p) {
  return (cptr<T>)(uintptr_t)p;
}

// Hides a value from the optimiser (an empty asm that "modifies" a register)
// so that per-element offsets derived from it are recomputed next to each
// access instead of being hoisted out of the tile loop and kept live.
__device__ __forceinline__ int opaque(int v) {
  asm volatile("" : "+v"(v));
  return v;
}

// The same for a pointer to per-plan constants: loads through the returned
// pointer cannot be merged with, or hoisted above, earlier loads of the same
// data, so each phase of a solve re-reads (with cheap scalar loads) the
// constants it uses instead of keeping all of them live in SGPRs.
template <typename T>
__device__ __forceinline__ cptr<T> fresh(cptr<T> p) {
  uint64_t v = (uint64_t)(uintptr_t)p;
  asm volatile("" : "+s"(v));
  return (cptr<T>)(uintptr_t)v;
}

// Raw buffer accesses: a wave-uniform resource (base, size in bytes) held in
// SGPRs plus one per-lane byte offset.  The hardware range check returns 0
// for reads at or past `bytes` (and for "negative" offsets, which wrap to
// huge unsigned ones) and drops such writes, which is how partial tiles and
// the rows just outside a system are handled.
// The base and size are wave-uniform by construction; readfirstlane states it
// to the compiler, which otherwise may not prove it and would wrap every
// access in a loop over distinct descriptors.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, int64_t bytes) {
  const uint64_t a = reinterpret_cast<uintptr_t>(base);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  const int nb = __builtin_amdgcn_readfirstlane((int)bytes);
  void* ub = reinterpret_cast<void*>((uintptr_t)(((uint64_t)hi << 32) | lo));
  return __builtin_amdgcn_make_buffer_rsrc(ub, (short)0, nb, 0x00020000);
}
template <typename T>
__device__ __forceinline__ T buf_load(__amdgpu_buffer_rsrc_t r, int off) {
  if constexpr (sizeof(T) == 8)
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
  else
    return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
}
// AUX: the instruction's cache-policy bits (0: default; 2: non-temporal).
template <typename T, int AUX = 0>
__device__ __forceinline__ void buf_store(__amdgpu_buffer_rsrc_t r, int off, T v) {
  if constexpr (sizeof(T) == 8) {
    using V = decltype(__builtin_amdgcn_raw_buffer_load_b64(r, 0, 0, 0));
    __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(V, v), r, off, 0, AUX);
  } else {
    using V = decltype(__builtin_amdgcn_raw_buffer_load_b32(r, 0, 0, 0));
    __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(V, v), r, off, 0, AUX);
  }
}
// The solution is stored non-temporal: it is not read again by this solve,
// and lines that do not linger dirty in the caches leave the next read of the
// right-hand side (the first pass of the next solve) at full speed.
constexpr int kStoreAux = 2;

// Cross-lane moves inside a wavefront.  DPP row shifts move a value by d lanes
// within each row of 16 lanes (lanes whose source falls outside the row keep
// `old`); readlane copies one lane's value to all lanes.
template <int CTRL>
__device__ __forceinline__ float dpp(float old, float src) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(__builtin_bit_cast(int, old),
                                                               __builtin_bit_cast(int, src),
                                                               CTRL, 0xf, 0xf, false));
}
template <int CTRL>
__device__ __forceinline__ double dpp(double old, double src) {
  const uint64_t o = __builtin_bit_cast(uint64_t, old), v = __builtin_bit_cast(uint64_t, src);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)o, (int)(uint32_t)v,
                                                            CTRL, 0xf, 0xf, false);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp((int)(uint32_t)(o >> 32),
                                                            (int)(uint32_t)(v >> 32), CTRL, 0xf,
                                                            0xf, false);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ float readlane(float v, int l) {
  return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}
__device__ __forceinline__ double readlane(double v, int l) {
  const uint64_t u = __builtin_bit_cast(uint64_t, v);
  const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)u, l);
  const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(u >> 32), l);
  return __builtin_bit_cast(double, ((uint64_t)hi << 32) | lo);
}
// Maximum over the 64 lanes (all lanes receive it).
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp<0x111>(v, v));
  v = fmaxf(v, dpp<0x112>(v, v));
  v = fmaxf(v, dpp<0x114>(v, v));
  v = fmaxf(v, dpp<0x118>(v, v));
  return fmaxf(fmaxf(readlane(v, 15), readlane(v, 31)), fmaxf(readlane(v, 47), readlane(v, 63)));
}
__device__ __forceinline__ double wave_max(double v) {
  v = fmax(v, dpp<0x111>(v, v));
  v = fmax(v, dpp<0x112>(v, v));
  v = fmax(v, dpp<0x114>(v, v));
  v = fmax(v, dpp<0x118>(v, v));
  return fmax(fmax(readlane(v, 15), readlane(v, 31)), fmax(readlane(v, 47), readlane(v, 63)));
}

// Sum over the 64 lanes in a fixed order (all lanes receive it).
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp<0x111>(0.0, v);
  v += dpp<0x112>(0.0, v);
  v += dpp<0x114>(0.0, v);
  v += dpp<0x118>(0.0, v);
  return (readlane(v, 15) + readlane(v, 31)) + (readlane(v, 47) + readlane(v, 63));
}

constexpr int kDppRowShr = 0x110;   // + d: row_shr:d
constexpr int kDppRowShl = 0x100;   // + d: row_shl:d

// Inclusive left-to-right scan over the 64 lanes of affine maps x -> A x + g
// (composition: the map of lane l applied after those of lanes < l): four
// in-row DPP steps, then the four row totals (readlane) carried across rows.
template <typename T>
__device__ __forceinline__ void wave_scan_affine_fwd(T& A, T& g) {
#define TDT_FWD_STEP(D)                                    \
  {                                                        \
    const T As = dpp<kDppRowShr + D>(T(1), A);             \
    const T gs = dpp<kDppRowShr + D>(T(0), g);             \
    g = A * gs + g;                                        \
    A = A * As;                                            \
  }
  TDT_FWD_STEP(1) TDT_FWD_STEP(2) TDT_FWD_STEP(4) TDT_FWD_STEP(8)
#undef TDT_FWD_STEP
  const int row = (threadIdx.x & 63) >> 4;
  const T A0 = readlane(A, 15), g0 = readlane(g, 15);
  const T A1 = readlane(A, 31), g1 = readlane(g, 31);
  const T A2 = readlane(A, 47), g2 = readlane(g, 47);
  // carry into row r: rows 0..r-1 composed
  const T cA1 = A0, cg1 = g0;
  const T cA2 = A1 * cA1, cg2 = A1 * cg1 + g1;
  const T cA3 = A2 * cA2, cg3 = A2 * cg2 + g2;
  const T cA = row == 0 ? T(1) : (row == 1 ? cA1 : (row == 2 ? cA2 : cA3));
  const T cg = row == 0 ? T(0) : (row == 1 ? cg1 : (row == 2 ? cg2 : cg3));
  g = A * cg + g;
  A = A * cA;
}

// Inclusive right-to-left scan of affine maps u -> C u + h (the map of lane l
// applied after those of lanes > l).
template <typename T>
__device__ __forceinline__ void wave_scan_affine_bwd(T& C, T& h) {
#define TDT_BWD_STEP(D)                                    \
  {                                                        \
    const T Cs = dpp<kDppRowShl + D>(T(1), C);             \
    const T hs = dpp<kDppRowShl + D>(T(0), h);             \
    h = C * hs + h;                                        \
    C = C * Cs;                                            \
  }
  TDT_BWD_STEP(1) TDT_BWD_STEP(2) TDT_BWD_STEP(4) TDT_BWD_STEP(8)
#undef TDT_BWD_STEP
  const int row = (threadIdx.x & 63) >> 4;
  const T C1 = readlane(C, 16), h1 = readlane(h, 16);
  const T C2 = readlane(C, 32), h2 = readlane(h, 32);
  const T C3 = readlane(C, 48), h3 = readlane(h, 48);
  // carry into row r from the right: rows r+1..3 composed
  const T eC2 = C3, eh2 = h3;
  const T eC1 = C2 * eC2, eh1 = C2 * eh2 + h2;
  const T eC0 = C1 * eC1, eh0 = C1 * eh1 + h1;
  const T eC = row == 3 ? T(1) : (row == 2 ? eC2 : (row == 1 ? eC1 : eC0));
  const T eh = row == 3 ? T(0) : (row == 2 ? eh2 : (row == 1 ? eh1 : eh0));
  h = C * eh + h;
  C = C * eC;
}

// Per-system constants in compute precision.
template <typename Tc>
struct Consts {
  cptr<Tc> iu;
  cptr<Tc> aiu;
  cptr<Tc> cp;
  cptr<Tc> phi;
  cptr<Tc> chi;
  Tc a;
  Tc pf, pl, cf;          // phi_first, phi_last, chi_first of a full block
  Tc tail_pf, tail_pl, tail_cf;   // the same of the system's last block
};

// Copy of a system descriptor read with scalar loads (wave-uniform index).
__device__ __forceinline__ SysDesc load_sys(const SysDesc* sys, int s) {
  SysDesc D;
  const cptr<uint64_t> src = as_const(reinterpret_cast<const uint64_t*>(sys + s));
  uint64_t* dst = reinterpret_cast<uint64_t*>(&D);
#pragma unroll
  for (int k = 0; k < (int)(sizeof(SysDesc) / 8); ++k) dst[k] = src[k];
  return D;
}

template <class SH, typename Tc>
__device__ __forceinline__ Consts<Tc> make_consts(const SysDesc& S, const double* vec64,
                                                  const float* vec32) {
  TDT_SHAPE(SH)
  Consts<Tc> K;
  const Tc* v;
  if constexpr (sizeof(Tc) == 8)
    v = reinterpret_cast<const Tc*>(vec64) + (int64_t)S.cidx * kVecN * kB;
  else
    v = reinterpret_cast<const Tc*>(vec32) + (int64_t)S.cidx * kVecN * kB;
  const cptr<Tc> c = as_const(v);
  K.iu = c + kVecIU * kB;
  K.aiu = c + kVecAIU * kB;
  K.cp = c + kVecCP * kB;
  K.phi = c + kVecPHI * kB;
  K.chi = c + kVecCHI * kB;
  K.a = (Tc)S.a;
  K.pf = (Tc)S.blk[0]; K.pl = (Tc)S.blk[1]; K.cf = (Tc)S.blk[2];
  K.tail_pf = (Tc)S.tail_pf; K.tail_pl = (Tc)S.tail_pl; K.tail_cf = (Tc)S.tail_cf;
  return K;
}

// A workgroup's refinement record, published once when it exits: rec[0] =
// most float solves of any tile, rec[1] = bits of the largest estimated
// remaining relative error (non-negative floats order like their bits).
// Thousands of workgroups publish to the same two words, and atomics on one
// address serialise; the record only grows, so a plain read that already
// shows a value at least as large (a stale read can only show a smaller one)
// makes the atomic unnecessary, and most workgroups skip it.
__device__ __forceinline__ void publish_refine_record(int* rec, int it_max, float est_max) {
  if (threadIdx.x == 0 && rec && it_max > 0) {
    const int e = __float_as_int(est_max);
    if (__atomic_load_n(rec, __ATOMIC_RELAXED) < it_max) atomicMax(rec, it_max);
    if (__atomic_load_n(rec + 1, __ATOMIC_RELAXED) < e) atomicMax(rec + 1, e);
  }
}

}  // namespace tdt
