// Device-side helpers shared by the HIP kernels (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include "../../include/fog.h"

typedef int v8i __attribute__((ext_vector_type(8)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef unsigned short us2 __attribute__((ext_vector_type(2)));

#define FOG_DEVICE static __device__ __forceinline__

// bf16 bit pattern (low 16 bits) -> float, exact.
FOG_DEVICE float bf16lo(uint32_t w) { return __uint_as_float(w << 16); }
FOG_DEVICE float bf16hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

// Two floats -> packed bf16 with the hardware convert: round to nearest even, a NaN becomes a quiet NaN with its upper payload
// bits (the same bits as the integer form (u + 0x7FFF + lsb) >> 16 for all 2^32 inputs, at one instruction instead of twelve).
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
FOG_DEVICE uint32_t pack_bf16x2(float lo, float hi) {
  f32x2 v = {lo, hi};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
FOG_DEVICE uint32_t f32_to_bf16(float f) { return pack_bf16x2(f, f) & 0xFFFFu; }

// A register whose contents do not matter.  The packed FP8 converts write one half of their destination and keep the
// other; a dword that both halves of are about to be written needs no initial value, and a literal 0 would cost a move.
FOG_DEVICE uint32_t any_u32() {
  uint32_t r;
  asm volatile("" : "=v"(r));
  return r;
}

// Saturating round-to-nearest-even cast of four floats to one dword of FP8 codes (byte i <- v_i).
// The hardware convert rounds to nearest even but turns overflow into NaN / infinity, so the
// magnitude is clamped to the largest finite value first.
template <int FMT>
FOG_DEVICE uint32_t cvt4_fp8(float a, float b, float c, float d) {
  uint32_t r = any_u32();
  if (FMT == FOG_E4M3) {
    const float mx = 448.0f;
    a = __builtin_amdgcn_fmed3f(a, -mx, mx); b = __builtin_amdgcn_fmed3f(b, -mx, mx);
    c = __builtin_amdgcn_fmed3f(c, -mx, mx); d = __builtin_amdgcn_fmed3f(d, -mx, mx);
    r = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, r, false);
    r = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, r, true);
  } else {
    const float mx = 57344.0f;
    a = __builtin_amdgcn_fmed3f(a, -mx, mx); b = __builtin_amdgcn_fmed3f(b, -mx, mx);
    c = __builtin_amdgcn_fmed3f(c, -mx, mx); d = __builtin_amdgcn_fmed3f(d, -mx, mx);
    r = __builtin_amdgcn_cvt_pk_bf8_f32(a, b, r, false);
    r = __builtin_amdgcn_cvt_pk_bf8_f32(c, d, r, true);
  }
  return r;
}

// Switches the wave's FP8 converts to saturation (MODE.FP16_OVFL): a finite value beyond the format becomes the largest finite
// code, which makes the clamp above unnecessary; a NaN keeps its NaN code, an infinity is not clamped.
// Only for kernels that neither convert to bf16 (finite values then round to the largest finite bf16 instead of infinity) nor run
// matrix instructions (they then drop NaNs and turn infinities into the largest finite float).
FOG_DEVICE void saturating_converts() { __builtin_amdgcn_s_setreg(1 | (23 << 6) | (0 << 11), 1); }

// The cast without the clamp, for waves that switched saturation on and values that are finite.
template <int FMT>
FOG_DEVICE uint32_t cvt4_fp8_finite(float a, float b, float c, float d) {
  uint32_t r = any_u32();
  if (FMT == FOG_E4M3) {
    r = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, r, false);
    r = __builtin_amdgcn_cvt_pk_fp8_f32(c, d, r, true);
  } else {
    r = __builtin_amdgcn_cvt_pk_bf8_f32(a, b, r, false);
    r = __builtin_amdgcn_cvt_pk_bf8_f32(c, d, r, true);
  }
  return r;
}

// The same cast for tensors that may hold NaN (the bulk casts): the clamp above returns the smallest of
// its operands for a NaN input, i.e. the largest finite code with a minus sign, so NaN inputs are patched
// afterwards to the NaN code 0x7F with the input's sign.  Infinities saturate through the clamp.  The test
// costs two unordered compares per four values; the patch runs only in waves that hold a NaN.
template <int FMT>
FOG_DEVICE uint32_t cvt4_fp8_nan(float a, float b, float c, float d, bool* saw_nan = nullptr) {
  uint32_t r = cvt4_fp8<FMT>(a, b, c, d);
  if (__builtin_expect(__builtin_isunordered(a, b) || __builtin_isunordered(c, d), 0)) {
    if (saw_nan) *saw_nan = true;
    if (a != a) r = (r & 0xFFFFFF00u) | 0x0000007Fu | ((__float_as_uint(a) >> 24) & 0x00000080u);
    if (b != b) r = (r & 0xFFFF00FFu) | 0x00007F00u | ((__float_as_uint(b) >> 16) & 0x00008000u);
    if (c != c) r = (r & 0xFF00FFFFu) | 0x007F0000u | ((__float_as_uint(c) >> 8) & 0x00800000u);
    if (d != d) r = (r & 0x00FFFFFFu) | 0x7F000000u | (__float_as_uint(d) & 0x80000000u);
  }
  return r;
}

// Bit pattern of a thread's running abs-max (a non-negative float, kept with fmaxf, which drops NaN
// operands) for the integer reductions that follow: a thread that saw a NaN contributes the NaN pattern,
// which orders above every finite value and infinity, so a diverged tensor shows in the abs-max.
FOG_DEVICE uint32_t amax_bits(float m, bool saw_nan) { return saw_nan ? 0x7FC00000u : __float_as_uint(m); }

// Wave-wide (64 lanes) reductions through cross-lane shuffles.
FOG_DEVICE uint32_t wave_max_u32(uint32_t v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) {
    uint32_t t = (uint32_t)__shfl_xor((int)v, o, 64);
    v = v > t ? v : t;
  }
  return v;
}
FOG_DEVICE float wave_max_f32(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}
FOG_DEVICE float wave_sum_f32(float v) {
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

// max over the magnitudes of the two bf16 halves of each dword, kept as packed u16 pairs.
FOG_DEVICE uint32_t pkmax_abs_bf16(uint32_t acc, uint32_t w) {
  us2 a = __builtin_bit_cast(us2, acc);
  us2 b = __builtin_bit_cast(us2, w & 0x7FFF7FFFu);
  us2 m = __builtin_elementwise_max(a, b);
  return __builtin_bit_cast(uint32_t, m);
}

// Larger of the two halves of a packed pair of u16.
FOG_DEVICE uint32_t max_of_pair(uint32_t p) { return (p & 0xFFFFu) > (p >> 16) ? (p & 0xFFFFu) : (p >> 16); }

// Streaming (non-temporal) 16- and 8-byte global accesses: data touched once should not evict
// what other kernels keep in cache.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
FOG_DEVICE uint4 ld_nt16(const void* p) {
  u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p));
  return make_uint4(v[0], v[1], v[2], v[3]);
}
FOG_DEVICE void st_nt16(void* p, uint4 v) {
  u32x4 w = {v.x, v.y, v.z, v.w};
  __builtin_nontemporal_store(w, reinterpret_cast<u32x4*>(p));
}
FOG_DEVICE void st_nt8(void* p, uint2 v) {
  u32x2 w = {v.x, v.y};
  __builtin_nontemporal_store(w, reinterpret_cast<u32x2*>(p));
}

// Stores written through: the lines stay in the caches for the next kernel, but clean, so that nothing is left to write back when the
// kernel ends or while the next one runs.  (The two wait states cover the rule that the data registers of a store of more than 8 bytes
// must not be written by the next two vector instructions; the compiler, which keeps it for its own stores, does not see the one inside
// the assembly.)
FOG_DEVICE void st_through16(void* p, uint4 v) {
  u32x4 w = {v.x, v.y, v.z, v.w};
  asm volatile("global_store_dwordx4 %0, %1, off sc1\n\ts_nop 1" ::"v"(p), "v"(w) : "memory");
}
FOG_DEVICE void st_through8(void* p, uint2 v) {
  u32x2 w = {v.x, v.y};
  asm volatile("global_store_dwordx2 %0, %1, off sc1" ::"v"(p), "v"(w) : "memory");
}

// A wave's result tile of 32 rows x (32 T) columns, from the accumulators of T 32 x 32 matrix tiles (lane & 31 = row, 8 (r / 4) +
// 4 (lane / 32) + r % 4 = column of a tile): scaled, rounded to bf16, parked in LDS (32 rows of 64 T + 16 bytes, the wave's own) and
// stored as whole 128-byte lines past the caches.
template <int T, typename RowOf>
FOG_DEVICE void store_tile_rows(uint8_t* stage, const v16f* x, float scale, uint16_t* out, int ld, RowOf row_of) {
  constexpr int STRIDE = 64 * T + 16, LPR = 4 * T, RPS = 64 / LPR;    // bytes of a staged row, lanes per row, rows per store
  const int l = threadIdx.x & 63;
  // (the wave's LDS instructions complete in order: all that is needed is that the compiler keeps their order, here against what
  // the wave has read from the area before, and between the two halves below)
  asm volatile("" ::: "memory");
#pragma unroll
  for (int d = 0; d < T; ++d)
#pragma unroll
    for (int qd = 0; qd < 4; ++qd)
      *reinterpret_cast<uint2*>(stage + (l & 31) * STRIDE + 64 * d + 16 * qd + 8 * (l >> 5)) =
          make_uint2(pack_bf16x2(x[d][4 * qd] * scale, x[d][4 * qd + 1] * scale), pack_bf16x2(x[d][4 * qd + 2] * scale, x[d][4 * qd + 3] * scale));
  asm volatile("" ::: "memory");
#pragma unroll
  for (int t = 0; t < 32 / RPS; ++t) {
    const int row = RPS * t + l / LPR, piece = l % LPR;
    st_nt16(out + (int64_t)row_of(row) * ld + 8 * piece, *reinterpret_cast<const uint4*>(stage + row * STRIDE + 16 * piece));
  }
  asm volatile("" ::: "memory");
}

// Makes the compiler treat `v` as used here.  Kernels that stream tiles into LDS with direct loads
// issued from inline assembly wait for those loads with explicit s_waitcnt immediates; the
// compiler does not see them, so any ordinary global load still "outstanding" in its bookkeeping
// when the loop starts would make it put s_waitcnt vmcnt(0) inside the loop (where the value is
// first used), which also waits for the whole prefetch stream.  Using every such value once
// before the first direct load moves that wait in front of the loop.
#define FOG_SETTLE(v) asm volatile("" ::"v"(v))
