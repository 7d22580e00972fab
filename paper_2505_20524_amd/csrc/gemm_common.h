// What the GEMM kernels share: the launch arguments, the direct global -> LDS load, the bf16 convert.
#pragma once
#include "common.h"
#include "launch.h"

struct GemmArgs {
  const uint8_t* A;
  const uint8_t* B;
  uint16_t* C;
  const float* sinv_a;
  const float* sinv_b;
  int64_t lda, ldb, ldc;
  int M, N, K;
  int tiles_m, tiles_n;
  int vec_store;  // C rows allow 16-byte stores
  int wide_store; // interior tiles are stored as whole 128-byte lines (launches of several tiles per workgroup)
  uint32_t a_bytes, b_bytes;  // addressable span of each operand
  // contraction split (splits == 1: none): work item = chunk * tiles + tile, chunk c covers
  // contraction indices [c * k_chunk, min(K, (c + 1) * k_chunk)); partial holds splits * tiles blocks of a tile's
  // floats in the register order of the accumulators
  int splits, k_chunk;
  float* partial;
};

// Launches one of the small-tile kernels (gemm_tile_kernels.hip) on checked arguments.
enum GemmTile { TILE_256x128, TILE_128x128, TILE_128x128_2WG, TILE_64x64 };
__attribute__((visibility("hidden"))) fog_status gemm_tile_launch(GemmTile tile, fog_layout layout, fog_fp8 fmt_a, fog_fp8 fmt_b, GemmArgs g, hipStream_t s);
// Adds up the partial tiles of a split product whose tiles are 64 ti x 64 tj.
__attribute__((visibility("hidden"))) void gemm_reduce_launch(const GemmArgs& g, int ti, int tj, hipStream_t s);

namespace {

constexpr int BK = 64;                       // contraction bytes of one matrix instruction
constexpr int PAIR_K = 2 * BK;               // contraction bytes per load unit: whole 128-byte lines of the operands
constexpr uint32_t OOB = 0x80000000u;        // a buffer offset past any operand (spans are < 2^31 bytes)

typedef __attribute__((address_space(3))) v2i* lds_v2i_ptr;

// 16 bytes per lane from buffer `rsrc` at byte offset `voff` (zero when out of range) to
// LDS[m0 + 16 * lane].  Issued as inline assembly so that the compiler's own wait-count
// insertion does not serialise the LDS reads of other stages behind these loads; completion is
// awaited explicitly with s_waitcnt vmcnt + barrier in the main loop.
FOG_DEVICE void load_to_lds(v4i rsrc, uint32_t voff, uint32_t lds_addr_uniform) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds"
               :
               : "v"(voff), "s"(rsrc), "s"(lds_addr_uniform)
               : "memory", "m0");
}

// Raw buffer descriptor (stride 0): 48-bit base, byte count for the bounds check, dword-format flags.
FOG_DEVICE v4i make_rsrc(const void* base, uint32_t bytes) {
  const uint64_t b = reinterpret_cast<uint64_t>(base);
  v4i r;
  r[0] = (int)(uint32_t)b;
  r[1] = (int)((uint32_t)(b >> 32) & 0xFFFFu);
  r[2] = (int)bytes;
  r[3] = 0x00020000;
  return r;
}

// Eight consecutive elements of row m of C from column n (< N) on: one 16-byte store where C allows it, element-wise at the
// right edge and where C is not aligned.
FOG_DEVICE void store_row_piece(const GemmArgs& g, int m, int n, uint4 v) {
  uint16_t* dst = g.C + (int64_t)m * g.ldc + n;
  if (g.vec_store && n + 8 <= g.N) {
    st_nt16(dst, v);
  } else {
    const uint32_t wv[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int e = 0; e < 8; ++e)
      if (n + e < g.N) dst[e] = (uint16_t)(wv[e >> 1] >> (16 * (e & 1)));
  }
}

}  // namespace
