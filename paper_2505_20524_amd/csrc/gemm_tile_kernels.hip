// Scaled FP8 GEMM on tiles smaller than 256 x 256 (same product, layouts and result rules as gemm_kernels.hip), for the
// launches whose 256 x 256 tiles leave much of the chip idle.
//
// One workgroup of 4 waves per tile, no persistence: with few tiles there is nothing to walk.  Operand stages of 128 contraction
// bytes go straight into an LDS ring of two to four stages (buffer_load ... lds); the fragments of a whole stage are read into
// registers one stage ahead, under the matrix instructions of the current one, so that a stage costs one barrier and no wait
// for LDS.  A stage of 64 x 64, 128 x 128 and 256 x 128 (16, 32 and 48 KB of operands) takes 0.11, 0.25 and 0.42 us with few
// workgroups on the chip, i.e. 150, 130 and 115 GB/s a compute unit, and 0.21, 0.46 and 0.77 us with one on each, 80, 70 and 62 GB/s
// (fits of plan_product); deeper rings, and fragments read later or earlier, change nothing.  Hence its rule: the largest tile that
// still spreads the product over the chip, and where even 64 x 64 leaves it idle, a split of the contraction.
// Kernel times (256 x 256 kernel before, with its own contraction split where it had one -> now), us:
//   512 x 1024 x 1024 NT  14.6 -> 4.7     1777 x 3088 x 2064 NT  46.9 -> 20.6    1777 x 2064 x 3088 NN  54.1 -> 20.2
//   4096 x 2048 x 8192 NN  69.5 -> 53.4   754 x 432 x 12832 NT   27.2 -> 18.2    8192 x 2048 x 4096 TN  55 -> 59 (not taken)
//
// Contraction split, of these kernels and of the 256 x 256 one.  With a caller workspace a product of few tiles and a long
// contraction is cut along K into chunks: the unit
// of work becomes (tile, chunk), every unit leaves its binary32 accumulators in the workspace, and a second kernel adds the
// chunks of a tile in ascending order, applies the scales and rounds once to bf16.  Deterministic (no atomics); the sums differ
// from the unsplit kernel's only in the order of binary32 additions.
#include "gemm_common.h"

namespace {

constexpr int kThreads = 256;
template <int N> struct Int { static constexpr int value = N; };

// s_waitcnt immediate: vmcnt and lgkmcnt at most these, expcnt unbounded.
constexpr int waitcnt(int vm, int lgkm) { return (vm & 15) | (7 << 4) | (lgkm << 8) | ((vm >> 4) << 14); }

// Direct loads of one operand of a tile of 64 T rows (K-contiguous) or columns (K-major).  A stage is a pair of K-steps
// (128 contraction bytes); a wave fetches NP = 2 T pieces of 1 KB of it, piece j to byte NP * 1024 w + 1024 j.
//   K-contiguous: [64 T rows][128 bytes], piece = 8 rows, chunk c of a row at position c ^ ((row >> 1) & 7)
//   K-major:      [128 k][64 T bytes], piece = 16 / T contraction rows, chunk c of a row at position c ^ key(k)
// with key(k) = k & 7 for T = 2 and 4 and 2 ((k >> 2) & 1) for T = 1: the eight consecutive rows and two neighbouring
// chunks that half a wave touches in one transposing read then lie in sixteen different 16-byte columns of the banks.
template <bool KM, int T>
struct Loader {
  static constexpr int NP = 2 * T;
  static constexpr int ROWS = KM ? 16 / T : 8;    // rows of a piece
  uint32_t off[2];    // byte offset of pieces 0 and 1 of the next stage; piece j is at off[j & 1] + (j >> 1) * stride2
  int klim[2];        // piece j of the stage that starts at k0 is inside the matrix iff k0 + (KM ? ROWS * j : 0) < klim[j & 1]
  int jlim;           // pieces j >= jlim lie below the last row of a K-contiguous operand
  uint32_t stride2, step;

  static __device__ __forceinline__ int key(int k) { return T == 1 ? ((k >> 2) & 1) << 1 : k & 7; }

  __device__ __forceinline__ void init(int64_t ld, int first0, int extent, int kb, int K) {
    const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
    stride2 = (uint32_t)(2 * ROWS * ld);
    if (KM) {
      const int k = 32 * w + l / (4 * T);
      step = (uint32_t)(PAIR_K * ld);
      jlim = NP;
#pragma unroll
      for (int par = 0; par < 2; ++par) {
        const int c = (l % (4 * T)) ^ key(k + ROWS * par);
        klim[par] = K - k;
        off[par] = first0 + 16 * c < extent ? (uint32_t)((int64_t)(kb + k + ROWS * par) * ld + first0 + 16 * c) : OOB;
      }
    } else {
      const int r8 = l >> 3, first = first0 + 16 * T * w + r8, rem = extent - first;
      step = PAIR_K;
      jlim = rem > 0 ? (rem + 7) >> 3 : 0;
#pragma unroll
      for (int par = 0; par < 2; ++par) {
        const int c = (l & 7) ^ (r8 >> 1) ^ (4 * par);
        klim[par] = K - 16 * c;
        off[par] = (uint32_t)((int64_t)(first + 8 * par) * ld + kb + 16 * c);
      }
    }
  }
  __device__ __forceinline__ void issue(int j, v4i rsrc, int k0, uint32_t lds_piece_addr) const {
    const bool ok = (KM || j < jlim) && (k0 + (KM ? ROWS * j : 0) < klim[j & 1]);
    load_to_lds(rsrc, ok ? off[j & 1] + (uint32_t)(j >> 1) * stride2 : OOB, lds_piece_addr);
  }
  __device__ __forceinline__ void advance() { off[0] += step; off[1] += step; }
};

// Operand fragments of a wave (32 rows x 64 contraction bytes each); see gemm_kernels.hip for the lane mapping.
template <bool KM, int T>
struct Frags {
  static constexpr int ROW = KM ? 64 * T : PAIR_K;
  uint32_t a[4];
  __device__ __forceinline__ void init(int base) {
    const int l = threadIdx.x & 63;
    if (KM) {
      const int i = l & 15, k = 32 * (l >> 5) + (i >> 1);
#pragma unroll
      for (int t = 0; t < T; ++t) {
        const int col = base + 32 * t + (l & 16) + 8 * (i & 1);
        a[t] = (uint32_t)(k * ROW + (((col >> 4) ^ Loader<KM, T>::key(k)) << 4) + (col & 8));
      }
    } else {
      const int row = base + (l & 31), s = (row >> 1) & 7;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const int c = 4 * h + 2 * (l >> 5);
        a[2 * h] = (uint32_t)(row * ROW + ((c ^ s) << 4));
        a[2 * h + 1] = (uint32_t)(row * ROW + (((c + 1) ^ s) << 4));
      }
    }
  }
  __device__ __forceinline__ v8i read(const uint8_t* stage, int i, int h) const {
    v8i f;
    if (KM) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const v2i v = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(stage + a[i] + (64 * h + 8 * r) * ROW));
        f[2 * r] = v[0];
        f[2 * r + 1] = v[1];
      }
    } else {
      const v4i lo = *reinterpret_cast<const v4i*>(stage + a[2 * h] + 32 * ROW * i);
      const v4i hi = *reinterpret_cast<const v4i*>(stage + a[2 * h + 1] + 32 * ROW * i);
      f[0] = lo[0]; f[1] = lo[1]; f[2] = lo[2]; f[3] = lo[3];
      f[4] = hi[0]; f[5] = hi[1]; f[6] = hi[2]; f[7] = hi[3];
    }
    return f;
  }
};

// Tile number -> origin of the tile in C: groups of tile rows (about 1024 rows of C) walked column by column, so that the
// tiles in flight on one XCD share a few panels of A and B in its L2.
FOG_DEVICE void tile_origin(int logical, int tiles_m, int tiles_n, int bm, int bn, int& m0, int& n0) {
  const int GM = 1024 / bm;
  const int width = GM * tiles_n, group = logical / width, first_m = group * GM;
  const int gsz = tiles_m - first_m < GM ? tiles_m - first_m : GM, rem = logical - group * width;
  m0 = (first_m + rem % gsz) * bm;
  n0 = (rem / gsz) * bn;
}

// One workgroup of 4 waves (2 x 2) computes one tile of 64 TI x 64 TJ, a wave TI x TJ matrix tiles of 32 x 32.
template <int LAYOUT, int FA, int FB, int TI, int TJ, int NST, int WPS>
__global__ __launch_bounds__(kThreads, WPS) void fp8_gemm_tile_kernel(GemmArgs g) {
  extern __shared__ __attribute__((aligned(1024))) uint8_t smem[];
  constexpr bool A_KM = LAYOUT == FOG_TN, B_KM = LAYOUT != FOG_NT;
  constexpr int A_BYTES = 64 * TI * PAIR_K, B_BYTES = 64 * TJ * PAIR_K;
  constexpr int RING_B = NST * A_BYTES;
  constexpr int LOADS = 2 * TI + 2 * TJ;          // direct loads per wave and stage
  constexpr int NM = TI * TJ, NF = TI + TJ;       // matrix instructions and fragments per K-step

  // workgroups are dealt round-robin to the 8 XCDs: each takes one contiguous run of logical tile numbers
  const int ntiles = g.tiles_m * g.tiles_n;
  const int nitems = ntiles * g.splits;
  const int per_xcd = (nitems + 7) >> 3;
  const int item = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
  if (item >= nitems) return;
  const int chunk = item / ntiles, kb = chunk * g.k_chunk, klen = min(g.K - kb, g.k_chunk);
  int m0, n0;
  tile_origin(item - chunk * ntiles, g.tiles_m, g.tiles_n, 64 * TI, 64 * TJ, m0, n0);

  const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
  const int wm = (w >> 1) * 32 * TI, wn = (w & 1) * 32 * TJ;
  const v4i rsrc_a = make_rsrc(g.A, g.a_bytes), rsrc_b = make_rsrc(g.B, g.b_bytes);
  const uint32_t lds0 = (uint32_t)(uintptr_t)smem;
  const uint32_t lds_a = (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds0 + 2048u * TI * w));
  const uint32_t lds_b = (uint32_t)__builtin_amdgcn_readfirstlane((int)(lds0 + RING_B + 2048u * TJ * w));
  Loader<A_KM, TI> la;
  Loader<B_KM, TJ> lb;
  la.init(g.lda, m0, g.M, kb, klen);
  lb.init(g.ldb, n0, g.N, kb, klen);
  Frags<A_KM, TI> fa;
  Frags<B_KM, TJ> fb;
  fa.init(wm);
  fb.init(wn);
  const float alpha = (*g.sinv_a) * (*g.sinv_b);

  v16f acc[TI][TJ];
#pragma unroll
  for (int i = 0; i < TI; ++i)
#pragma unroll
    for (int j = 0; j < TJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  auto load_piece = [&](int t, int k0, int slot) {
    if (t < 2 * TI) la.issue(t, rsrc_a, k0, lds_a + (uint32_t)slot * A_BYTES + 1024u * t);
    else            lb.issue(t - 2 * TI, rsrc_b, k0, lds_b + (uint32_t)slot * B_BYTES + 1024u * (t - 2 * TI));
  };
  auto read_one = [&](int t, int slot, v8i* xa, v8i* xb) {       // fragment t of a stage: K-step 0 first, B before A
    const int h = t / NF, u = t % NF;
    if (u < TJ) xb[h * TJ + u] = fb.read(smem + RING_B + slot * B_BYTES, u, h);
    else        xa[h * TI + u - TJ] = fa.read(smem + slot * A_BYTES, u - TJ, h);
  };

  const int nst = (klen + PAIR_K - 1) / PAIR_K;
#pragma unroll
  for (int s = 0; s < NST; ++s) {
#pragma unroll
    for (int t = 0; t < LOADS; ++t) load_piece(t, s * PAIR_K, s);
    la.advance();
    lb.advance();
  }
  __builtin_amdgcn_s_waitcnt(waitcnt((NST - 1) * LOADS, 15));   // stage 0 has landed
  __syncthreads();
  v8i xa[2 * TI], xb[2 * TJ], ya[2 * TI], yb[2 * TJ];             // fragments of a whole stage (both K-steps), twice
#pragma unroll
  for (int t = 0; t < 2 * NF; ++t) read_one(t, 0, xa, xb);

  // Stage p, whose fragments are in ca / cb: the matrix instructions of its two K-steps, dealt out with the LDS reads of
  // the next stage's fragments (which have the rest of the stage to return) and the direct loads that refill its slot.
  auto stage = [&](auto slot, int p, const v8i* ca, const v8i* cb, v8i* na, v8i* nb) {
    constexpr int S = decltype(slot)::value, NEXT = (S + 1) % NST;
    // Stage p + 1 has landed (this wave's share: the younger stages may be in flight) and this wave has its fragments of
    // stage p; after the barrier that holds for all four, and the slot of stage p is refilled with stage p + NST (zeros past the end).
    __builtin_amdgcn_s_waitcnt(waitcnt((NST - 2) * LOADS, 0));
    __syncthreads();
    const int k0 = (p + NST) * PAIR_K;
    constexpr int SLOTS = 2 * NM, READS_PER = NM > 1 ? 1 : 2;
#pragma unroll
    for (int n = 0; n < SLOTS; ++n) {
      const int h = n / NM, i = (n % NM) / TJ, j = n % TJ;
      __builtin_amdgcn_sched_barrier(0);
      acc[i][j] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(cb[h * TJ + j], ca[h * TI + i], acc[i][j], FB, FA, 0, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = n * READS_PER; t < (n + 1) * READS_PER; ++t)
        if (t < 2 * NF) read_one(t, NEXT, na, nb);
#pragma unroll
      for (int t = n * LOADS / SLOTS; t < (n + 1) * LOADS / SLOTS; ++t) load_piece(t, k0, S);
    }
    __builtin_amdgcn_sched_barrier(0);
    la.advance();
    lb.advance();
  };
  // the ring slot and the fragment set of a stage are compile-time constants: the loop is unrolled over both
  constexpr int UNROLL = NST % 2 == 0 ? NST : 2 * NST;
  for (int p = 0; p < nst; p += UNROLL) {
#define FOG_STAGE(U)                                                                        \
  if (UNROLL > (U) && ((U) == 0 || p + (U) < nst)) {                                        \
    if ((U) % 2 == 0) stage(Int<(U) % NST>{}, p + (U), xa, xb, ya, yb);                     \
    else              stage(Int<(U) % NST>{}, p + (U), ya, yb, xa, xb);                     \
  }
    FOG_STAGE(0) FOG_STAGE(1) FOG_STAGE(2) FOG_STAGE(3) FOG_STAGE(4) FOG_STAGE(5)
#undef FOG_STAGE
  }
  __builtin_amdgcn_s_waitcnt(waitcnt(0, 0));   // no direct load may still be writing LDS: the ring becomes the staging area
  __syncthreads();

  if (g.splits > 1) {
    // the accumulators as they are, 1 KB per wave and store: float4 number (((item * 4 + w) * NM + TJ i + j) * 4 + qd) * 64 + l
    float4* dst = reinterpret_cast<float4*>(g.partial) + (int64_t)(item * 4 + w) * (NM * 256) + l;
#pragma unroll
    for (int i = 0; i < TI; ++i)
#pragma unroll
      for (int j = 0; j < TJ; ++j)
#pragma unroll
        for (int qd = 0; qd < 4; ++qd)
          dst[((i * TJ + j) * 4 + qd) * 64] = make_float4(acc[i][j][4 * qd + 0], acc[i][j][4 * qd + 1], acc[i][j][4 * qd + 2], acc[i][j][4 * qd + 3]);
    return;
  }

  // Epilogue: lane l holds rows wm + 32 i + (l & 31), columns wn + 32 j + 8 (r / 4) + 4 (l / 32) + (r % 4).  Blocks of
  // 32 x (32 JW) are scaled, converted and staged in the wave's own LDS, then stored as 16-byte pieces of whole rows.
  constexpr int JW = TJ >= 2 ? 2 : 1;
  constexpr int STRIDE = 64 * JW + (JW == 2 ? 8 : 16);
  constexpr int LPR = 4 * JW, RPS = 64 / LPR;    // lanes per row, rows per store instruction
  uint8_t* epi = smem + w * (32 * STRIDE);
  const int prow = l / LPR, piece = l % LPR;
#pragma unroll
  for (int i = 0; i < TI; ++i) {
#pragma unroll
    for (int jp = 0; jp < TJ / JW; ++jp) {
#pragma unroll
      for (int jj = 0; jj < JW; ++jj)
#pragma unroll
        for (int qd = 0; qd < 4; ++qd) {
          const v16f& x = acc[i][jp * JW + jj];
          *reinterpret_cast<uint2*>(epi + (l & 31) * STRIDE + 64 * jj + 16 * qd + 8 * (l >> 5)) =
              make_uint2(pack_bf16x2(x[4 * qd + 0] * alpha, x[4 * qd + 1] * alpha), pack_bf16x2(x[4 * qd + 2] * alpha, x[4 * qd + 3] * alpha));
        }
#pragma unroll
      for (int t = 0; t < 32 / RPS; ++t) {
        const uint2 lo = *reinterpret_cast<const uint2*>(epi + (RPS * t + prow) * STRIDE + 16 * piece);
        const uint2 hi = *reinterpret_cast<const uint2*>(epi + (RPS * t + prow) * STRIDE + 16 * piece + 8);
        const int m = m0 + wm + 32 * i + RPS * t + prow, n = n0 + wn + 32 * JW * jp + 8 * piece;
        if (m < g.M && n < g.N) store_row_piece(g, m, n, make_uint4(lo.x, lo.y, hi.x, hi.y));
      }
    }
  }
}

// Second pass of a split product: a workgroup owns one 32 x 32 block of C (the 256 float4 that one wave left there with four
// store instructions), adds the chunks in ascending order, scales, rounds once to bf16 and stores through LDS as row pieces.
__global__ __launch_bounds__(kThreads) void gemm_tile_reduce_kernel(GemmArgs g, int ti, int tj) {
  constexpr int STRIDE = 64 + 16;
  __shared__ __attribute__((aligned(16))) uint8_t blk[32 * STRIDE];
  const int ntiles = g.tiles_m * g.tiles_n, nm = ti * tj, per_tile = 4 * nm;
  const int logical = blockIdx.x / per_tile, sub = blockIdx.x - logical * per_tile;     // sub = w * nm + tj i + j
  const int w = sub / nm, ij = sub - w * nm, i = ij / tj, j = ij - i * tj;
  int m0, n0;
  tile_origin(logical, g.tiles_m, g.tiles_n, 64 * ti, 64 * tj, m0, n0);
  const int mb = m0 + (w >> 1) * 32 * ti + 32 * i, nb = n0 + (w & 1) * 32 * tj + 32 * j;   // origin of the block in C
  if (mb >= g.M || nb >= g.N) return;
  const int t = threadIdx.x, l = t & 63, qd = t >> 6;
  const float4* src = reinterpret_cast<const float4*>(g.partial) + ((int64_t)logical * per_tile + sub) * 256 + t;
  float4 acc = src[0];
#pragma unroll 4
  for (int c = 1; c < g.splits; ++c) {
    const float4 v = src[(int64_t)c * ntiles * per_tile * 256];
    acc.x += v.x; acc.y += v.y; acc.z += v.z; acc.w += v.w;
  }
  const float alpha = (*g.sinv_a) * (*g.sinv_b);
  *reinterpret_cast<uint2*>(blk + (l & 31) * STRIDE + 16 * qd + 8 * (l >> 5)) =
      make_uint2(pack_bf16x2(acc.x * alpha, acc.y * alpha), pack_bf16x2(acc.z * alpha, acc.w * alpha));
  __syncthreads();
  if (t < 128) {
    const int m = mb + (t >> 2), n = nb + 8 * (t & 3);
    if (m < g.M && n < g.N) store_row_piece(g, m, n, *reinterpret_cast<const uint4*>(blk + (t >> 2) * STRIDE + 16 * (t & 3)));
  }
}

template <int LAYOUT, int FA, int FB, int TI, int TJ, int NST, int WPS>
fog_status launch(GemmArgs g, hipStream_t s) {
  constexpr int LDS = NST * 64 * (TI + TJ) * PAIR_K;
  g.tiles_m = (g.M + 64 * TI - 1) / (64 * TI);
  g.tiles_n = (g.N + 64 * TJ - 1) / (64 * TJ);
  static bool configured = false;  // per instantiation; the attribute is sticky for the process
  if (!configured) {
    if (hipFuncSetAttribute(reinterpret_cast<const void*>(fp8_gemm_tile_kernel<LAYOUT, FA, FB, TI, TJ, NST, WPS>), hipFuncAttributeMaxDynamicSharedMemorySize, LDS) != hipSuccess)
      return FOG_ERR_HIP;
    configured = true;
  }
  const int grid = 8 * ((g.tiles_m * g.tiles_n * g.splits + 7) / 8);
  fp8_gemm_tile_kernel<LAYOUT, FA, FB, TI, TJ, NST, WPS><<<grid, kThreads, LDS, s>>>(g);
  if (g.splits > 1) gemm_reduce_launch(g, TI, TJ, s);
  return fog_launch_status();
}

template <int LAYOUT, int FA, int FB>
fog_status launch_tile(GemmTile tile, const GemmArgs& g, hipStream_t s) {
  switch (tile) {
    case TILE_256x128: return launch<LAYOUT, FA, FB, 4, 2, 3, 1>(g, s);
    case TILE_128x128: return launch<LAYOUT, FA, FB, 2, 2, 4, 1>(g, s);
    case TILE_128x128_2WG: return launch<LAYOUT, FA, FB, 2, 2, 2, 2>(g, s);
    default: return launch<LAYOUT, FA, FB, 1, 1, 4, 2>(g, s);
  }
}

template <int LAYOUT>
fog_status launch_fmt(GemmTile tile, int fa, int fb, const GemmArgs& g, hipStream_t s) {
  if (fa == FOG_E4M3) return fb == FOG_E4M3 ? launch_tile<LAYOUT, 0, 0>(tile, g, s) : launch_tile<LAYOUT, 0, 1>(tile, g, s);
  return fb == FOG_E4M3 ? launch_tile<LAYOUT, 1, 0>(tile, g, s) : launch_tile<LAYOUT, 1, 1>(tile, g, s);
}

}  // namespace

void gemm_reduce_launch(const GemmArgs& g, int ti, int tj, hipStream_t s) {
  gemm_tile_reduce_kernel<<<g.tiles_m * g.tiles_n * 4 * ti * tj, kThreads, 0, s>>>(g, ti, tj);
}

fog_status gemm_tile_launch(GemmTile tile, fog_layout layout, fog_fp8 fmt_a, fog_fp8 fmt_b, GemmArgs g, hipStream_t s) {
  switch (layout) {
    case FOG_NT: return launch_fmt<FOG_NT>(tile, fmt_a, fmt_b, g, s);
    case FOG_NN: return launch_fmt<FOG_NN>(tile, fmt_a, fmt_b, g, s);
    default: return launch_fmt<FOG_TN>(tile, fmt_a, fmt_b, g, s);
  }
}
