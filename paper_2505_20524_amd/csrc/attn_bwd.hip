// FP8 dot-product attention, backward (gfx950): dQ, dK, dV with all five products in FP8.
//
// The paper runs every GEMM of the block, attention included, in FP8 in both passes (abstract;
// Appendix E, FP8DPA row), with E5M2 for backward tensors (Section 2).  Per (batch, head):
//     D_i = sum_d dO_id O_id                        x_ij = s log2(e) sinv_q sinv_k (Q~ K~^T)_ij
//     P   = 2^(x - lse_i),  P~ = E4M3(rho_p P)      dV = sinv_do / rho_p (P~^T dO~)
//     dP  = sinv_do sinv_v (dO~ V~^T)               dS = P o (dP - D_i),  dS~ = E5M2(rho_ds dS)
//     dQ  = s sinv_k / rho_ds (dS~ K~)              dK = s sinv_q / rho_ds (dS~^T Q~)
//
// Two kernels.  (1) dQ: a workgroup owns 128 queries, sums their D_i from the bf16 tensors and walks the key blocks; it leaves
// two constants per row for the other kernel.  (2) dK/dV: a workgroup owns 64 keys and walks the query blocks at or below
// its diagonal.  Both produce the score tile with lane = query; its packed dS is then the B operand of
// dQ^T += K^T dS^T as it lies in the registers, and reaches lane = key, the B operand of dV^T += dO^T P and
// dK^T += Q^T dS, through a small exchange tile in LDS.  Recomputing S and dP in both kernels costs two extra
// products but keeps every accumulator in registers, needs no atomics and is deterministic.
// Operands whose contraction index is their row index (dO^T, Q^T, K^T) are gathered from the
// row-major LDS tiles with the byte-transposing read, in the order the packed scores have.
#include <cfloat>
#include <mutex>

#include "common.h"
#include "launch.h"

namespace {

constexpr int kThreads = 256;
constexpr int HD = 128;
constexpr int BLK = 128;           // queries owned by a workgroup of the dQ kernel
constexpr int STEP = 64;           // rows of the streamed operands per step
constexpr int TILE = STEP * HD;    // 8 KB, 16-byte chunks swizzled by swz(row)
constexpr int NSTAGE = 4;          // ring of the dQ kernel
constexpr uint32_t OOB = 0x80000000u;
// The ring stage of a block as a compile-time constant: the loops are unrolled over the ring so that every LDS address is a
// per-lane constant plus an immediate offset (a stage taken from the block number at run time costs an integer add per
// group of fragment reads).
template <int N> struct Stg { static constexpr int value = N; };

typedef __attribute__((address_space(3))) v2i* lds_v2i_ptr;

struct BwdArgs {
  const uint8_t* Q; const uint8_t* K; const uint8_t* V; const uint8_t* dO8;
  const uint16_t* O; const uint16_t* dO;
  const float* sinv_q; const float* sinv_k; const float* sinv_v; const float* sinv_do;
  const float* lse; const float* scale_p; const float* scale_ds;
  uint16_t* dQ; uint16_t* dK; uint16_t* dV;
  uint32_t* amax_ds; float* Dws;
  float softmax_scale;
  int BH, S, nblk;
  int BHkv, G;   // key/value heads in all, query heads per key/value head (grouped-query attention)
  int splits;    // dK/dV in turns: parts that a key block's stream of query blocks is cut into, each a workgroup's
  float4* partial;   // ... and where they leave their sums (splits > 1)
};

// LDS tiles are [64 rows][128 bytes]; the 16-byte chunks of a row sit at position chunk ^ swz(row).
// The key is a Gray code of the row: it is injective on any 8 (and, per row parity, 16) consecutive
// rows (16-byte row reads of 32 consecutive rows) and on the row sets {r..r+3, r+8..r+11} that one
// byte-transposing read touches, so both kinds of fragment read are bank-conflict free.
FOG_DEVICE int swz(int row) { return (row ^ (row >> 1)) & 7; }

FOG_DEVICE void load16_to_lds(v4i rsrc, uint32_t voff, uint32_t lds_addr_uniform) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, 0 offen lds"
               :
               : "v"(voff), "s"(rsrc), "s"(__builtin_amdgcn_readfirstlane((int)lds_addr_uniform))
               : "memory", "m0");
}
// ... from byte voff + soff
FOG_DEVICE void load16_to_lds(v4i rsrc, uint32_t voff, uint32_t soff, uint32_t lds_addr_uniform) {
  asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
               :
               : "v"(voff), "s"(rsrc), "s"(soff), "s"(lds_addr_uniform)
               : "memory", "m0");
}
FOG_DEVICE void load4_to_lds(v4i rsrc, uint32_t voff, uint32_t lds_addr_uniform) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tbuffer_load_dword %0, %1, 0 offen lds"
               :
               : "v"(voff), "s"(rsrc), "s"(__builtin_amdgcn_readfirstlane((int)lds_addr_uniform))
               : "memory", "m0");
}
FOG_DEVICE v4i make_rsrc(const void* base, uint32_t bytes) {
  const uint64_t b = reinterpret_cast<uint64_t>(base);
  v4i r;
  r[0] = (int)(uint32_t)b;
  r[1] = (int)((uint32_t)(b >> 32) & 0xFFFFu);
  r[2] = (int)bytes;
  r[3] = 0x00020000;
  return r;
}

// Per-lane byte offsets inside a tile, computed once per kernel.
struct RowFrag { uint32_t a[2][2]; };   // [h][chunk]: row (l & 31) (+ 32 per row tile: + 4096 bytes), chunks 4 h + 2 g, + 1
struct ColFrag { uint32_t a[4]; };      // [d]: transposing read 0 of head-dim tile d (+ 16 rows = 2048 bytes per read)
FOG_DEVICE RowFrag rowfrag_addr() {
  const int l = threadIdx.x & 63, g = l >> 5, row = l & 31;
  RowFrag f;
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    f.a[h][0] = (uint32_t)(row * HD + (((4 * h + 2 * g) ^ swz(row)) << 4));
    f.a[h][1] = (uint32_t)(row * HD + (((4 * h + 2 * g + 1) ^ swz(row)) << 4));
  }
  return f;
}
// Lane p of a 16-lane block addresses row 16 r + vrow (r = read number) and the 8-byte half (p & 1)
// of chunk 2 d + ((l & 16) >> 4); lane i of the block then receives column 32 d + (l & 16) + i of the
// rows 16 r + 8 (jj / 4) + 4 g + (jj % 4), jj = 0..7: the order in which the packed score bytes list them.
FOG_DEVICE ColFrag colfrag_addr() {
  const int l = threadIdx.x & 63, g = l >> 5, i16 = l & 15, jj = i16 >> 1;
  const int vrow = 8 * (jj >> 2) + 4 * g + (jj & 3);
  const int cbase = (l & 16) >> 4;
  ColFrag f;
#pragma unroll
  for (int d = 0; d < 4; ++d) f.a[d] = (uint32_t)(vrow * HD + (((2 * d + cbase) ^ swz(vrow)) << 4) + 8 * (i16 & 1));
  return f;
}
FOG_DEVICE v8i read_rowfrag(const uint8_t* tile, const RowFrag& f, int rt, int h) {
  v4i lo = *reinterpret_cast<const v4i*>(tile + f.a[h][0] + 4096 * rt);
  v4i hi = *reinterpret_cast<const v4i*>(tile + f.a[h][1] + 4096 * rt);
  v8i r;
  r[0] = lo[0]; r[1] = lo[1]; r[2] = lo[2]; r[3] = lo[3];
  r[4] = hi[0]; r[5] = hi[1]; r[6] = hi[2]; r[7] = hi[3];
  return r;
}
FOG_DEVICE v8i read_colfrag(const uint8_t* tile, const ColFrag& f, int d) {
  v8i r;
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    v2i v = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(tile + f.a[d] + 2048 * k));
    r[2 * k] = v[0];
    r[2 * k + 1] = v[1];
  }
  return r;
}
// Fragment of rows straight from global memory (row-major, stride HD): row, contraction bytes 64 h + 32 g.
FOG_DEVICE v8i frag_global(const uint8_t* base, int64_t row, int h) {
  const int l = threadIdx.x & 63;
  const uint8_t* p = base + row * HD + 64 * h + 32 * (l >> 5);
  uint4 lo = *reinterpret_cast<const uint4*>(p), hi = *reinterpret_cast<const uint4*>(p + 16);
  v8i f;
  f[0] = lo.x; f[1] = lo.y; f[2] = lo.z; f[3] = lo.w;
  f[4] = hi.x; f[5] = hi.y; f[6] = hi.z; f[7] = hi.w;
  return f;
}
// Direct-load offsets of a [64][128] tile: 2 pieces of 1 KB (8 rows) per wave; lane -> (row, global chunk).
FOG_DEVICE void tile_load_offsets(uint32_t* off) {
  const int l = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int row = 8 * (2 * w + j) + (l >> 3), cpos = l & 7;
    off[j] = (uint32_t)(row * HD + ((cpos ^ swz(row)) << 4));
  }
}

FOG_DEVICE float lane_xor32(float v) { return __shfl_xor(v, 32, 64); }

// D_i = sum_d dO_id O_id of 32 consecutive rows by one wave of the dQ kernel, before it walks the keys.  (As a kernel of its own, one
// pass over O and dO in front of the others, this took 27, 15 and 4 us at 2 x 32 heads x 4096, 4 x 16 x 2048 and 1 x 16/4 x 576; here
// its loads fly under other workgroups' matrix instructions: forward + backward with casts 781 -> 762, 265 -> 259, 55.6 -> 54.6 us.)
// Layout: sixteen lanes hold a row, four rows per load, the sums of lane l's row
// l & 31 come back through `park` (32 floats of LDS, the wave's own).  The exchange rotates within rows of 16 lanes by 8, 4, 2 and 1.
template <int N>
FOG_DEVICE float ror_add(float s) {
  return s + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(s), 0x120 + N, 0xF, 0xF, false));
}
FOG_DEVICE float row_dots(const uint16_t* __restrict__ O, const uint16_t* __restrict__ dO, float* park) {
  const int l = threadIdx.x & 63, at = (l >> 4) * HD + (l & 15) * 8;
  uint4 x[8], y[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    x[i] = ld_nt16(O + at + 4 * i * HD);
    y[i] = ld_nt16(dO + at + 4 * i * HD);
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint4 a = x[i], b = y[i];
    float s = bf16lo(a.x) * bf16lo(b.x) + bf16hi(a.x) * bf16hi(b.x) + bf16lo(a.y) * bf16lo(b.y) + bf16hi(a.y) * bf16hi(b.y) +
              bf16lo(a.z) * bf16lo(b.z) + bf16hi(a.z) * bf16hi(b.z) + bf16lo(a.w) * bf16lo(b.w) + bf16hi(a.w) * bf16hi(b.w);
    s = ror_add<1>(ror_add<2>(ror_add<4>(ror_add<8>(s))));
    if ((l & 15) == 0) park[4 * i + (l >> 4)] = s;
  }
  asm volatile("" ::: "memory");   // (a wave's LDS instructions complete in order)
  return park[l & 31];
}

// Largest magnitude among the 16 T values of a lane's T score tiles (NaN operands are dropped by the maximum), as 2 T
// independent chains, and the clamp of two tiles to the finite range of E5M2.
template <int T>
FOG_DEVICE float block_absmax(const v16f* x) {
  float cm[2 * T];
#pragma unroll
  for (int ch = 0; ch < 2 * T; ++ch) {
    const v16f& t = x[ch >> 1];
    const int b = 8 * (ch & 1);
    float m = fmaxf(fmaxf(fabsf(t[b]), fabsf(t[b + 1])), fabsf(t[b + 2]));
    m = fmaxf(fmaxf(m, fabsf(t[b + 3])), fabsf(t[b + 4]));
    m = fmaxf(fmaxf(m, fabsf(t[b + 5])), fabsf(t[b + 6]));
    cm[ch] = fmaxf(m, fabsf(t[b + 7]));
  }
#pragma unroll
  for (int ch = 1; ch < 2 * T; ++ch) cm[0] = fmaxf(cm[0], cm[ch]);
  return cm[0];
}
FOG_DEVICE void clamp_block(v16f* x) {
#pragma unroll
  for (int kt = 0; kt < 2; ++kt)
#pragma unroll
    for (int r = 0; r < 16; ++r) x[kt][r] = __builtin_amdgcn_fmed3f(x[kt][r], -57344.0f, 57344.0f);
}

// ------------------------------------------------------------------ dK, dV
// A workgroup of four waves owns 64 keys, a pair of waves 32 of them.  Of every block of 64 queries each wave of a pair takes 32
// through scores, dP, softmax and the casts (lane = query, so the row constants are one register per lane), and sums dV and dK
// over all 64 for its half of the head dimension.  The packed probabilities and dS travel between the two, and from lane = query
// to lane = key, through a 4 KB exchange tile in LDS that is written by rows and read with the byte-transposing read.
//
// Why pairs: dV and dK of 32 keys are 128 accumulator registers; with the score tiles and the keys' own fragments a wave that
// holds them all needs more than 256 registers and runs alone on its SIMD.  As two launches, one per output, S was computed
// twice; a pair holds 64 accumulators per wave, computes S and P once, and at 168 registers three workgroups share a CU.  What
// bounds the kernel is the vector ALU (exponential, dS, two casts per score), the matrix core close behind it (54 % and 47 % of the
// cycles); two barriers per block of queries are the price, which three independent workgroups hide.  Tried and slower: eight
// waves and 128 keys per workgroup (335 us), the products of one block dealt out between the vector work of the next inside the
// wave (311 us), a three-stage ring with one barrier and two workgroups per CU (318 us).
// Times of dK and dV, 2 x 32 heads x 4096 causal: 177 + 243 us as two launches -> 292 us, 286 us with the
// gradients stored as whole lines; whole backward there 622 -> 508 us, 4 x 16 x 2048 198 -> 146 us, 1 x 32/8 (grouped) x 4096 511 ->
// 296 us, 1 x 16/4 x 576 80 -> 33 us.
// Saturating converts (MODE.FP16_OVFL) would save the search for overflow in front of the cast of dS, 2 % of the backward (508
// against 518 us), but under that mode matrix instructions drop NaNs, and a diverged gradient left dK and dV finite.
//
// Ring stage: Q tile, dO tile, then 64 lse and 64 D values.  Five direct loads per thread and stage.
constexpr int KV_STAGE = 2 * TILE + 512;
constexpr int PAIR_THREADS = 256;
constexpr int PAIR_KEYS = 64;
constexpr int XCHG = 2 * 64 * 32;               // exchange tiles of a pair: P and dS, [64 queries][32 keys] each
constexpr int PAIR_STAGES = 2;
// Position of a key among the 32 bytes of an exchange row (and so the lane that ends up with it): a lane of the scores holds
// keys 8 qd + 4 g + b, and stores them as its 16 bytes 4 qd + b of half g.
FOG_DEVICE int key_of_position(int pos) { return 8 * ((pos >> 2) & 3) + 4 * (pos >> 4) + (pos & 3); }
// QSPLIT: both pairs own the same 32 keys and take the query blocks in turns, each through a ring of its own; the second pair's
// sums are added to the first's at the end.  Twice the workgroups and half the blocks in each, for launches that cannot fill the
// chip otherwise; a stage then serves 32 keys instead of 64.
template <bool CAUSAL, bool QSPLIT>
__global__ __launch_bounds__(PAIR_THREADS, QSPLIT ? 2 : 3) void attn_bwd_dkdv_kernel(BwdArgs a) {
  constexpr int KEYS = QSPLIT ? 32 : PAIR_KEYS, TURNS = QSPLIT ? 2 : 1;   // keys of a workgroup, pairs that share them
  constexpr int RING = PAIR_STAGES * KV_STAGE;                            // bytes of one ring
  __shared__ __attribute__((aligned(1024))) uint8_t smem[TURNS * RING + 2 * XCHG];
  const int S = a.S, G = a.G;
  const int wgs = a.BHkv * (S / KEYS);                 // workgroups of a part
  const int part = QSPLIT ? blockIdx.x / wgs : 0, bid = blockIdx.x - part * wgs;
  const int bhk = bid % a.BHkv;                        // key/value head; its query heads are bhk * G .. + G - 1
  const int kblk = bid / a.BHkv;                       // early key blocks see the most queries: launched first
  const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t >> 6), l = t & 63, g = l >> 5, pair = w >> 1, half = w & 1;
  const int64_t hoff = (int64_t)bhk * S;               // rows of this K/V head
  const int64_t qoff = hoff * G;                       // first row of the group's first query head
  const int key0 = kblk * KEYS + (QSPLIT ? 0 : 32 * pair);

  v8i kf[2], vf[2];                                    // the pair's 32 keys, both halves of d
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    kf[h] = frag_global(a.K + hoff * HD, key0 + (l & 31), h);
    vf[h] = frag_global(a.V + hoff * HD, key0 + (l & 31), h);
  }
  const float rho_p = *a.scale_p, rho_ds = *a.scale_ds;
  const float c = a.softmax_scale * 1.44269504088896340736f * (*a.sinv_q) * (*a.sinv_k);
  const float cdpk = (*a.sinv_do) * (*a.sinv_v) * (rho_ds / rho_p);   // dP scale times rho_ds / rho_p

  v16f dv[2], dk[2];
#pragma unroll
  for (int d = 0; d < 2; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) { dv[d][r] = 0.0f; dk[d][r] = 0.0f; }

  const int qb_first = CAUSAL ? key0 / STEP : 0;       // the diagonal block comes first
  const int nqb = S / STEP - qb_first;                 // query blocks of one head this workgroup walks
  // ... and of the whole group: head after head, one stream, of which this workgroup takes blocks `begin` to `end`
  const int begin = QSPLIT ? nqb * G * part / a.splits : 0, end = QSPLIT ? nqb * G * (part + 1) / a.splits : nqb * G;

  const uint32_t group_bytes = (uint32_t)G * S * HD;
  const v4i rsrc_q = make_rsrc(a.Q + qoff * HD, group_bytes), rsrc_do = make_rsrc(a.dO8 + qoff * HD, group_bytes);
  const int64_t nrows = (int64_t)a.BH * S;
  const v4i rsrc_lse = make_rsrc(a.Dws + 2 * nrows + qoff, (uint32_t)G * S * 4), rsrc_d = make_rsrc(a.Dws + nrows + qoff, (uint32_t)G * S * 4);
  // direct loads: the waves that share a ring fetch NP pieces (8 rows each) of Q and of dO each per block, and the 64 row constants
  // (even waves lse, odd waves D; four waves leave two copies each, identical bytes)
  constexpr int NP = 2 * TURNS, LOADS = 2 * NP + 1;
  const int lw = QSPLIT ? half : w;                    // number of this wave among those of its ring
  uint32_t off[NP];
#pragma unroll
  for (int j = 0; j < NP; ++j) {
    const int row = 8 * (NP * lw + j) + (l >> 3);
    off[j] = (uint32_t)(row * HD + (((l & 7) ^ swz(row)) << 4));
  }
  uint8_t* ring = smem + (QSPLIT ? pair * RING : 0);
  const uint32_t lds0 = (uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(uintptr_t)ring);
  const uint32_t lds_w = lds0 + 1024u * NP * (uint32_t)lw;
  const bool rows_d = w & 1;
  // query block and head of the next block to issue (issue() is called once per block, in order); a pair that takes turns starts
  // at its own and skips the other's
  int iss_i = QSPLIT ? begin % nqb : 0, iss_g = QSPLIT ? begin / nqb : 0, iss_at = begin + (QSPLIT ? pair : 0);
  auto next_block = [&](int& i, int& head) { if (++i == nqb) { i = 0; ++head; } };
  if (QSPLIT && pair) next_block(iss_i, iss_g);
  int cur_i = iss_i;          // query block (within its head) of the block in hand
  auto issue = [&](auto stg) {  // the next block of the stream -> stage stg; blocks past the end fetch zeros
    const uint32_t row0 = (uint32_t)(iss_g * S + (qb_first + iss_i) * STEP);
    const uint32_t adv = iss_at < end ? row0 * HD : OOB;
    const uint32_t radv = iss_at < end ? row0 * 4 : OOB;
    const uint32_t base = (uint32_t)decltype(stg)::value * KV_STAGE;
#pragma unroll
    for (int j = 0; j < NP; ++j) {
      load16_to_lds(rsrc_q, off[j] + adv, lds_w + base + 1024u * j);
      load16_to_lds(rsrc_do, off[j] + adv, lds_w + base + TILE + 1024u * j);
    }
    load4_to_lds(rows_d ? rsrc_d : rsrc_lse, (uint32_t)(4 * l) + radv, lds0 + base + 2 * TILE + (rows_d ? 256u : 0u));
#pragma unroll
    for (int n = 0; n < TURNS; ++n) next_block(iss_i, iss_g);
    iss_at += TURNS;
  };
  // fragment addresses: rows of this wave's 32 queries; columns of its half of the head dimension, read r of the transposing
  // read covering queries 16 r + 8 g .. + 7 (the swizzle does not change from read to read); the exchange tiles in that order
  RowFrag rf = rowfrag_addr();
#pragma unroll
  for (int h = 0; h < 2; ++h) { rf.a[h][0] += 4096u * half; rf.a[h][1] += 4096u * half; }
  const int crow = 8 * g + ((l & 15) >> 1);
  uint32_t ca[2];
#pragma unroll
  for (int d = 0; d < 2; ++d) ca[d] = (uint32_t)(crow * HD + (((4 * half + 2 * d + ((l & 16) >> 4)) ^ swz(crow)) << 4) + 8 * (l & 1));
  const uint8_t* xbase = smem + TURNS * RING + pair * XCHG;   // + 2048 for dS
  // (the 16-byte halves of an exchange row trade places with bit 3 of the row: one read touches rows 0..7 and 8..15 together)
  const uint8_t* xread = xbase + crow * 32 + ((l & 16) ^ (16 * g)) + 8 * (l & 1);
  uint8_t* xwrite = const_cast<uint8_t*>(xbase) + (32 * half + (l & 31)) * 32 + ((16 * g) ^ (2 * (l & 8)));
  const uint32_t row_const = 2 * TILE + 4 * (32 * half + (l & 31));           // lse - log2 rho_p; + 256: D rho_ds / rho_p
  const int q_rel = qb_first * STEP + 32 * half + (l & 31) - key0 - 4 * g;    // this lane's query of the diagonal block against key register 0

  FOG_SETTLE(kf[0]); FOG_SETTLE(kf[1]); FOG_SETTLE(vf[0]); FOG_SETTLE(vf[1]);
  issue(Stg<0>{});
  issue(Stg<1>{});

  auto colfrag = [&](const uint8_t* tile, int d) {
    v8i f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const v2i v = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(tile + ca[d] + 2048 * r));
      f[2 * r] = v[0];
      f[2 * r + 1] = v[1];
    }
    return f;
  };
  auto packed = [&](int which) {   // 0: P~, 1: dS~ of a block of 64 queries, lane = key position
    v8i f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const v2i v = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_v2i_ptr)(xread + 2048 * which + 512 * r));
      f[2 * r] = v[0];
      f[2 * r + 1] = v[1];
    }
    return f;
  };
  auto clear = [&](v16f& x) {
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = 0.0f;
  };

  __builtin_amdgcn_s_waitcnt(0x0F70 | LOADS);   // vmcnt = LOADS: block 0 has landed
  __syncthreads();
  auto block = [&](const bool CLAMP_P, auto stg) __attribute__((always_inline)) {
    constexpr int STG = decltype(stg)::value;
    const uint8_t* sq = ring + STG * KV_STAGE;
    const uint8_t* sdo = sq + TILE;
    const float lse = *reinterpret_cast<const float*>(sq + row_const);
    // A row whose output gradient holds an infinity has an infinite D, and 0 times that is no number: where P is 0 its dS is 0
    // (a NaN stays).
    const float D_row = *reinterpret_cast<const float*>(sq + row_const + 256);
    const float Dq = fabsf(D_row) > FLT_MAX ? __builtin_copysignf(FLT_MAX, D_row) : D_row;
    v16f st, dp;
    clear(st); clear(dp);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      st = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(kf[h], read_rowfrag(sq, rf, 0, h), st, 0, 0, 0, 0, 0, 0);
      dp = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(vf[h], read_rowfrag(sdo, rf, 0, h), dp, 0, 1, 0, 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    uint32_t pk[4], dsk[4];
#pragma unroll
    for (int qd = 0; qd < 4; ++qd) {
      float p[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = 4 * qd + e;
        p[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(st[r], c, -lse));          // rho_p P
        dp[r] = p[e] * __builtin_fmaf(dp[r], cdpk, -Dq);                        // rho_ds dS, left in the registers of dP
        if (CLAMP_P) p[e] = p[e] > 448.0f ? 448.0f : p[e];                      // (a NaN stays)
      }
      const uint32_t lo = __builtin_amdgcn_cvt_pk_fp8_f32(p[0], p[1], any_u32(), false);
      pk[qd] = __builtin_amdgcn_cvt_pk_fp8_f32(p[2], p[3], lo, true);
    }
    // The hardware convert turns overflow into infinity: dS is clamped before its cast where the block holds a magnitude above the
    // largest finite E5M2 value (finding that out costs half an instruction per value, the clamp three; a NaN stays).
    if (__builtin_expect(__any(block_absmax<1>(&dp) > 57344.0f), 0)) {
#pragma unroll
      for (int r = 0; r < 16; ++r) dp[r] = fabsf(dp[r]) > 57344.0f ? __builtin_copysignf(57344.0f, dp[r]) : dp[r];
    }
#pragma unroll
    for (int qd = 0; qd < 4; ++qd) {
      const uint32_t lo = __builtin_amdgcn_cvt_pk_bf8_f32(dp[4 * qd], dp[4 * qd + 1], any_u32(), false);
      dsk[qd] = __builtin_amdgcn_cvt_pk_bf8_f32(dp[4 * qd + 2], dp[4 * qd + 3], lo, true);
    }
    if (CAUSAL && cur_i == 0) {
      // The first query block of every head is the diagonal one (KEYS divides STEP): a query sees nothing of the keys after it.
      // The codes of those are cleared here, whatever the exponential of a score that has no place in its row became.
      int q = q_rel;
      asm volatile("" : "+v"(q));           // the masks are made here, not kept in registers over the loop
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        const int n = q - 8 * qd + 1;       // keys 8 qd .. 8 qd + n - 1 count
        const uint32_t m = n <= 0 ? 0u : n >= 4 ? 0xFFFFFFFFu : (1u << (8 * n)) - 1u;
        pk[qd] &= m;
        dsk[qd] &= m;
      }
    }
#pragma unroll
    for (int n = 0; n < TURNS; ++n) cur_i = cur_i + 1 == nqb ? 0 : cur_i + 1;
    *reinterpret_cast<uint4*>(xwrite) = make_uint4(pk[0], pk[1], pk[2], pk[3]);
    *reinterpret_cast<uint4*>(xwrite + 2048) = make_uint4(dsk[0], dsk[1], dsk[2], dsk[3]);
    __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt = 0
    __syncthreads();                      // both halves of the block are in the exchange tiles
    const v8i pf = packed(0), dsf = packed(1);
    const v8i o0 = colfrag(sdo, 0), q0 = colfrag(sq, 0), o1 = colfrag(sdo, 1), q1 = colfrag(sq, 1);
    __builtin_amdgcn_s_waitcnt(0x0070);   // every fragment of this block is in registers, block it + 1 has landed
    __syncthreads();
    issue(stg);                           // block it + 2, into the stage of this block
    dv[0] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(o0, pf, dv[0], 1, 0, 0, 0, 0, 0);
    dk[0] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(q0, dsf, dk[0], 0, 1, 0, 0, 0, 0);
    dv[1] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(o1, pf, dv[1], 1, 0, 0, 0, 0, 0);
    dk[1] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(q1, dsf, dk[1], 0, 1, 0, 0, 0, 0);
  };
  // Blocks of a pair (one past the end is a block of zeros: P is 1 there, but dO, D and dP are 0 and add nothing).
  const int turns = (end - begin + TURNS - 1) / TURNS;
  // two blocks per trip: the ring stage is a constant in each copy
  auto trips = [&](const bool CLAMP_P) __attribute__((always_inline)) {
    for (int it = 0; it < turns; it += PAIR_STAGES) {
      block(CLAMP_P, Stg<0>{});
      if (it + 1 < turns) block(CLAMP_P, Stg<1>{});
    }
  };
  if (!(rho_p <= 448.0f)) trips(true);   // rho_p P <= rho_p: the cast of P only overflows under a scale above the format's maximum
  else                    trips(false);
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): no direct load may still be writing LDS when the workgroup retires
  if (QSPLIT) {
    // the second pair's sums through LDS (both rings are done with): 16 bytes per lane and instruction
    float4* part = reinterpret_cast<float4*>(smem) + half * (16 * 64) + l;
    static_assert(2 * 16 * 64 * 16 <= TURNS * RING || !QSPLIT, "the sums of two waves fit the rings");
    __syncthreads();
    if (pair) {
#pragma unroll
      for (int d = 0; d < 2; ++d)
#pragma unroll
        for (int qd = 0; qd < 4; ++qd) {
          part[(8 * d + qd) * 64] = make_float4(dv[d][4 * qd], dv[d][4 * qd + 1], dv[d][4 * qd + 2], dv[d][4 * qd + 3]);
          part[(8 * d + 4 + qd) * 64] = make_float4(dk[d][4 * qd], dk[d][4 * qd + 1], dk[d][4 * qd + 2], dk[d][4 * qd + 3]);
        }
    }
    __syncthreads();
    if (pair) return;
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        const float4 x = part[(8 * d + qd) * 64], y = part[(8 * d + 4 + qd) * 64];
        dv[d][4 * qd] += x.x; dv[d][4 * qd + 1] += x.y; dv[d][4 * qd + 2] += x.z; dv[d][4 * qd + 3] += x.w;
        dk[d][4 * qd] += y.x; dk[d][4 * qd + 1] += y.y; dk[d][4 * qd + 2] += y.z; dk[d][4 * qd + 3] += y.w;
      }
  }
  const float sdv = (*a.sinv_do) / rho_p;
  const float sdk = a.softmax_scale * (*a.sinv_q) / rho_ds;
  if (!QSPLIT) __syncthreads();   // every wave's direct loads have landed: the rings become the staging areas
  uint8_t* stage = QSPLIT ? smem + half * (16 * 64 * 16) : smem + w * (32 * 144);   // split: where this wave has read its partner's sums
  const int64_t out0 = (hoff + key0) * HD + 64 * half;
  if (QSPLIT && a.splits > 1) {   // binary32, as they are: attn_bwd_dkdv_sum_kernel adds the parts
    float4* part_sums = a.partial + ((int64_t)blockIdx.x * 2 + half) * (16 * 64) + l;
#pragma unroll
    for (int d = 0; d < 2; ++d)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        part_sums[(4 * d + qd) * 64] = make_float4(dv[d][4 * qd], dv[d][4 * qd + 1], dv[d][4 * qd + 2], dv[d][4 * qd + 3]);
        part_sums[(8 + 4 * d + qd) * 64] = make_float4(dk[d][4 * qd], dk[d][4 * qd + 1], dk[d][4 * qd + 2], dk[d][4 * qd + 3]);
      }
  } else {
  // Stored as 8-byte pieces straight from the registers, the three gradients (200 MB at 2 x 32 heads x 4096) stay in the caches as
  // dirty lines that leave them during whatever runs next: the abs-max pass after it took 60 us instead of 50, the forward 180
  // instead of 172.  Pieces stored past the caches are worse still: a line then goes to memory in parts (this kernel + 100 us).
  store_tile_rows<2>(stage, dv, sdv, a.dV + out0, HD, [](int pos) { return key_of_position(pos); });
  store_tile_rows<2>(stage, dk, sdk, a.dK + out0, HD, [](int pos) { return key_of_position(pos); });
  }
  if (a.amax_ds && w == 0) {
    // this workgroup's share of the maxima that the dQ kernel left, one per 32 rows
    const int64_t n = nrows / 32, per = (n + gridDim.x - 1) / gridDim.x, first = per * blockIdx.x, last = first + per < n ? first + per : n;
    float m = 0.0f;
    for (int64_t i = first + l; i < last; i += 64) m = fmaxf(m, a.Dws[i]);
    m = wave_max_f32(m);
    // only a wave that would raise the maximum pays for the atomic (a stale read can only be too small)
    if (l == 0 && m > 0.0f && __float_as_uint(m) > __hip_atomic_load(a.amax_ds, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(a.amax_ds, __float_as_uint(m));
  }
}

// The sums of a split dK/dV launch: workgroup n adds the parts of 32 keys in ascending order, scales and rounds once; a wave has one
// half of the head dimension of dV (waves 0, 1) or dK (2, 3), in the layout of the accumulators.
__global__ __launch_bounds__(256) void attn_bwd_dkdv_sum_kernel(BwdArgs a) {
  __shared__ __attribute__((aligned(16))) uint8_t smem[4 * 32 * 144];
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63, half = w & 1, which = w >> 1;
  const int wgs = (int)gridDim.x, bid = (int)blockIdx.x;
  const float4* src = a.partial + ((int64_t)bid * 2 + half) * (16 * 64) + which * (8 * 64) + l;
  v16f x[2];
  float4 v[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) v[i] = src[64 * i];
  for (int n = 1; n < a.splits; ++n) {
    src += (int64_t)wgs * (2 * 16 * 64);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float4 y = src[64 * i];
      v[i].x += y.x; v[i].y += y.y; v[i].z += y.z; v[i].w += y.w;
    }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    x[i >> 2][4 * (i & 3)] = v[i].x; x[i >> 2][4 * (i & 3) + 1] = v[i].y;
    x[i >> 2][4 * (i & 3) + 2] = v[i].z; x[i >> 2][4 * (i & 3) + 3] = v[i].w;
  }
  const float scale = which ? a.softmax_scale * (*a.sinv_q) / (*a.scale_ds) : (*a.sinv_do) / (*a.scale_p);
  const int64_t out0 = ((int64_t)(bid % a.BHkv) * a.S + 32 * (bid / a.BHkv)) * HD + 64 * half;
  store_tile_rows<2>(smem + w * (32 * 144), x, scale, (which ? a.dK : a.dV) + out0, HD, [](int pos) { return key_of_position(pos); });
}

// ------------------------------------------------------------------ dQ (and max |dS|), and the constants of its rows
// ws[1][row] = D_i * rho_ds / rho_p    (for the dK/dV kernel: its probabilities carry the factor rho_p)
// ws[2][row] = lse_i - log2 rho_p      (for the dK/dV kernel: 2^(x - that) = rho_p P)
// ws[0][n]   = max |dS| of the n-th 32 rows, for the dK/dV kernel to reduce (one word raised by every wave of this launch would have
//              to be cleared by a launch before it)
// Folding the scales into per-row constants once saves three vector instructions per score.
template <bool CAUSAL, bool AMAX>
__global__ __launch_bounds__(kThreads, 2) void attn_bwd_dq_kernel(BwdArgs a) {
  __shared__ __attribute__((aligned(1024))) uint8_t smem[NSTAGE * 2 * TILE];     // {K, V} x 4 stages
  const int bh = blockIdx.x % a.BH;
  const int qblk = a.nblk - 1 - blockIdx.x / a.BH;
  const int t = threadIdx.x, w = __builtin_amdgcn_readfirstlane(t >> 6), l = t & 63, g = l >> 5;
  const int S = a.S;
  const int64_t hoff = (int64_t)bh * S;
  const int q0 = qblk * BLK + 32 * w;
  const int q = q0 + (l & 31);
  const bool wave_on = q0 < S;

  v8i qf[2], dof[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    qf[h] = frag_global(a.Q + hoff * HD, wave_on ? q : 0, h);
    dof[h] = frag_global(a.dO8 + hoff * HD, wave_on ? q : 0, h);
  }
  const float rho_ds = *a.scale_ds, rho_p = *a.scale_p;
  const float lse_row = wave_on ? a.lse[hoff + q] : 0.0f;
  const float lse = lse_row - __log2f(rho_ds);   // 2^(x - this) = rho_ds P
  const float c = a.softmax_scale * 1.44269504088896340736f * (*a.sinv_q) * (*a.sinv_k);
  const float cdp = (*a.sinv_do) * (*a.sinv_v);

  v16f dq[4];
#pragma unroll
  for (int d = 0; d < 4; ++d)
#pragma unroll
    for (int r = 0; r < 16; ++r) dq[d][r] = 0.0f;
  float ds_max = 0.0f;

  const int kv_end = CAUSAL ? min(S, qblk * BLK + BLK) : S;
  const int nkb = (kv_end + STEP - 1) / STEP;
  const int nkb_wave = !wave_on ? 0 : (CAUSAL ? min(nkb, (q0 + 31) / STEP + 1) : nkb);

  const uint32_t head_bytes = (uint32_t)S * HD;
  const int64_t kvoff = (int64_t)(bh / a.G) * S;   // the G query heads of a group are consecutive and share one K/V head
  const v4i rsrc_k = make_rsrc(a.K + kvoff * HD, head_bytes), rsrc_v = make_rsrc(a.V + kvoff * HD, head_bytes);
  uint32_t off[2];
  tile_load_offsets(off);
  const uint32_t lds_w = (uint32_t)__builtin_amdgcn_readfirstlane((int)((uint32_t)(uintptr_t)smem + 2048u * w));
  auto issue = [&](int kb, auto stg) {   // block kb -> stage kb % NSTAGE = stg
    const uint32_t adv = (uint32_t)(kb < nkb ? kb : nkb - 1) * (STEP * HD);   // (past the end the last block once more: nothing reads it)
    const uint32_t base = lds_w + (uint32_t)decltype(stg)::value * (2 * TILE);
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      load16_to_lds(rsrc_k, off[j], adv, base + 1024u * j);
      load16_to_lds(rsrc_v, off[j], adv, base + TILE + 1024u * j);
    }
  };
  const RowFrag rf = rowfrag_addr();
  const ColFrag cf = colfrag_addr();

  issue(0, Stg<0>{});
  issue(1, Stg<1>{});
  issue(2, Stg<2>{});
  // The rows' D, under the flight of the first key blocks (stage 3 of the ring is free until the barrier below).
  float Dq = 0.0f;
  if (wave_on) {
    Dq = row_dots(a.O + (hoff + q0) * HD, a.dO + (hoff + q0) * HD, reinterpret_cast<float*>(smem + 3 * 2 * TILE) + 32 * w);
    if (g == 0) {
      const int64_t nrows = (int64_t)a.BH * S;
      a.Dws[nrows + hoff + q] = Dq * (rho_ds / rho_p);
      a.Dws[2 * nrows + hoff + q] = lse_row - __log2f(rho_p);
    }
  }
  if (AMAX && blockIdx.x == 0 && t == 0) *a.amax_ds = 0u;   // raised by the dK/dV kernel, from the maxima left below
  FOG_SETTLE(qf[0]); FOG_SETTLE(qf[1]); FOG_SETTLE(dof[0]); FOG_SETTLE(dof[1]); FOG_SETTLE(lse); FOG_SETTLE(Dq);
  __builtin_amdgcn_s_waitcnt(0x0F78);  // vmcnt = 8: block 0 has landed (4 direct loads per thread and block)
  __syncthreads();

  // One of the four matrix instructions of a block's scores (or, on V and dO, of its dP): tile n / 2, half n % 2 of the head dimension.
  auto clear16 = [&](v16f& x) __attribute__((always_inline)) {
#pragma unroll
    for (int r = 0; r < 16; ++r) x[r] = 0.0f;
  };
  auto score = [&](v16f* st, int n, v8i f) __attribute__((always_inline)) {
    if ((n & 1) == 0) clear16(st[n >> 1]);
    st[n >> 1] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(f, qf[n & 1], st[n >> 1], 0, 0, 0, 0, 0, 0);
  };
  // The wave overlaps the two units by itself as well: dP of block kb is produced under its exponentials, the scores of block kb + 1 while its dS are
  // formed, and every operand is read from LDS one matrix instruction ahead.  (All eight products in front of the vector part before, and
  // uniform load offsets in vector registers: 4 x 16 x 2048 73.5 -> 69.2 us.  The whole backward, us, before / offsets alone / order alone / both:
  // 4 x 16 x 2048 155.0 / 153.6 / 146.9 / 148.5, 1 x 4 x 8192 208 / 209 / 197 / 198, 2 x 32 x 4096 501 / 498 / 501 / 504.  Where four rounds of workgroups keep every
  // wave slot busy the clock is what gives, and it is half a percent to one behind: 1 x 32/8 x 8192 955 -> 962, 8 x 32/8 x 1024 173.0 -> 175.0; two
  // rounds are ahead: 8 x 16 x 1024 97.5 -> 95.2, 2 x 32/8 x 2048 not causal 290 -> 284.)
  auto block = [&](int kb, v16f* st, v16f* next, auto stg) __attribute__((always_inline)) {
    constexpr int STG = decltype(stg)::value;
    __builtin_amdgcn_s_waitcnt(0x0074);  // vmcnt = 4: block kb + 1 landed (block kb + 2 may be in flight); lgkmcnt = 0
    __syncthreads();
    issue(kb + 3, Stg<(STG + 3) % NSTAGE>{});   // into the stage of block kb - 1
    if (kb >= nkb_wave) return;
    const uint8_t* sk = smem + STG * (2 * TILE);
    const uint8_t* sv = sk + TILE;
    const int kbase = kb * STEP;
    // transposed tiles, lane = query: element r of tile kt is key kbase + 32 kt + 8 (r/4) + 4 g + (r%4)
    if (CAUSAL && kbase + STEP - 1 > q0) {   // diagonal blocks: keys after the query are masked
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int r = 0; r < 16; ++r)
          if (kbase + 32 * kt + 8 * (r >> 2) + 4 * g + (r & 3) > q) st[kt][r] = -INFINITY;
    }
    v16f dp[2];
    const uint8_t* sn = smem + (STG + 1) % NSTAGE * (2 * TILE);
    auto frag = [&](int n) __attribute__((always_inline)) {   // operands in the order of the matrix instructions below, each read one of them ahead
      return n < 4 ? read_rowfrag(sv, rf, n >> 1, n & 1) : n < 8 ? read_rowfrag(sn, rf, (n >> 1) & 1, n & 1) : read_colfrag(sk, cf, n & 3);
    };
    v8i f[2];
    f[0] = frag(0);
#pragma unroll
    for (int n = 0; n < 8; ++n) {
      const int kt = (n >> 1) & 1, h = n & 1;
      __builtin_amdgcn_sched_barrier(0);
      if (n < 4) {
        if (h == 0) clear16(dp[kt]);
        dp[kt] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(f[n & 1], dof[h], dp[kt], 0, 1, 0, 0, 0, 0);
      } else {
        score(next, n & 3, f[n & 1]);   // (past the wave's last block: of no use, and nothing reads it)
      }
      f[(n + 1) & 1] = frag(n + 1);
      __builtin_amdgcn_sched_barrier(0);
      // rho_ds P under the products of dP, then rho_ds dS = (rho_ds P) (dP - D), left in the registers of dP
#pragma unroll
      for (int r = 8 * h; r < 8 * h + 8; ++r) {
        if (n < 4) st[kt][r] = __builtin_amdgcn_exp2f(__builtin_fmaf(st[kt][r], c, -lse));
        else       dp[kt][r] = st[kt][r] * __builtin_fmaf(dp[kt][r], cdp, -Dq);
      }
    }
    f[1] = frag(9);
    const float bm = block_absmax<2>(dp);
    ds_max = fmaxf(ds_max, bm);
    // The hardware convert turns overflow into infinity, so magnitudes above the largest finite E5M2 value have to be clamped
    // first; whether any of the block's 32 values per lane needs that is known from the block maximum (which the abs-max of dS
    // wants anyway), and with a scale fitted to the tensor none does: the clamp (one instruction per value) runs only then.
    if (__builtin_expect(__any(bm > 57344.0f), 0)) clamp_block(dp);
    v8i dsf;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd) {
        const uint32_t pk = __builtin_amdgcn_cvt_pk_bf8_f32(dp[kt][4 * qd + 0], dp[kt][4 * qd + 1], any_u32(), false);
        dsf[4 * kt + qd] = (int)__builtin_amdgcn_cvt_pk_bf8_f32(dp[kt][4 * qd + 2], dp[kt][4 * qd + 3], pk, true);
      }
    // dQ^T += K^T dS~^T  (contraction over the 64 keys of this step)
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      dq[d] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(f[d & 1], dsf, dq[d], 0, 1, 0, 0, 0, 0);
      if (d < 2) f[d & 1] = frag(10 + d);
    }
  };
  static_assert(NSTAGE == 4, "the loops are unrolled over a ring of four stages");
  v16f sa[2], sb[2];
#pragma unroll
  for (int n = 0; n < 4; ++n) score(sa, n, read_rowfrag(smem, rf, n >> 1, n & 1));
  for (int kb = 0; kb < nkb; kb += NSTAGE) {
    block(kb, sa, sb, Stg<0>{});
    if (kb + 1 < nkb) block(kb + 1, sb, sa, Stg<1>{});
    if (kb + 2 < nkb) block(kb + 2, sa, sb, Stg<2>{});
    if (kb + 3 < nkb) block(kb + 3, sb, sa, Stg<3>{});
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): no direct load may still be writing LDS when the workgroup retires
  __syncthreads();                     // ... of any wave: the ring becomes the staging area
  if (!wave_on) return;
  const float sdq = a.softmax_scale * (*a.sinv_k) / rho_ds;
  store_tile_rows<4>(smem + w * (32 * 272), dq, sdq, a.dQ + (hoff + q0) * HD, HD, [](int row) { return row; });
  if (AMAX) {
    ds_max = wave_max_f32(ds_max) / rho_ds;   // the running maximum was taken on rho_ds dS
    if (l == 0) a.Dws[(hoff + q0) / 32] = ds_max;
  }
}

__global__ void zero_u32b(uint32_t* p) { *p = 0u; }

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

// Parts that the query blocks of every 32 keys are cut into for the dK/dV kernel in turns: as many as two workgroups per CU allow,
// each of kSplitBlocks blocks or more where the stream is longest, because the sums of the parts cost a launch and a pass over memory.
// A launch of few workgroups takes what its longest one takes, 0.43 us a block, while other CUs idle.  Backward of B x H/H_kv heads x S,
// us, whole streams -> parts: 1 x 16/4 x 576 32.8 -> 28.9 (two parts; three of 12 blocks 32.9), 1 x 8/2 x 1024 50.0 -> 36.5, 1 x 4/1 x 2048
// 87.6 -> 56.4, 1 x 2/2 x 2048 50.0 -> 48.2, 1 x 1/1 x 4096 not causal 84.6 -> 77.2; two parts of 8 blocks each lose: 1 x 4/4 x 1024
// 30.5 -> 31.6.  Two workgroups per CU against one: 1 x 4/1 x 4096 119.0 -> 110.6, 1 x 16/4 x 2048 89.7 -> 83.7.  (Four pairs in turns inside one workgroup instead gain nothing: two waves on a SIMD take twice the time for a block each.)
constexpr int kSplitBlocks = 16, kSplitsMost = 8;
static int kv_splits(int64_t BHkv, int S, int G, int cus) {
  const int64_t wgs = BHkv * (S / 32), longest = (int64_t)(S / STEP) * G;
  const int64_t room = 2 * cus / wgs, p = room < longest / kSplitBlocks ? room : longest / kSplitBlocks;
  return p < 2 ? 1 : p < kSplitsMost ? (int)p : kSplitsMost;
}
// Bytes of the three constants per row, and of the parts' sums behind them.
static size_t rows_bytes(int B, int H, int S) { return (size_t)3 * B * H * S * sizeof(float); }
static size_t parts_bytes(int splits, int B, int H_kv, int S) { return splits > 1 ? (size_t)splits * 2 * B * H_kv * S * HD * sizeof(float) : 0; }

extern "C" size_t fog_fp8_attn_workspace(int B, int H, int H_kv, int S, int D, int is_bwd) {
  if (!is_bwd || B <= 0 || H <= 0 || S <= 0) return 0;
  if (D != HD || S % STEP != 0 || H_kv <= 0 || H % H_kv != 0) return rows_bytes(B, H, S);   // refused by the call
  return rows_bytes(B, H, S) + parts_bytes(kv_splits((int64_t)B * H_kv, S, H / H_kv, fog_compute_units()), B, H_kv, S);
}

// Argument checks shared by the two entry points (everything but the workspace); FOG_OK with *empty set
// means there is nothing to compute.
static fog_status bwd_checks(int B, int H, int H_kv, int S, int D, float softmax_scale,
                             const uint8_t* Q, const uint8_t* K, const uint8_t* V,
                             const float* sinv_q, const float* sinv_k, const float* sinv_v,
                             const void* O_bf16, const void* dO_bf16, const uint8_t* dO_e5m2, const float* sinv_do,
                             const float* lse, const float* scale_p, const float* scale_ds,
                             void* dQ_bf16, void* dK_bf16, void* dV_bf16, bool* empty) {
  *empty = false;
  if (B < 0 || H < 0 || H_kv < 0 || S < 0 || D < 0) return FOG_ERR_SHAPE;
  if ((H > 0) != (H_kv > 0) || (H_kv > 0 && H % H_kv != 0)) return FOG_ERR_SHAPE;
  if (!(softmax_scale > 0.0f)) return FOG_ERR_UNSUPPORTED;
  if (D != HD || S % STEP != 0) return FOG_ERR_UNSUPPORTED;
  if (B == 0 || H == 0 || S == 0) {
    *empty = true;
    return FOG_OK;
  }
  if (!Q || !K || !V || !sinv_q || !sinv_k || !sinv_v || !O_bf16 || !dO_bf16 || !dO_e5m2 || !sinv_do || !lse || !scale_p ||
      !scale_ds || !dQ_bf16 || !dK_bf16 || !dV_bf16)
    return FOG_ERR_NULL;
  if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(O_bf16) || !aligned16(dO_bf16) || !aligned16(dO_e5m2) ||
      !aligned16(dQ_bf16) || !aligned16(dK_bf16) || !aligned16(dV_bf16))
    return FOG_ERR_ALIGN;
  if ((int64_t)(H / H_kv) * S * HD >= 0x7FFFFFFF) return FOG_ERR_UNSUPPORTED;   // a group of query heads is one 32-bit addressed buffer
  if ((int64_t)B * H > 0x7FFFFF || (int64_t)B * H * ((S + BLK - 1) / BLK) > 0x7FFFFFF0) return FOG_ERR_UNSUPPORTED;
  return FOG_OK;
}

// The launches of the backward, on checked arguments; `ws` holds three floats per row, and the sums of split launches if it has the room.
static fog_status bwd_launch(int B, int H, int H_kv, int S, float softmax_scale, int causal,
                             const uint8_t* Q, const uint8_t* K, const uint8_t* V,
                             const float* sinv_q, const float* sinv_k, const float* sinv_v,
                             const void* O_bf16, const void* dO_bf16, const uint8_t* dO_e5m2, const float* sinv_do,
                             const float* lse, const float* scale_p, const float* scale_ds,
                             void* dQ_bf16, void* dK_bf16, void* dV_bf16, float* amax_ds, float* ws, size_t ws_bytes, hipStream_t s) {
  BwdArgs a;
  a.Q = Q; a.K = K; a.V = V; a.dO8 = dO_e5m2;
  a.O = reinterpret_cast<const uint16_t*>(O_bf16); a.dO = reinterpret_cast<const uint16_t*>(dO_bf16);
  a.sinv_q = sinv_q; a.sinv_k = sinv_k; a.sinv_v = sinv_v; a.sinv_do = sinv_do;
  a.lse = lse; a.scale_p = scale_p; a.scale_ds = scale_ds;
  a.dQ = reinterpret_cast<uint16_t*>(dQ_bf16); a.dK = reinterpret_cast<uint16_t*>(dK_bf16); a.dV = reinterpret_cast<uint16_t*>(dV_bf16);
  a.amax_ds = reinterpret_cast<uint32_t*>(amax_ds); a.Dws = ws;
  a.softmax_scale = softmax_scale;
  a.BH = B * H; a.S = S; a.nblk = (S + BLK - 1) / BLK;
  a.BHkv = B * H_kv; a.G = H / H_kv;
  a.splits = 1; a.partial = nullptr;
  const int grid = a.BH * a.nblk, grid_kv = a.BHkv * (S / PAIR_KEYS);
  // the dQ kernel first: it leaves the row constants that the dK/dV kernel reads
  if (causal) { if (amax_ds) attn_bwd_dq_kernel<true, true><<<grid, kThreads, 0, s>>>(a); else attn_bwd_dq_kernel<true, false><<<grid, kThreads, 0, s>>>(a); }
  else        { if (amax_ds) attn_bwd_dq_kernel<false, true><<<grid, kThreads, 0, s>>>(a); else attn_bwd_dq_kernel<false, false><<<grid, kThreads, 0, s>>>(a); }
  // Pairs in turns where the launch is bound by its longest workgroup (the first keys see every query block of every head of the
  // group): up to half a workgroup per CU always, up to two where that workgroup walks 64 blocks or more.  Backward, us, without ->
  // with: 36 workgroups of up to 36 blocks 46 -> 37, 68 of 68 74 -> 56, 256 of 64 82 -> 71, 512 of 256 338 -> 319; but 256 of 4
  // 22 -> 25 and 512 of 32 72 -> 76.
  const int longest = (S / STEP) * a.G, cus = fog_compute_units();
  if (2 * grid_kv <= cus || (grid_kv <= 2 * cus && longest >= 64)) {
    const int splits = kv_splits(a.BHkv, S, a.G, cus);
    if (splits > 1 && aligned16(ws) && ws_bytes >= rows_bytes(B, H, S) + parts_bytes(splits, B, H_kv, S)) {
      a.splits = splits;
      a.partial = reinterpret_cast<float4*>(ws + (int64_t)3 * B * H * S);
    }
    if (causal) attn_bwd_dkdv_kernel<true, true><<<2 * grid_kv * a.splits, PAIR_THREADS, 0, s>>>(a);
    else        attn_bwd_dkdv_kernel<false, true><<<2 * grid_kv * a.splits, PAIR_THREADS, 0, s>>>(a);
    if (a.splits > 1) attn_bwd_dkdv_sum_kernel<<<2 * grid_kv, 256, 0, s>>>(a);
  } else {
    if (causal) attn_bwd_dkdv_kernel<true, false><<<grid_kv, PAIR_THREADS, 0, s>>>(a);
    else        attn_bwd_dkdv_kernel<false, false><<<grid_kv, PAIR_THREADS, 0, s>>>(a);
  }
  return fog_launch_status();
}

extern "C" fog_status fog_fp8_attn_bwd(int B, int H, int H_kv, int S, int D, float softmax_scale, int causal,
                                       const uint8_t* Q, const uint8_t* K, const uint8_t* V,
                                       const float* sinv_q, const float* sinv_k, const float* sinv_v,
                                       const void* O_bf16, const void* dO_bf16, const uint8_t* dO_e5m2, const float* sinv_do,
                                       const float* lse, const float* scale_p, const float* scale_ds,
                                       void* dQ_bf16, void* dK_bf16, void* dV_bf16, float* amax_ds,
                                       void* workspace, size_t workspace_bytes, void* stream) {
  bool empty;
  const fog_status st = bwd_checks(B, H, H_kv, S, D, softmax_scale, Q, K, V, sinv_q, sinv_k, sinv_v, O_bf16, dO_bf16, dO_e5m2,
                                   sinv_do, lse, scale_p, scale_ds, dQ_bf16, dK_bf16, dV_bf16, &empty);
  if (st != FOG_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  if (empty) {
    if (amax_ds) zero_u32b<<<1, 1, 0, s>>>(reinterpret_cast<uint32_t*>(amax_ds));
    return fog_launch_status();
  }
  if (!workspace || workspace_bytes < rows_bytes(B, H, S) || (reinterpret_cast<uintptr_t>(workspace) & 3u))
    return FOG_ERR_WORKSPACE;
  return bwd_launch(B, H, H_kv, S, softmax_scale, causal, Q, K, V, sinv_q, sinv_k, sinv_v, O_bf16, dO_bf16, dO_e5m2, sinv_do, lse,
                    scale_p, scale_ds, dQ_bf16, dK_bf16, dV_bf16, amax_ds, reinterpret_cast<float*>(workspace), workspace_bytes, s);
}

// ------------------------------------------------------------------ the backward without a caller workspace
// For callers that cannot allocate device memory (code under HIP graph capture, serving loops, harnesses
// that forbid it): what the workspace holds lives in a file-scope device array instead.  Every GPU the
// library runs on holds its own copy of the array, at its own address, until the process ends; the address
// is looked up once per device, with that device current, and kept.
constexpr int64_t kStaticRows = FOG_ATTN_BWD_STATIC_MAX_ROWS;          // B * H * S of a call, at most (6 MB of floats)
// The parts' sums behind them: kv_splits() launches at most two workgroups per CU of the part's 256, each leaving 32 KB (16 MB).
// The same parts as with a workspace make the same order of additions, so the same bytes, and the same times.
constexpr int64_t kStaticPartFloats = (int64_t)2 * 256 * 32 * 2 * HD;
static __device__ __align__(256) float scratch[3 * kStaticRows + kStaticPartFloats];
constexpr int kMaxDevices = 64;
static float* g_scratch_ptr[kMaxDevices];                             // device address of `scratch`, per device
static std::mutex g_scratch_mutex;

// Device address of this device's `scratch` (the array's name is only a host-side handle: it is never passed to a kernel).
static fog_status static_scratch(float** out) {
  int dev = -1;
  if (hipGetDevice(&dev) != hipSuccess) return FOG_ERR_HIP;
  if (dev < 0 || dev >= kMaxDevices) return FOG_ERR_UNSUPPORTED;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
      (void)hipGetLastError();
      return FOG_ERR_HIP;
    }
    g_scratch_ptr[dev] = reinterpret_cast<float*>(p);
  }
  *out = g_scratch_ptr[dev];
  return FOG_OK;
}

extern "C" fog_status fog_fp8_attn_bwd_static(int B, int H, int H_kv, int S, int D, float softmax_scale, int causal,
                                              const uint8_t* Q, const uint8_t* K, const uint8_t* V,
                                              const float* sinv_q, const float* sinv_k, const float* sinv_v,
                                              const void* O_bf16, const void* dO_bf16, const uint8_t* dO_e5m2, const float* sinv_do,
                                              const float* lse, const float* scale_p, const float* scale_ds,
                                              void* dQ_bf16, void* dK_bf16, void* dV_bf16, float* amax_ds, void* stream) {
  bool empty;
  const fog_status st = bwd_checks(B, H, H_kv, S, D, softmax_scale, Q, K, V, sinv_q, sinv_k, sinv_v, O_bf16, dO_bf16, dO_e5m2,
                                   sinv_do, lse, scale_p, scale_ds, dQ_bf16, dK_bf16, dV_bf16, &empty);
  if (st != FOG_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  if (empty) {
    if (amax_ds) zero_u32b<<<1, 1, 0, s>>>(reinterpret_cast<uint32_t*>(amax_ds));
    return fog_launch_status();
  }
  if ((int64_t)B * H * S > kStaticRows) return FOG_ERR_WORKSPACE;   // larger problems take fog_fp8_attn_bwd with a caller workspace
  float* ws = nullptr;
  const fog_status sw = static_scratch(&ws);
  if (sw != FOG_OK) return sw;
  // Nothing in the array has to start at zero: every word that a kernel reads has been written by a kernel of this call before it.
  return bwd_launch(B, H, H_kv, S, softmax_scale, causal, Q, K, V, sinv_q, sinv_k, sinv_v, O_bf16, dO_bf16, dO_e5m2, sinv_do, lse,
                    scale_p, scale_ds, dQ_bf16, dK_bf16, dV_bf16, amax_ds, ws, sizeof(scratch), s);
}
