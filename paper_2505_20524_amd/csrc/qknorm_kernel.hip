// QK RMS normalisation with a frozen scalar gain, fused with the FP8 cast (Section 3 of the paper:
// N_gamma(x) = gamma x / rms(x), rms(x) = ||x||_2 / sqrt(D), gains frozen in the FOG variants;
// cast of Appendix E with a caller-provided scale, as under delayed scaling).  The normalised
// tensor is never stored: every bf16 element is read once and one FP8 byte is written, against
// 2 + 2 + 2 + 2 + 1 bytes per element for normalise -> abs-max -> cast as separate passes.
// Bound by HBM, with the vector ALU close behind: the square root and the divisions of a row are computed by one lane of four (each
// takes one of the four rows in flight), row sums are exchanged inside the vector ALU, and the casts go without clamp and NaN test
// where the row's norm, the gain and the scale say so (262144 x 128, whole call: 26.1 -> 23.9 us, 19.2 with one workgroup per
// compute unit and ordinary loads).
// A row of D elements is handled by D / 8 adjacent lanes (16 for the head size 128,
// four rows per wave); longer or odd rows take one wave per row and read the row twice.
#include "common.h"
#include "launch.h"

namespace {

constexpr int kThreads = 256;          // general kernel, and the rows kernel on few rows
// Rows kernel otherwise: one workgroup per compute unit.  Every workgroup raises the one abs-max word when it ends, nearly all at the same time,
// and same-address atomics are served one after the other: 2048 workgroups of 256 threads took 8 us for the abs-max, 256 of 1024
// take 2-3, its clearing launch included.
constexpr int kRowThreads = 1024;

__global__ void zero_u32q(uint32_t* p) { *p = 0u; }

FOG_DEVICE float inv_rms(float sumsq, float cols, float gain) {
  // gain / sqrt(sumsq / D), correctly rounded square root and divisions; 0 for a row of zeros
  return sumsq > 0.0f ? gain / __builtin_sqrtf(sumsq / cols) : 0.0f;
}

// Workgroup maximum raised into *amax_out; reduced on bit patterns (non-negative floats order like them,
// and the NaN pattern of a thread that saw a NaN orders above everything).
template <int THREADS>
FOG_DEVICE void block_amax(float m, bool nan, uint32_t* amax_out) {
  const uint32_t h = wave_max_u32(amax_bits(m, nan));
  __shared__ uint32_t part[THREADS / 64];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = h;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t b = part[0];
#pragma unroll
    for (int w = 1; w < THREADS / 64; ++w) b = b > part[w] ? b : part[w];
    if (b > __hip_atomic_load(amax_out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(amax_out, b);
  }
}

// Sum over the LPR adjacent lanes of a row, in every lane: exchanges inside the vector ALU (quad permutes and mirrors within rows of
// 16 lanes) where a shuffle goes through LDS; the partners hold the same partial sums as under an xor shuffle, so the bits agree.
template <int CTRL>
FOG_DEVICE float dpp_add(float s) {
  return s + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(s), CTRL, 0xF, 0xF, false));
}
template <int LPR>
FOG_DEVICE float row_sum(float s) {
  s = dpp_add<0xB1>(s);                  // lane ^ 1
  s = dpp_add<0x4E>(s);                  // lane ^ 2
  s = dpp_add<0x141>(s);                 // the other four of eight (half-row mirror)
  if (LPR >= 16) s = dpp_add<0x140>(s);  // the other eight of sixteen (row mirror)
  if (LPR >= 32) s += __shfl_xor(s, 16, 64);
  if (LPR >= 64) s += __shfl_xor(s, 32, 64);
  return s;
}
// Value of lane u of every four.
template <int U>
FOG_DEVICE float quad_lane(float v) { return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x55 * U, 0xF, 0xF, false)); }

// LPR lanes per row, each holding 8 consecutive elements (cols = 8 LPR); 64 / LPR rows per wave.
// REREAD: ordinary loads, for tensors that may still lie in the memory-side cache (non-temporal ones find them there less often).
template <int FMT, int LPR, int THREADS, bool REREAD>
__global__ __launch_bounds__(THREADS) void qknorm_rows_kernel(const uint16_t* __restrict__ x, int64_t rows, int64_t ldx, float gain,
                                                              const float* __restrict__ scale, uint8_t* __restrict__ q, int64_t ldq,
                                                              uint32_t* __restrict__ amax_out) {
  constexpr int RPB = THREADS / LPR;   // rows per workgroup and load
  constexpr int U = 4;                  // rows per lane group and trip: four loads in flight
  const float rho = *scale;
  const int sub = threadIdx.x % LPR, rloc = threadIdx.x / LPR;
  // |y| <= 1.5 gain sqrt(cols) in rows whose sum of squares and inverse norm are finite (squares that vanish below the smallest
  // subnormal included): with such a gain and scale no product overflows, and the saturating converts, which let infinities
  // through, need neither a clamp nor a NaN test
  const bool plain = gain <= 1.0e30f && fabsf(rho) * gain <= 1.0e30f;
  saturating_converts();
  float m = 0.0f;
  bool nan = false;
  auto fetch = [&](int64_t r0, uint4 (&v)[U]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t r = r0 + u * RPB + rloc;
      v[u] = make_uint4(0u, 0u, 0u, 0u);
      const uint16_t* p = x + r * ldx + 8 * sub;
      if (r < rows) v[u] = REREAD ? *reinterpret_cast<const uint4*>(p) : ld_nt16(p);
    }
  };
  auto process = [&](int64_t r0, const uint4 (&v)[U]) {
    float sum[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float f[8] = {bf16lo(v[u].x), bf16hi(v[u].x), bf16lo(v[u].y), bf16hi(v[u].y), bf16lo(v[u].z), bf16hi(v[u].z), bf16lo(v[u].w), bf16hi(v[u].w)};
      float s = 0.0f;
#pragma unroll
      for (int k = 0; k < 8; ++k) s = __builtin_fmaf(f[k], f[k], s);
      sum[u] = row_sum<LPR>(s);
    }
    // The square root and the two divisions cost as much as the rest of a row: of every four lanes each takes one of the four rows.
    static_assert(U == 4, "one row per lane of a quad");
    const float mine = sub & 2 ? (sub & 1 ? sum[3] : sum[2]) : (sub & 1 ? sum[1] : sum[0]);
    const float inv_mine = inv_rms(mine, (float)(8 * LPR), gain);
    const float invs[U] = {quad_lane<0>(inv_mine), quad_lane<1>(inv_mine), quad_lane<2>(inv_mine), quad_lane<3>(inv_mine)};
    // (the inverse norm is infinite where the mean of tiny squares rounds to 0 or the gain is large against the norm)
    const bool all_plain = plain && __all(mine < INFINITY && inv_mine < INFINITY);   // every row of the wave's trip
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t r = r0 + u * RPB + rloc;
      const float f[8] = {bf16lo(v[u].x), bf16hi(v[u].x), bf16lo(v[u].y), bf16hi(v[u].y), bf16lo(v[u].z), bf16hi(v[u].z), bf16lo(v[u].w), bf16hi(v[u].w)};
      const float inv = invs[u];
      float y[8];
#pragma unroll
      for (int k = 0; k < 8; ++k) {
        y[k] = f[k] * inv;
        m = fmaxf(m, fabsf(y[k]));
      }
      if (r < rows) {
        uint2 o;
        if (__builtin_expect(all_plain, 1)) {
          o.x = cvt4_fp8_finite<FMT>(y[0] * rho, y[1] * rho, y[2] * rho, y[3] * rho);
          o.y = cvt4_fp8_finite<FMT>(y[4] * rho, y[5] * rho, y[6] * rho, y[7] * rho);
        } else {
          o.x = cvt4_fp8_nan<FMT>(y[0] * rho, y[1] * rho, y[2] * rho, y[3] * rho, &nan);
          o.y = cvt4_fp8_nan<FMT>(y[4] * rho, y[5] * rho, y[6] * rho, y[7] * rho, &nan);
        }
        st_nt8(q + r * ldq + 8 * sub, o);
      }
    }
  };
  // the next trip's loads are requested before the current trip is normalised
  const int64_t step = (int64_t)gridDim.x * (RPB * U);
  int64_t r0 = (int64_t)blockIdx.x * (RPB * U);
  uint4 va[U], vb[U];
  if (r0 < rows) fetch(r0, va);
  while (r0 < rows) {
    const int64_t r1 = r0 + step;
    if (r1 < rows) fetch(r1, vb);
    process(r0, va);
    if (r1 >= rows) break;
    const int64_t r2 = r1 + step;
    if (r2 < rows) fetch(r2, va);
    process(r1, vb);
    r0 = r2;
  }
  if (amax_out) block_amax<THREADS>(m, nan, amax_out);
}

// Any row length: one wave per row, two passes over the row (the second is served from cache).
template <int FMT>
__global__ __launch_bounds__(kThreads) void qknorm_general_kernel(const uint16_t* __restrict__ x, int64_t rows, int64_t cols, int64_t ldx,
                                                                  float gain, const float* __restrict__ scale, uint8_t* __restrict__ q,
                                                                  int64_t ldq, uint32_t* __restrict__ amax_out) {
  const float rho = *scale;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  float m = 0.0f;
  bool nan = false;
  for (int64_t r = (int64_t)blockIdx.x * 4 + w; r < rows; r += (int64_t)gridDim.x * 4) {
    const uint16_t* row = x + r * ldx;
    float s = 0.0f;
    for (int64_t i = lane; i < cols; i += 64) {
      const float a = bf16lo(row[i]);
      s = __builtin_fmaf(a, a, s);
    }
    s = wave_sum_f32(s);
    const float inv = inv_rms(s, (float)cols, gain);
    for (int64_t i = lane; i < cols; i += 64) {
      const float y = bf16lo(row[i]) * inv;
      m = fmaxf(m, fabsf(y));
      const float t = y * rho;
      q[r * ldq + i] = (uint8_t)(cvt4_fp8_nan<FMT>(t, t, t, t, &nan) & 0xFFu);
    }
  }
  if (amax_out) block_amax<kThreads>(m, nan, amax_out);
}

template <int FMT>
void launch_qknorm(const uint16_t* x, int64_t rows, int64_t cols, int64_t ldx, float gain, const float* scale, uint8_t* q, int64_t ldq,
                   uint32_t* amax_out, hipStream_t s) {
  const bool vec = (reinterpret_cast<uintptr_t>(x) & 15u) == 0 && (reinterpret_cast<uintptr_t>(q) & 7u) == 0 && ldx % 8 == 0 && ldq % 8 == 0;
  // Up to a quarter of the 256 MB memory-side cache the input is read with ordinary loads.  us, non-temporal -> ordinary, the same three
  // tensors in turn and tensors that no call has just read: 131072 x 128 14.5 -> 14.2 and 14.2 -> 15.6, 262144 x 128 21.8 -> 19.3 and
  // 21.7 -> 22.7; 400000 x 128 31.6 -> 33.4 and 31.9 -> 33.8, 900000 x 128 63.5 -> 67.2 and 62.9 -> 67.2.  In front of the attention
  // forward: 1 x 16 x 1024 41.9 -> 40.6, 1 x 32/8 x 4096 121.5 -> 119.4, 2 x 32 x 4096 242.7 -> 244.3, 4 x 32 x 4096 476 -> 483.
  const bool reread = rows * cols <= (int64_t)32 << 20;
  // A workgroup of 1024 threads takes 4096 / LPR rows: below 1 M elements these are too few workgroups, and the smaller form is the faster
  // (1024 x 128 6.5 -> 5.5 us, 6000 x 128 6.6 -> 6.2; 9216 x 128 6.9 against 6.8, 16384 x 128 7.2 against 8.0).
  const bool few = rows * cols < (int64_t)1 << 20;
#define FOG_QKT(LPR, T, RE)                                                                                                   \
  do {                                                                                                                        \
    constexpr int ROWS = 4 * (T / LPR);   /* of a workgroup and trip */                                                       \
    int64_t blocks = (rows + ROWS - 1) / ROWS;                                                                                \
    if (blocks > fog_compute_units()) blocks = fog_compute_units();                                                           \
    qknorm_rows_kernel<FMT, LPR, T, RE><<<(int)blocks, T, 0, s>>>(x, rows, ldx, gain, scale, q, ldq, amax_out);               \
    return;                                                                                                                   \
  } while (0)
#define FOG_QKN(LPR)                                                                                                          \
  do {                                                                                                                        \
    if (few) FOG_QKT(LPR, kThreads, true);                                                                                    \
    if (reread) FOG_QKT(LPR, kRowThreads, true);                                                                              \
    FOG_QKT(LPR, kRowThreads, false);                                                                                         \
  } while (0)
  if (vec && cols == 128) FOG_QKN(16);
  if (vec && cols == 64) FOG_QKN(8);
  if (vec && cols == 256) FOG_QKN(32);
  if (vec && cols == 512) FOG_QKN(64);
#undef FOG_QKN
#undef FOG_QKT
  int64_t blocks = (rows + 3) / 4;
  if (blocks > 4096) blocks = 4096;
  qknorm_general_kernel<FMT><<<(int)blocks, kThreads, 0, s>>>(x, rows, cols, ldx, gain, scale, q, ldq, amax_out);
}

}  // namespace

extern "C" fog_status fog_rmsnorm_quantize(const void* x_bf16, int64_t rows, int64_t cols, int64_t ldx, float gain, fog_fp8 fmt,
                                           const float* scale, uint8_t* q, int64_t ldq, float* amax_out, void* stream) {
  if (!scale) return FOG_ERR_NULL;
  if (rows < 0 || cols < 0) return FOG_ERR_SHAPE;
  if (fmt != FOG_E4M3 && fmt != FOG_E5M2) return FOG_ERR_UNSUPPORTED;
  if (!(gain > 0.0f) || !(gain <= 3.402823466e38f)) return FOG_ERR_UNSUPPORTED;
  hipStream_t s = (hipStream_t)stream;
  if (amax_out) zero_u32q<<<1, 1, 0, s>>>(reinterpret_cast<uint32_t*>(amax_out));
  if (rows == 0 || cols == 0) return fog_launch_status();
  if (!x_bf16 || !q) return FOG_ERR_NULL;
  if (ldx < cols || ldq < cols) return FOG_ERR_SHAPE;
  if (reinterpret_cast<uintptr_t>(x_bf16) & 1u) return FOG_ERR_ALIGN;
  const uint16_t* x = reinterpret_cast<const uint16_t*>(x_bf16);
  uint32_t* am = reinterpret_cast<uint32_t*>(amax_out);
  if (fmt == FOG_E4M3) launch_qknorm<FOG_E4M3>(x, rows, cols, ldx, gain, scale, q, ldq, am, s);
  else                 launch_qknorm<FOG_E5M2>(x, rows, cols, ldx, gain, scale, q, ldq, am, s);
  return fog_launch_status();
}
