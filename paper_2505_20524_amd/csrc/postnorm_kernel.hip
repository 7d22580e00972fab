// Post-RMSNorm with its residual connection, fused with the FP8 cast of the new residual stream
// (Section 3 of the paper: the sub-layer output y goes through N_gamma(y) = gamma (.) y / rms(y),
// rms(y) = ||y||_2 / sqrt(D), gamma a trainable vector, before it is added to the residual stream x;
// the block has no pre-normalisation, so x + N_gamma(y) is also the next GEMM's input and gets the
// cast of Appendix E with a caller-provided scale, as under delayed scaling).
// One pass: y and x are read once (2 + 2 B per element), the new stream is written as bf16 (2 B) and
// as FP8 codes (1 B); the abs-max of the stored bf16 tensor comes with it.  Done as separate passes
// the same work moves 2+2 (norm) + 2+2+2 (add) + 2 (abs-max) + 2+1 (cast) bytes.  HBM-bound.
#include <cfloat>

#include "common.h"
#include "launch.h"

namespace {

constexpr int kThreads = 256;
constexpr int kWideThreads = 1024;

__global__ void zero_u32p(uint32_t* p) { *p = 0u; }

FOG_DEVICE float inv_rms(float sumsq, float cols) {
  // 1 / sqrt(sumsq / D), correctly rounded square root and divisions; 0 for a vector of zeros
  return sumsq > 0.0f ? 1.0f / __builtin_sqrtf(sumsq / cols) : 0.0f;
}

// abs-max of bf16 values kept as their 15-bit magnitude patterns (ordered like the values)
template <int THREADS>
FOG_DEVICE void block_amax_bits(uint32_t m, uint32_t* amax_out) {
  m = wave_max_u32(m);
  __shared__ uint32_t part[THREADS / 64];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t r = part[0];
#pragma unroll
    for (int w = 1; w < THREADS / 64; ++w) r = r > part[w] ? r : part[w];
    r <<= 16;   // the float with that bf16 pattern
    if (r > __hip_atomic_load(amax_out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(amax_out, r);
  }
}

// One element before its one rounding to bf16.
FOG_DEVICE float residual(float x, float y, float g, float inv) { return __builtin_fmaf(g * y, inv, x); }

// Bound by HBM (7 bytes per element).  Whole calls, other buffers each time, with the bf16 rounding in integers, the NaN test in every
// cast and a workgroup for every four rows -> now: 8192 x 4096 54.7 -> 46.5 us, 777 x 8192 19.4 -> 15.9 us.
// One wave per row; a lane owns C <= CMAX chunks of 8 consecutive elements (chunk c of lane l is
// elements [8 (64 c + l), +8): consecutive lanes read consecutive 16 bytes).  All loads of y and x
// of a row are issued before the first is used.
// Non-temporal loads at every size: ordinary ones find a tensor in the memory-side cache more often where the same few are used over
// and over (8192 x 4096 46.8 -> 45.0 us), but lose everywhere else: on tensors that no call has just read 46.8 -> 50.8, 2048 x 4096
// 17.3 -> 21.3, 1024 x 8192 17.0 -> 28.1, and behind the product that writes y, feed-forward half of 4096 x 4096 98.5 -> 105.0.
template <int FMT, int CMAX, int THREADS>
__global__ __launch_bounds__(THREADS) void postnorm_rows_kernel(const uint16_t* x, int64_t ldx, const uint16_t* __restrict__ y,
                                                                 int64_t ldy, int64_t rows, int C, const float* __restrict__ gamma,
                                                                 const float* __restrict__ scale, uint16_t* out, int64_t ldo,
                                                                 uint8_t* __restrict__ q, int64_t ldq, uint32_t* __restrict__ amax_out) {
  const float rho = *scale;
  // Finite values under a finite scale give no NaN (products that overflow are clamped): a lane that has met another value, and
  // every lane under another scale, casts its rows a second time with the NaN test.  (Saturating converts would spare the clamp,
  // but the same mode rounds bf16 sums beyond the largest finite value down to it.)
  const uint32_t limit = fabsf(rho) <= FLT_MAX ? 0x7F80u : 0u;
  const float cols = (float)(C * 512);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t m = 0u;
  for (int64_t r = (int64_t)blockIdx.x * (THREADS / 64) + w; r < rows; r += (int64_t)gridDim.x * (THREADS / 64)) {
    uint4 vy[CMAX], vx[CMAX];
#pragma unroll
    for (int c = 0; c < CMAX; ++c)
      if (c < C) vy[c] = ld_nt16(y + r * ldy + 8 * (64 * c + lane));
#pragma unroll
    for (int c = 0; c < CMAX; ++c)
      if (c < C) vx[c] = ld_nt16(x + r * ldx + 8 * (64 * c + lane));
    float s = 0.0f;
#pragma unroll
    for (int c = 0; c < CMAX; ++c)
      if (c < C) {
        const float f[8] = {bf16lo(vy[c].x), bf16hi(vy[c].x), bf16lo(vy[c].y), bf16hi(vy[c].y),
                            bf16lo(vy[c].z), bf16hi(vy[c].z), bf16lo(vy[c].w), bf16hi(vy[c].w)};
#pragma unroll
        for (int k = 0; k < 8; ++k) s = __builtin_fmaf(f[k], f[k], s);
      }
    s = wave_sum_f32(s);
    const float inv = inv_rms(s, cols);
#pragma unroll
    for (int c = 0; c < CMAX; ++c)
      if (c < C) {
        const int64_t col = 8 * (64 * c + lane);
        const float4 g0 = *reinterpret_cast<const float4*>(gamma + col), g1 = *reinterpret_cast<const float4*>(gamma + col + 4);
        const uint4 o = make_uint4(
            pack_bf16x2(residual(bf16lo(vx[c].x), bf16lo(vy[c].x), g0.x, inv), residual(bf16hi(vx[c].x), bf16hi(vy[c].x), g0.y, inv)),
            pack_bf16x2(residual(bf16lo(vx[c].y), bf16lo(vy[c].y), g0.z, inv), residual(bf16hi(vx[c].y), bf16hi(vy[c].y), g0.w, inv)),
            pack_bf16x2(residual(bf16lo(vx[c].z), bf16lo(vy[c].z), g1.x, inv), residual(bf16hi(vx[c].z), bf16hi(vy[c].z), g1.y, inv)),
            pack_bf16x2(residual(bf16lo(vx[c].w), bf16lo(vy[c].w), g1.z, inv), residual(bf16hi(vx[c].w), bf16hi(vy[c].w), g1.w, inv)));
        m = pkmax_abs_bf16(m, o.x); m = pkmax_abs_bf16(m, o.y); m = pkmax_abs_bf16(m, o.z); m = pkmax_abs_bf16(m, o.w);
        st_nt16(out + r * ldo + col, o);
        if (q)
          st_nt8(q + r * ldq + col, make_uint2(cvt4_fp8<FMT>(bf16lo(o.x) * rho, bf16hi(o.x) * rho, bf16lo(o.y) * rho, bf16hi(o.y) * rho),
                                               cvt4_fp8<FMT>(bf16lo(o.z) * rho, bf16hi(o.z) * rho, bf16lo(o.w) * rho, bf16hi(o.w) * rho)));
        vx[c] = o;
      }
    if (__builtin_expect(q && max_of_pair(m) >= limit, 0)) {
#pragma unroll
      for (int c = 0; c < CMAX; ++c)
        if (c < C) {
          const uint4 o = vx[c];
          st_nt8(q + r * ldq + 8 * (64 * c + lane), make_uint2(cvt4_fp8_nan<FMT>(bf16lo(o.x) * rho, bf16hi(o.x) * rho, bf16lo(o.y) * rho, bf16hi(o.y) * rho),
                                                               cvt4_fp8_nan<FMT>(bf16lo(o.z) * rho, bf16hi(o.z) * rho, bf16lo(o.w) * rho, bf16hi(o.w) * rho)));
        }
    }
  }
  if (amax_out) {
    block_amax_bits<THREADS>(max_of_pair(m), amax_out);
  }
}

// Any row length and alignment: one wave per row, two passes over y (the second is served from cache).
template <int FMT>
__global__ __launch_bounds__(kThreads) void postnorm_general_kernel(const uint16_t* x, int64_t ldx, const uint16_t* __restrict__ y,
                                                                    int64_t ldy, int64_t rows, int64_t cols, const float* __restrict__ gamma,
                                                                    const float* __restrict__ scale, uint16_t* out, int64_t ldo,
                                                                    uint8_t* __restrict__ q, int64_t ldq, uint32_t* __restrict__ amax_out) {
  const float rho = *scale;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t m = 0u;
  for (int64_t r = (int64_t)blockIdx.x * 4 + w; r < rows; r += (int64_t)gridDim.x * 4) {
    const uint16_t* yr = y + r * ldy;
    float s = 0.0f;
    for (int64_t i = lane; i < cols; i += 64) {
      const float a = bf16lo(yr[i]);
      s = __builtin_fmaf(a, a, s);
    }
    s = wave_sum_f32(s);
    const float inv = inv_rms(s, (float)cols);
    for (int64_t i = lane; i < cols; i += 64) {
      const uint32_t b = f32_to_bf16(residual(bf16lo(x[r * ldx + i]), bf16lo(yr[i]), gamma[i], inv));
      out[r * ldo + i] = (uint16_t)b;
      const uint32_t mag = b & 0x7FFFu;
      m = m > mag ? m : mag;
      if (q) {
        const float t = bf16lo(b) * rho;
        q[r * ldq + i] = (uint8_t)(cvt4_fp8_nan<FMT>(t, t, t, t) & 0xFFu);
      }
    }
  }
  if (amax_out) block_amax_bits<kThreads>(m, amax_out);
}

template <int FMT>
void launch_postnorm(const uint16_t* x, int64_t ldx, const uint16_t* y, int64_t ldy, int64_t rows, int64_t cols, const float* gamma,
                     const float* scale, uint16_t* out, int64_t ldo, uint8_t* q, int64_t ldq, uint32_t* amax_out, hipStream_t s) {
  auto al = [](const void* p, uintptr_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0; };
  const bool vec = cols % 512 == 0 && cols <= 8192 && al(x, 16) && al(y, 16) && al(out, 16) && al(gamma, 16) && (!q || al(q, 8)) &&
                   ldx % 8 == 0 && ldy % 8 == 0 && ldo % 8 == 0 && ldq % 8 == 0;
  int64_t blocks = (rows + 3) / 4;
  if (vec) {
    // Few workgroups that walk the rows, whatever the registers allow: with more waves in flight the streams past the caches get in
    // each other's way, and every workgroup raises the abs-max word when it ends.  Two of 256 threads per CU, or, for rows of up to
    // 1024 elements and small tensors of up to 2048, one of 1024.  us, 512 x 256 threads -> 256 x 1024: 16384 x 512 18.4 -> 14.5,
    // 65536 x 1024 97.1 -> 83.5, 2048 x 512 11.2 -> 7.4, 4096 x 2048 18.2 -> 15.2; 65536 x 2048 168 -> 174, 4096 x 4096 24 -> 35.
    // (512 workgroups of 256 threads against up to 8192: 4096 x 1024 20.0 -> 13.6, 8192 x 4096 49.7 -> 47.0.)
    // At fewer rows than columns the 16 rows of a wide workgroup leave it too few workgroups: 64 x 512 5.5 -> 6.0, 512 x 2048 7.7 -> 8.2,
    // feed-forward half of 1024 x 2048 41.9 -> 42.6; 2048 x 2048 52.4 -> 52.0.
    // A trip of the wide form takes 16 rows per CU, of the narrow one 8, and a trip that is nearly empty takes as long as a full one: over
    // several trips the wide form has to fill them, the more the longer its rows (tensors that no call has just read, narrow -> wide:
    // 4926 x 512 11.1 -> 11.4, 9000 x 512 14.2 -> 12.8; 4926 x 1024 13.0 -> 14.7, 5500 x 1024 15.4 -> 14.7, 9000 x 1024 18.4 -> 18.8, 9800 x
    // 1024 20.5 -> 18.9; 4926 x 2048 18.5 -> 21.0, 6144 x 2048 22.0 -> 22.3, 8192 x 2048 27.2 -> 25.9, 8400 x 2048 28.2 -> 30.5).
    const int C = (int)(cols / 512), cus = fog_compute_units();
    const int64_t trip = (int64_t)(kWideThreads / 64) * cus, trips = (rows + trip - 1) / trip;
    const bool filled = trips <= 1 || 20 * rows >= (C <= 2 ? 13 : 16) * trips * trip;
    const bool wide = rows >= cols && filled && (C <= 2 || (C <= 4 && rows * cols <= (int64_t)16 << 20));
    const int threads = wide ? kWideThreads : kThreads;
    const int64_t most = wide ? cus : 2 * cus;
    blocks = (rows + threads / 64 - 1) / (threads / 64);
    if (blocks > most) blocks = most;
#define FOG_PN(CM, T) postnorm_rows_kernel<FMT, CM, T><<<(int)blocks, T, 0, s>>>(x, ldx, y, ldy, rows, C, gamma, scale, out, ldo, q, ldq, amax_out)
    if (wide)        FOG_PN(4, kWideThreads);
    else if (C <= 4) FOG_PN(4, kThreads);
    else if (C <= 8) FOG_PN(8, kThreads);
    else             FOG_PN(16, kThreads);
#undef FOG_PN
    return;
  }
  if (blocks > 8192) blocks = 8192;
  postnorm_general_kernel<FMT><<<(int)blocks, kThreads, 0, s>>>(x, ldx, y, ldy, rows, cols, gamma, scale, out, ldo, q, ldq, amax_out);
}

}  // namespace

extern "C" fog_status fog_postnorm_residual_quantize(const void* x_bf16, int64_t ldx, const void* y_bf16, int64_t ldy, int64_t rows,
                                                     int64_t cols, const float* gamma, fog_fp8 fmt, const float* scale, void* xnew_bf16,
                                                     int64_t ldo, uint8_t* q, int64_t ldq, float* amax_out, void* stream) {
  if (!scale) return FOG_ERR_NULL;
  if (rows < 0 || cols < 0) return FOG_ERR_SHAPE;
  if (fmt != FOG_E4M3 && fmt != FOG_E5M2) return FOG_ERR_UNSUPPORTED;
  hipStream_t s = (hipStream_t)stream;
  if (amax_out) zero_u32p<<<1, 1, 0, s>>>(reinterpret_cast<uint32_t*>(amax_out));
  if (rows == 0 || cols == 0) return fog_launch_status();
  if (!x_bf16 || !y_bf16 || !gamma || !xnew_bf16) return FOG_ERR_NULL;
  if (ldx < cols || ldy < cols || ldo < cols || (q && ldq < cols)) return FOG_ERR_SHAPE;
  if ((reinterpret_cast<uintptr_t>(x_bf16) | reinterpret_cast<uintptr_t>(y_bf16) | reinterpret_cast<uintptr_t>(xnew_bf16)) & 1u) return FOG_ERR_ALIGN;
  if (reinterpret_cast<uintptr_t>(gamma) & 3u) return FOG_ERR_ALIGN;
  const uint16_t* x = reinterpret_cast<const uint16_t*>(x_bf16);
  const uint16_t* y = reinterpret_cast<const uint16_t*>(y_bf16);
  uint16_t* out = reinterpret_cast<uint16_t*>(xnew_bf16);
  uint32_t* am = reinterpret_cast<uint32_t*>(amax_out);
  if (fmt == FOG_E4M3) launch_postnorm<FOG_E4M3>(x, ldx, y, ldy, rows, cols, gamma, scale, out, ldo, q, ldq, am, s);
  else                 launch_postnorm<FOG_E5M2>(x, ldx, y, ldy, rows, cols, gamma, scale, out, ldo, q, ldq, am, s);
  return fog_launch_status();
}
