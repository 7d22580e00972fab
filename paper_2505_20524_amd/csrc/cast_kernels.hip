// Per-tensor scaling kernels: abs-max, scale, FP8 cast (optionally fused with a transpose).
//
// What they compute (Appendix E of the paper): rho = FP8MaxValue / (2^m max H) and
// FP8cast(rho X); Section 2 calls the two-pass flow (abs-max, then cast) just-in-time scaling
// and the one-pass flow (cast with last iteration's scale, abs-max as a by-product) delayed
// scaling.  All of these are HBM-bound: every element is read once with 16-byte loads and
// every output byte is written once with 8- or 16-byte stores.  Casts alone run at the copy rate; what their memory accesses do to the
// kernels around them counts as much.
#include "common.h"
#include "launch.h"
#include "words.h"
#include "../../include/fog_probe.h"

namespace {

constexpr int kThreads = 256;

__global__ void zero_u32_kernel(uint32_t* p) { *p = 0u; }

// ---------------------------------------------------------------- abs-max
// bf16 magnitudes order like unsigned 16-bit integers, so the running maximum is a packed
// u16 max over the sign-cleared bit patterns; the result is the float whose upper half is it.
//
// PARTIALS: the form used by the one-call just-in-time flow.  Every workgroup stores its maximum in
// its own word of the caller's workspace (no atomics, no zero-initialisation, no fence); a
// one-workgroup kernel then reduces the words and derives the scale.  This form reads with ordinary
// (cache-retaining) loads, because the cast pass re-reads the tensor right away, back to front.
FOG_DEVICE void scale_from_amax(float a, int fmt, int margin, float* scale, float* scale_inv);
FOG_DEVICE void publish_block_max(uint32_t r, uint32_t* out, bool partials, int bid) {
  if (partials) {
    out[bid] = r << 16;
    return;
  }
  // same-address atomics are served one at a time: skip the ones that cannot raise the maximum
  if (r && (r << 16) > __hip_atomic_load(out, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(out, r << 16);
}

// Workgroup `bid` of `nb` over one contiguous tensor (a whole launch, or one job's share of a batched launch).
template <bool PARTIALS>
FOG_DEVICE void amax_span(const uint4* __restrict__ x, int64_t nvec, const uint16_t* __restrict__ tail, int ntail,
                          uint32_t* __restrict__ out, int bid, int nb) {
  // Every workgroup owns one contiguous span and walks it in batches of eight 16-byte loads per
  // thread; the next batch is requested before the current one is reduced, so loads never stop.
  constexpr int NL = 8;
  const int64_t per = (nvec + nb - 1) / nb;
  const int64_t b0 = per * bid, b1 = b0 + per < nvec ? b0 + per : nvec;
  uint32_t m[4] = {0, 0, 0, 0};
  int64_t i = b0 + threadIdx.x;
  uint4 v[NL];
  bool have = i + (NL - 1) * kThreads < b1;
  if (have) {
#pragma unroll
    for (int k = 0; k < NL; ++k) v[k] = PARTIALS ? x[i + k * kThreads] : ld_nt16(x + i + k * kThreads);
  }
  while (have) {
    const int64_t n = i + NL * kThreads;
    const bool more = n + (NL - 1) * kThreads < b1;
    uint4 nx[NL];
    if (more) {
#pragma unroll
      for (int k = 0; k < NL; ++k) nx[k] = PARTIALS ? x[n + k * kThreads] : ld_nt16(x + n + k * kThreads);
    }
#pragma unroll
    for (int k = 0; k < NL; ++k) {
      m[0] = pkmax_abs_bf16(m[0], v[k].x); m[1] = pkmax_abs_bf16(m[1], v[k].y);
      m[2] = pkmax_abs_bf16(m[2], v[k].z); m[3] = pkmax_abs_bf16(m[3], v[k].w);
    }
    if (more) {
#pragma unroll
      for (int k = 0; k < NL; ++k) v[k] = nx[k];
    }
    i = n;
    have = more;
  }
  for (; i < b1; i += kThreads) {
    uint4 a = ld_nt16(x + i);
    m[0] = pkmax_abs_bf16(m[0], a.x); m[1] = pkmax_abs_bf16(m[1], a.y);
    m[2] = pkmax_abs_bf16(m[2], a.z); m[3] = pkmax_abs_bf16(m[3], a.w);
  }
  uint32_t mm = pkmax_abs_bf16(pkmax_abs_bf16(m[0], m[1]), pkmax_abs_bf16(m[2], m[3]));
  uint32_t h = (mm >> 16) > (mm & 0xFFFFu) ? (mm >> 16) : (mm & 0xFFFFu);
  if (bid == 0 && (int)threadIdx.x < ntail) {
    uint32_t t = tail[threadIdx.x] & 0x7FFFu;
    h = h > t ? h : t;
  }
  h = wave_max_u32(h);
  __shared__ uint32_t part[kThreads / 64];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = h;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t r = part[0];
#pragma unroll
    for (int w = 1; w < kThreads / 64; ++w) r = r > part[w] ? r : part[w];
    publish_block_max(r, out, PARTIALS, bid);
  }
}

template <bool PARTIALS>
__global__ __launch_bounds__(kThreads) void amax_kernel(const uint4* __restrict__ x, int64_t nvec,
                                                        const uint16_t* __restrict__ tail, int ntail,
                                                        uint32_t* __restrict__ out) {
  amax_span<PARTIALS>(x, nvec, tail, ntail, out, (int)blockIdx.x, (int)gridDim.x);
}

// Abs-max of a matrix whose rows are not contiguous or not 16-byte aligned (slow, same result).
template <bool PARTIALS>
__global__ __launch_bounds__(kThreads) void amax_strided_kernel(const uint16_t* __restrict__ x, int64_t rows, int64_t cols,
                                                                int64_t ldx, uint32_t* __restrict__ out) {
  const int64_t total = rows * cols;
  uint32_t m = 0;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < total; i += (int64_t)gridDim.x * kThreads) {
    const int64_t r = i / cols, c = i - r * cols;
    const uint32_t a = x[r * ldx + c] & 0x7FFFu;
    m = m > a ? m : a;
  }
  m = wave_max_u32(m);
  __shared__ uint32_t part[kThreads / 64];
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t r = part[0];
#pragma unroll
    for (int w = 1; w < kThreads / 64; ++w) r = r > part[w] ? r : part[w];
    publish_block_max(r, out, PARTIALS, (int)blockIdx.x);
  }
}

// ---------------------------------------------------------------- scale
FOG_DEVICE void scale_from_amax(float a, int fmt, int margin, float* scale, float* scale_inv) {
  const float fmax = fmt == FOG_E4M3 ? 448.0f : 57344.0f;
  float rho = 1.0f;
  if (a > 0.0f && a <= 3.402823466e38f) {
    float denom = ldexpf(a, margin);
    rho = fmax / denom;  // correctly rounded binary32 division
    if (rho > 3.402823466e38f) rho = 3.402823466e38f;
    if (!(rho > 0.0f)) rho = 1.0f;
  }
  *scale = rho;
  if (scale_inv) *scale_inv = 1.0f / rho;
}

__global__ void scale_kernel(const float* amax, int fmt, int margin, float* scale, float* scale_inv) {
  scale_from_amax(*amax, fmt, margin, scale, scale_inv);
}

// One workgroup: maximum of the per-workgroup maxima of the abs-max pass, then the scale.
__global__ __launch_bounds__(kThreads) void scale_partials_kernel(const uint32_t* __restrict__ part, int n, int fmt, int margin,
                                                                 float* amax, float* scale, float* scale_inv) {
  uint32_t m = 0;
  for (int i = threadIdx.x; i < n; i += kThreads) m = m > part[i] ? m : part[i];   // non-negative floats order like their bits
  m = wave_max_u32(m);
  __shared__ uint32_t wmax[kThreads / 64];
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t r = wmax[0];
#pragma unroll
    for (int w = 1; w < kThreads / 64; ++w) r = r > wmax[w] ? r : wmax[w];
    const float a = __uint_as_float(r);
    *amax = a;
    scale_from_amax(a, fmt, margin, scale, scale_inv);
  }
}

// The same reduction inside a cast kernel: under just-in-time scaling every workgroup of the cast pass
// derives the scale itself from the per-workgroup maxima of the abs-max pass (at most 4 KB, served from
// L2), so no launch sits between the two passes; workgroup 0 publishes abs-max, scale and 1/scale.
// Under delayed scaling in one launch (fog_quantize_delayed) the maxima are those the PREVIOUS cast of
// this tensor left behind: their maximum enters the abs-max history (a ring: entry `slot` is replaced,
// every workgroup takes the maximum over the other entries and the new value, workgroup 0 stores it),
// the scale comes from the history's maximum, and this pass's own maxima go to `cur`, 1024 words that
// the previous pass cleared; workgroup 0 clears `next` for the pass after this one.  Three buffers in
// rotation: no word is read and written by different workgroups of one launch.
struct ScaleSource {
  const uint32_t* part;   // NULL: the scale is read from memory instead
  int n, fmt, margin;
  float* amax;
  float* scale;
  float* scale_inv;
  float* hist;            // delayed scaling only (else NULL): the history, hlen entries, entry `slot` is replaced
  int hlen, slot;
  uint32_t* cur;          // delayed scaling only: where this pass's workgroup maxima are raised (atomic max)
  uint32_t* next;         // delayed scaling only: cleared by workgroup 0
};
constexpr int kDelayedSlots = 1024;
FOG_DEVICE float scale_from_partials(const ScaleSource& js, bool publisher) {
  uint32_t m = 0;
  for_words<kThreads>(js.part, js.n, -1, (int)threadIdx.x, [&](int, uint32_t v) { m = m > v ? m : v; });
  uint32_t h = 0;   // maximum of the history entries that stay
  if (js.hist) {
    for_words<kThreads>((const float*)js.hist, js.hlen, js.slot, (int)threadIdx.x, [&](int, float f) {
      const uint32_t v = __float_as_uint(f);   // abs-maxes: non-negative floats order like their bits
      h = h > v ? h : v;
    });
    if (publisher)
      for (int i = threadIdx.x; i < kDelayedSlots; i += kThreads) js.next[i] = 0u;
  }
  m = wave_max_u32(m);
  h = wave_max_u32(h);
  __shared__ uint32_t wmax[kThreads / 64], hmax[kThreads / 64];
  if ((threadIdx.x & 63) == 0) {
    wmax[threadIdx.x >> 6] = m;
    hmax[threadIdx.x >> 6] = h;
  }
  __syncthreads();
  uint32_t r = wmax[0], rh = hmax[0];
#pragma unroll
  for (int w = 1; w < kThreads / 64; ++w) {
    r = r > wmax[w] ? r : wmax[w];
    rh = rh > hmax[w] ? rh : hmax[w];
  }
  const float a = __uint_as_float(r);                       // abs-max of the tensor the maxima belong to
  const float basis = __uint_as_float(r > rh ? r : rh);     // what the scale is derived from
  float sc, si;
  scale_from_amax(basis, js.fmt, js.margin, &sc, &si);
  if (publisher && threadIdx.x == 0) {
    if (js.amax) *js.amax = a;
    if (js.hist) js.hist[js.slot] = a;
    *js.scale = sc;
    if (js.scale_inv) *js.scale_inv = si;
  }
  return sc;
}

// One workgroup of the above without a cast (empty tensors), and the maximum of one buffer of maxima.
__global__ __launch_bounds__(kThreads) void delayed_scale_only_kernel(ScaleSource js) { scale_from_partials(js, true); }
__global__ __launch_bounds__(kThreads) void partials_max_kernel(const uint32_t* __restrict__ part, int n, float* __restrict__ amax) {
  uint32_t m = 0;
  for (int i = threadIdx.x; i < n; i += kThreads) m = m > part[i] ? m : part[i];
  m = wave_max_u32(m);
  __shared__ uint32_t wmax[kThreads / 64];
  if ((threadIdx.x & 63) == 0) wmax[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t r = wmax[0];
#pragma unroll
    for (int w = 1; w < kThreads / 64; ++w) r = r > wmax[w] ? r : wmax[w];
    *amax = __uint_as_float(r);
  }
}

// One workgroup: roll the history by one (newest first), then scale from its maximum.
__global__ __launch_bounds__(kThreads) void scale_delayed_kernel(float* hist, int len, const float* new_amax, int fmt,
                                                                int margin, float* scale, float* scale_inv) {
  __shared__ float part[kThreads / 64];
  const float na = *new_amax;
  float m = 0.0f;
  // Walk the history from the back in blocks so that every element is read before it is overwritten.
  for (int base = ((len - 1) / kThreads) * kThreads; base >= 0; base -= kThreads) {
    int i = base + threadIdx.x;
    float v = 0.0f;
    bool in = i < len;
    if (in) v = i == 0 ? na : hist[i - 1];
    __syncthreads();
    if (in) hist[i] = v;
    m = fmaxf(m, v);
    __syncthreads();
  }
  m = wave_max_f32(m);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    float r = part[0];
    for (int w = 1; w < kThreads / 64; ++w) r = fmaxf(r, part[w]);
    scale_from_amax(r, fmt, margin, scale, scale_inv);
  }
}

// ---------------------------------------------------------------- cast, row-major output only
template <int FMT>
FOG_DEVICE uint2 cast8(uint4 v, float rho) {
  uint2 o;
  o.x = cvt4_fp8_nan<FMT>(bf16lo(v.x) * rho, bf16hi(v.x) * rho, bf16lo(v.y) * rho, bf16hi(v.y) * rho);
  o.y = cvt4_fp8_nan<FMT>(bf16lo(v.z) * rho, bf16hi(v.z) * rho, bf16lo(v.w) * rho, bf16hi(v.w) * rho);
  return o;
}

// Each thread turns 16 bf16 (two 16-byte loads) into 16 FP8 codes (one 16-byte store), two such
// chunks per trip so that four loads are in flight; the first trip's are requested before the scale is known, later ones before the
// chunks in hand are cast.
// REREAD: the abs-max pass of just-in-time scaling has read the tensors just before, and the memory-side cache (256 MB) holds them
// beside their codes (reread_stays below).  A tensor read for the first time keeps the non-temporal loads (512 MB read and 256 written:
// 5.9 TB/s against 4.6-5.1).
// The codes are written through: the products that follow find them in the caches, and no dirty lines are left to the kernels that run
// meanwhile.  Linear layers forward + backward, us, past the caches -> ordinary stores -> written through: 2048 x 2048 x 2048 48.8 -> 45.8
// -> 44.8, 1777 x 3088 x 2064 80.7 -> 74.5 -> 74.3, 4096 x 4096 x 4096 203.4 -> 197.0 -> 196.5, 8192 x 4096 x 14336 delayed 1111 -> 1090
// -> 1092.  The price is paid by casts that no product follows: codes take room from the bf16 tensors that the second pass reads again.
// Batches back to back on tensors that nothing has just read, us: 3 + 6 + 6 M elements 17.3 -> 20.5 -> 19.1, 8 + 16 + 16 M 37.1 -> 41.3 ->
// 41.0, 3 x 32 M 84.8 -> 97.9 -> 97.3; half or less of what the products gain.
// Workgroup `bid` of `nb` over one tensor (a whole launch, or one job's share of a batched launch).
template <int FMT, bool AMAX, bool REREAD>
FOG_DEVICE void quantize_rows_body(const uint16_t* __restrict__ x, int64_t rows, int64_t chunks_per_row, int64_t ldx,
                                   const float* __restrict__ scale, uint8_t* __restrict__ q, int64_t ldq,
                                   uint32_t* __restrict__ amax_out, const ScaleSource& js, int bid, int nb) {
  const int64_t total = rows * chunks_per_row;
  const int64_t stride = (int64_t)nb * kThreads;
  uint32_t m = 0;
  // Chunks are visited back to front: under just-in-time scaling the abs-max pass ran front to back
  // just before, so the END of the tensor is what the caches still hold.
  auto src_of = [&](int64_t i) {
    i = total - 1 - i;
    if (rows == 1) return x + i * 16;
    const int64_t r = i / chunks_per_row, c = i - r * chunks_per_row;
    return x + r * ldx + c * 16;
  };
  auto dst_of = [&](int64_t i) {
    i = total - 1 - i;
    if (rows == 1) return q + i * 16;
    const int64_t r = i / chunks_per_row, c = i - r * chunks_per_row;
    return q + r * ldq + c * 16;
  };
  auto fetch = [&](int64_t i, uint4* v) {
    if (i < total) {
      const uint16_t* p = src_of(i);
      v[0] = REREAD ? *reinterpret_cast<const uint4*>(p) : ld_nt16(p);
      v[1] = REREAD ? *reinterpret_cast<const uint4*>(p + 8) : ld_nt16(p + 8);
    }
  };
  int64_t i = (int64_t)bid * kThreads + threadIdx.x;
  uint4 v[4], nx[4];
  fetch(i, v);
  fetch(i + stride, v + 2);
  const float rho = js.part ? scale_from_partials(js, bid == 0) : *scale;
  auto emit = [&](uint4 a, uint4 b, uint8_t* dst) {
    if (AMAX) {
      m = pkmax_abs_bf16(pkmax_abs_bf16(pkmax_abs_bf16(pkmax_abs_bf16(m, a.x), a.y), a.z), a.w);
      m = pkmax_abs_bf16(pkmax_abs_bf16(pkmax_abs_bf16(pkmax_abs_bf16(m, b.x), b.y), b.z), b.w);
    }
    uint2 lo = cast8<FMT>(a, rho), hi = cast8<FMT>(b, rho);
    st_through16(dst, make_uint4(lo.x, lo.y, hi.x, hi.y));
  };
  while (i < total) {
    const int64_t n = i + 2 * stride;
    fetch(n, nx);
    fetch(n + stride, nx + 2);
    emit(v[0], v[1], dst_of(i));
    if (i + stride < total) emit(v[2], v[3], dst_of(i + stride));
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = nx[k];
    i = n;
  }
  if (AMAX) {
    uint32_t h = (m >> 16) > (m & 0xFFFFu) ? (m >> 16) : (m & 0xFFFFu);
    h = wave_max_u32(h);
    __shared__ uint32_t part[kThreads / 64];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = h;
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t r = part[0];
#pragma unroll
      for (int w = 1; w < kThreads / 64; ++w) r = r > part[w] ? r : part[w];
      if (r) atomicMax(js.cur ? js.cur + (bid & (kDelayedSlots - 1)) : amax_out, r << 16);
    }
  }
}

template <int FMT, bool AMAX, bool REREAD>
__global__ __launch_bounds__(kThreads) void quantize_rows_kernel(const uint16_t* __restrict__ x, int64_t rows,
                                                                 int64_t chunks_per_row, int64_t ldx,
                                                                 const float* __restrict__ scale, uint8_t* __restrict__ q,
                                                                 int64_t ldq, uint32_t* __restrict__ amax_out, ScaleSource js) {
  quantize_rows_body<FMT, AMAX, REREAD>(x, rows, chunks_per_row, ldx, scale, q, ldq, amax_out, js, (int)blockIdx.x, (int)gridDim.x);
}

// ---------------------------------------------------------------- several tensors per launch (just-in-time scaling)
// A launch costs about 4 us of ramp and tail whatever it does, a fifth of what the abs-max or the cast of a
// 100 MB tensor takes; fog_quantize_jit_batch therefore runs the abs-max pass of up to kBatchMax contiguous
// tensors as ONE launch and their cast pass as another.  Workgroups are dealt to the jobs by their
// sizes; inside its job a workgroup does exactly what it does in the one-tensor kernels.
constexpr int kBatchMax = FOG_CAST_BATCH_MAX;
struct BatchJobs {
  int count;
  int amax_first[kBatchMax + 1];   // first workgroup of each job in the abs-max launch (prefix sums)
  int cast_first[kBatchMax + 1];   // ... and in the cast launch, where the jobs run in reverse order
  const uint16_t* x[kBatchMax];
  int64_t n[kBatchMax];            // elements, a multiple of 16
  uint8_t* q[kBatchMax];
  int fmt[kBatchMax], margin[kBatchMax];
  float* amax[kBatchMax];
  float* scale[kBatchMax];
  float* scale_inv[kBatchMax];
};
constexpr int kJitSlots = 1024;    // workspace words per job = most workgroups a job gets in the abs-max launch

__global__ __launch_bounds__(kThreads) void amax_batch_kernel(BatchJobs b, uint32_t* __restrict__ ws) {
  int j = 0;
  for (int k = 1; k < b.count; ++k)
    if ((int)blockIdx.x >= b.amax_first[k]) j = k;
  const int nb = b.amax_first[j + 1] - b.amax_first[j];
  amax_span<true>(reinterpret_cast<const uint4*>(b.x[j]), b.n[j] / 8, nullptr, 0, ws + j * kJitSlots, (int)blockIdx.x - b.amax_first[j], nb);
}

template <bool REREAD>
__global__ __launch_bounds__(kThreads) void quantize_batch_kernel(BatchJobs b, const uint32_t* __restrict__ ws) {
  // position p in the launch order is job count - 1 - p: the tensor whose abs-max pass ran last is cast first
  int p = 0;
  for (int k = 1; k < b.count; ++k)
    if ((int)blockIdx.x >= b.cast_first[k]) p = k;
  const int j = b.count - 1 - p;
  const int bid = (int)blockIdx.x - b.cast_first[p], nb = b.cast_first[p + 1] - b.cast_first[p];
  const ScaleSource js{ws + j * kJitSlots, b.amax_first[j + 1] - b.amax_first[j], b.fmt[j], b.margin[j], b.amax[j], b.scale[j], b.scale_inv[j],
                    nullptr, 0, 0, nullptr, nullptr};
  const int64_t chunks = b.n[j] / 16;
  if (b.fmt[j] == FOG_E4M3) quantize_rows_body<FOG_E4M3, false, REREAD>(b.x[j], 1, chunks, chunks * 16, nullptr, b.q[j], chunks * 16, nullptr, js, bid, nb);
  else                      quantize_rows_body<FOG_E5M2, false, REREAD>(b.x[j], 1, chunks, chunks * 16, nullptr, b.q[j], chunks * 16, nullptr, js, bid, nb);
}

// ---------------------------------------------------------------- abs-max and cast in one launch
// Two passes read every tensor twice over the fabric (neither L2, invalid at a kernel's start, nor the memory-side cache, which is no faster,
// helps the second), 5 bytes an element in all where 3 have to move.  Here one workgroup per compute unit reads its share once, keeps 21 x 512 chunks
// of 16 elements of it in registers (44 M elements on the chip), leaves its maximum in a word of the workspace, gathers those
// of the tensor's other workgroups and casts what it holds; of a larger share the rest is read twice, as before.  A small launch in front clears the words.
// No workgroup depends on another one being resident, because beside another stream's kernel not all of them are (each fills the registers of a CU): a
// workgroup takes its share, in four pieces with a word each, with its first instruction, and one that has its own maximum and finds pieces that nobody has
// taken takes them too and casts them behind its own; a workgroup that starts later and finds its share gone ends.  So every word belongs to a
// workgroup that is running, and all waits end.  Beside attention forwards of 0 / 16 / 64 / 192 workgroups on another stream, us, two passes: 20 M elements
// 22 / 26 / 26 / 25, 67 M in four tensors 63 / 64 / 65 / 68, 134 M 123 / 126 / 127 / 130; this: 18 / 33 / 37 / 44, 48 / 56-59 / 62 / 84, 116 / 117 / 135 / 149.  (With a
// wait of 50 us before shares were taken, all workgroups asking for the same one and what a workgroup held given up for it: 19 / 39 / 175 / 105, 50 / 57 / 63 / 85,
// 117 / 120 / 137 / 151; one word a share: the same times here, 20 M alone 19.4, 117 M with a transposed copy beside 64 workgroups 187 for 151.)
// Workgroups of 256 threads, two a CU, of which one fits beside a foreign one: 5 us more at every size, for 512 words to gather.
constexpr int kHeldThreads = 512, kHeldRegs = 21;
constexpr int kPieces = 4, kHeldShares = kJitSlots / kPieces;   // a share is taken in four pieces, each with its word; shares of a tensor at most
constexpr uint32_t kMaxIsIn = 0x80000000u, kIsTaken = 0x40000000u;
struct HeldJobs {
  int first[kBatchMax + 1];   // first workgroup of each job
  int64_t total;              // elements of all jobs
  int absent;                 // for tests: that many of every absent + 1 workgroups end without having begun
};
__global__ __launch_bounds__(256) void clear_maxima_kernel(HeldJobs h, uint32_t* __restrict__ ws) {
  const int j = blockIdx.x, n = kPieces * (h.first[j + 1] - h.first[j]);
  for (int i = threadIdx.x; i < n; i += 256) ws[j * kJitSlots + i] = 0u;
}
// Raw buffer over a workgroup's share: loads past its end return zeros, so the unrolled code below needs few branches (the compiler waits for
// everything in flight behind one that holds loads).  The bounds check covers the vector offset, not the scalar one, which stays 0.
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
FOG_DEVICE __amdgpu_buffer_rsrc_t span(const void* base, int64_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, (int)bytes, 0x00020000);
}
struct HeldShared {
  uint32_t part[kHeldThreads / 64], free[kJitSlots / 64], word;
  uint16_t extra[kJitSlots], extra_to[kJitSlots];   // pieces taken besides the workgroup's own share: first, and one past the last, of each take
};
// Maximum over a workgroup's threads of packed pairs.
FOG_DEVICE uint32_t held_block_max(HeldShared& sh, uint32_t packed) {
  uint32_t r = wave_max_u32(max_of_pair(packed));
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh.part[threadIdx.x >> 6] = r;
  __syncthreads();
  r = sh.part[0];
#pragma unroll
  for (int w = 1; w < kHeldThreads / 64; ++w) r = r > sh.part[w] ? r : sh.part[w];
  return r;
}
// Takes the pieces of share `bid` that nobody has: zero in the threads of those that were free.
FOG_DEVICE uint32_t take_share(uint32_t* words, int bid) {
  uint32_t before = 1u;
  if (threadIdx.x < kPieces) before = atomicCAS(words + kPieces * bid + threadIdx.x, 0u, kIsTaken);
  return before;
}
// Whether any was (behind held_block_max's barriers, between the two calls, for all threads).
FOG_DEVICE void note_taken(HeldShared& sh, uint32_t before) {
  const uint64_t got = __ballot(before == 0u);
  if (threadIdx.x == 0) sh.word = got != 0;
}
// Leaves `own`, the maximum of this workgroup's share, in the words of the pieces that it has, takes pieces that nobody has, and returns the maximum of
// all `nb` shares.  pieces_max(i, j) is the maximum of pieces i ..< j of one share; the *extra takes stand in sh.extra and sh.extra_to.
template <typename F>
FOG_DEVICE uint32_t gather_maxima(HeldShared& sh, uint32_t* __restrict__ words, int bid, int nb, uint32_t before, uint32_t own, int* extra, F pieces_max) {
  constexpr int kWords = kJitSlots / kHeldThreads, kWaves = kHeldThreads / 64;   // words of a thread
  static_assert(kWords == 2, "the tests below name two");
  const int tid = threadIdx.x;
  *extra = 0;
  if (before == 0u) __hip_atomic_store(words + kPieces * bid + tid, kMaxIsIn | own, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  for (;;) {
    uint32_t w[kWords];
#pragma unroll
    for (int k = 0; k < kWords; ++k) {
      const int at = tid + k * kHeldThreads;
      w[k] = at < kPieces * nb ? __hip_atomic_load(words + at, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : kMaxIsIn;
    }
    if (__syncthreads_and(w[0] & w[1] & kMaxIsIn)) return held_block_max(sh, pkmax_abs_bf16(w[0] & 0x7FFFu, w[1] & 0x7FFFu));
    if (!__syncthreads_or(w[0] == 0u || w[1] == 0u)) {   // every piece has a workgroup
      __builtin_amdgcn_s_sleep(1);
      continue;
    }
    // One of the pieces that have none, if it still has none: number bid of them, so that the workgroups ask for different ones (all asking for
    // the same one queue up at its word: 100 us for 64 shares).
    uint64_t free[kWords];
#pragma unroll
    for (int k = 0; k < kWords; ++k) {
      free[k] = __ballot(w[k] == 0u);
      if ((tid & 63) == 0) sh.free[k * kWaves + (tid >> 6)] = (uint32_t)__popcll(free[k]);
    }
    __syncthreads();
    uint32_t total = 0, ahead[kWords] = {};
#pragma unroll
    for (int n = 0; n < kWords * kWaves; ++n) {
#pragma unroll
      for (int k = 0; k < kWords; ++k) ahead[k] += n < k * kWaves + (tid >> 6) ? sh.free[n] : 0u;
      total += sh.free[n];
    }
#pragma unroll
    for (int k = 0; k < kWords; ++k)
      if (w[k] == 0u && ahead[k] + (uint32_t)__popcll(free[k] & ((1ull << (tid & 63)) - 1u)) == (uint32_t)bid % total) sh.word = (uint32_t)(tid + k * kHeldThreads);
    __syncthreads();
    // It, or the two or four beside it in its share where there are that many for each workgroup that runs: a take costs 3 us whatever its size.
    const uint32_t running = (uint32_t)nb - total / kPieces;
    const int n = total <= running ? 1 : total <= 2 * running ? 2 : 4, first = (int)sh.word & -n;
    bool mine = false;
    if (tid < n) mine = atomicCAS(words + first + tid, 0u, kIsTaken) == 0u;
    const uint64_t got = __ballot(mine);
    __syncthreads();
    if (tid == 0) sh.word = (uint32_t)got;
    __syncthreads();
    if (sh.word == 0u) continue;
    const int from = first + __builtin_ctz(sh.word), to = first + 32 - __builtin_clz(sh.word);   // (a piece in between that another workgroup has is done twice)
    const uint32_t r = pieces_max(from, to);
    if (mine) __hip_atomic_store(words + first + tid, kMaxIsIn | r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (tid == 0) {
      sh.extra[*extra] = (uint16_t)from;
      sh.extra_to[*extra] = (uint16_t)to;
    }
    ++*extra;
  }
}
// Whether thread 0's workgroup is the one that has the first piece.
FOG_DEVICE bool publishes(const HeldShared& sh, int bid, uint32_t before, int extra) {
  for (int k = 0; k < extra; ++k)
    if (sh.extra[k] == 0) return true;
  return bid == 0 && before == 0u;
}
template <int N> struct Count { static constexpr int value = N; };
struct Plain { static constexpr int value = 0; };
struct Stream { static constexpr int value = 2; };   // non-temporal
template <int FMT>
FOG_DEVICE void held_body(HeldShared& sh, const BatchJobs& b, uint32_t* __restrict__ words, int j, int bid, int nb, bool plain) {
  constexpr int STEP = kHeldThreads;                                     // chunks that the workgroup takes at a time
  constexpr int REGS = kHeldRegs * STEP;                                 // chunks of the share that stay in registers
  constexpr int NL = 8, GRP = 7;
  const int tid = threadIdx.x;
  const int64_t chunks = b.n[j] / 16, per = (chunks + nb - 1) / nb;
  auto begin = [&](int i) { return per * i < chunks ? per * i : chunks; };
  const int64_t c0 = begin(bid);
  const int mine = (int)(begin(bid + 1) - c0);                           // chunks of this workgroup's share
  const uint32_t before = take_share(words, bid);   // (the answer is waited for behind the loads)
  auto part = [&](int p) { return begin(p / kPieces) + (per + kPieces - 1) / kPieces * (p % kPieces); };   // chunk that piece p begins at, if it has any
  auto part_end = [&](int p) { const int64_t end = begin(p / kPieces + 1), to = p % kPieces == kPieces - 1 ? end : part(p + 1); return to < end ? to : end; };
  auto source = [&](int64_t from, int64_t to) { return span(b.x[j] + from * 16, to > from ? (to - from) * 32 : 0); };
  const auto src = source(c0, c0 + mine);
  uint32_t m[4] = {0, 0, 0, 0};
  auto take = [&](const v4u* a) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      m[0] = pkmax_abs_bf16(m[0], a[k][0]); m[1] = pkmax_abs_bf16(m[1], a[k][1]);
      m[2] = pkmax_abs_bf16(m[2], a[k][2]); m[3] = pkmax_abs_bf16(m[3], a[k][3]);
    }
  };
  auto fetch = [&](decltype(src) from, int c, v4u* to, auto policy) __attribute__((always_inline)) {   // this thread's chunk of those from c on
    to[0] = __builtin_amdgcn_raw_buffer_load_b128(from, (c + tid) * 32, 0, decltype(policy)::value);
    to[1] = __builtin_amdgcn_raw_buffer_load_b128(from, (c + tid) * 32 + 16, 0, decltype(policy)::value);
  };
  auto walk = [&](decltype(src) from, int c, int n, auto ahead) __attribute__((always_inline)) {
    constexpr int N = decltype(ahead)::value;
    for (; c < n; c += N * STEP) {
      v4u t[N][2];
#pragma unroll
      for (int k = 0; k < N; ++k) fetch(from, c + k * STEP, t[k], Plain{});
#pragma unroll
      for (int k = 0; k < N; ++k) take(t[k]);
    }
  };
  auto block_max = [&]() __attribute__((always_inline)) {
    return held_block_max(sh, pkmax_abs_bf16(pkmax_abs_bf16(m[0], m[1]), pkmax_abs_bf16(m[2], m[3])));
  };
  walk(src, REGS, mine, Count<NL>{});
  v4u v[kHeldRegs][2];
#pragma unroll
  for (int g = 0; g < kHeldRegs; g += GRP)
    if (g * STEP < mine) {
      if (plain) {
#pragma unroll
        for (int i = g; i < g + GRP && i < kHeldRegs; ++i) fetch(src, i * STEP, v[i], Plain{});
      } else {
#pragma unroll
        for (int i = g; i < g + GRP && i < kHeldRegs; ++i) fetch(src, i * STEP, v[i], Stream{});
      }
    }
#pragma unroll
  for (int g = 0; g < kHeldRegs; g += GRP)
    if (g * STEP < mine) {
#pragma unroll
      for (int i = g; i < g + GRP && i < kHeldRegs; ++i) take(v[i]);
    }
  int extra;
  note_taken(sh, before);
  const uint32_t own = block_max();
  if (sh.word == 0u) return;   // taken while this workgroup could not start
  const uint32_t r = gather_maxima(sh, words, bid, nb, before, own, &extra, [&](int p, int q) {
    m[0] = m[1] = m[2] = m[3] = 0u;
    walk(source(part(p), part_end(q - 1)), 0, (int)(part_end(q - 1) - part(p)), Count<NL - 2>{});   // (what is held leaves registers for six)
    return block_max();
  });
  const float a = __uint_as_float(r << 16);
  float rho, inv;
  scale_from_amax(a, FMT, b.margin[j], &rho, &inv);
  if (tid == 0 && publishes(sh, bid, before, extra)) {
    *b.amax[j] = a;
    *b.scale[j] = rho;
    if (b.scale_inv[j]) *b.scale_inv[j] = inv;
  }
  auto put = [&](int64_t at, int c, int n, uint2 lo, uint2 hi) __attribute__((always_inline)) {
    if (c + tid < n) st_through16(b.q[j] + (at + c + tid) * 16, make_uint4(lo.x, lo.y, hi.x, hi.y));
  };
  auto cast_all = [&](auto cast) __attribute__((always_inline)) {
#pragma unroll
    for (int g = 0; g < kHeldRegs; g += GRP)
      if (g * STEP < mine) {
#pragma unroll
        for (int i = g; i < g + GRP && i < kHeldRegs; ++i) put(c0, i * STEP, mine, cast(v[i][0]), cast(v[i][1]));
      }
    for (int e = -1; e < extra; ++e) {   // what is not held: of this share, and the pieces that were taken
      const int64_t at = e < 0 ? c0 : part(sh.extra[e]), to = e < 0 ? c0 + mine : part_end(sh.extra_to[e] - 1);
      const auto from = source(at, to);
      const int n = (int)(to - at);
      for (int c = e < 0 ? REGS : 0; c < n; c += NL * STEP) {
        v4u t[NL][2];
#pragma unroll
        for (int k = 0; k < NL; ++k) fetch(from, c + k * STEP, t[k], Plain{});
#pragma unroll
        for (int k = 0; k < NL; ++k) put(at, c + k * STEP, n, cast(t[k][0]), cast(t[k][1]));
      }
    }
  };
  // Finite values that fit: up to a rounding above the format's maximum, which the convert takes back (it overflows from half a step above, 464 and 61440).
  if (r < 0x7F80u && a * rho <= (FMT == FOG_E4M3 ? 449.0f : 57400.0f))
    cast_all([&](v4u t) __attribute__((always_inline)) {
      return make_uint2(cvt4_fp8_finite<FMT>(bf16lo(t[0]) * rho, bf16hi(t[0]) * rho, bf16lo(t[1]) * rho, bf16hi(t[1]) * rho),
                        cvt4_fp8_finite<FMT>(bf16lo(t[2]) * rho, bf16hi(t[2]) * rho, bf16lo(t[3]) * rho, bf16hi(t[3]) * rho));
    });
  else
    cast_all([&](v4u t) __attribute__((always_inline)) { return cast8<FMT>(make_uint4(t[0], t[1], t[2], t[3]), rho); });
}
__global__ __launch_bounds__(kHeldThreads, 2) void quantize_held_kernel(BatchJobs b, HeldJobs h, uint32_t* __restrict__ ws) {
  __shared__ HeldShared sh;
  int j = 0;
  for (int k = 1; k < b.count; ++k)
    if ((int)blockIdx.x >= h.first[k]) j = k;
  const int bid = (int)blockIdx.x - h.first[j], nb = h.first[j + 1] - h.first[j];
  if (h.absent && bid % (h.absent + 1) != 0) return;
  // Ordinary loads for tensors that are a small part of the batch: the activations of few tokens beside two weights, say, which a later kernel reads
  // again and finds in the caches then (feed-forward half of 176 tokens, 2944 x 13696: 172.9 -> 171.4 us; two passes 171.5).  Everything by ordinary
  // loads is slower: 42 M in three tensors 29.5 -> 37, 67 M in four 52 -> 57; so is every tensor of up to 2 M elements, 47 M in 32 of them 32 -> 38.
  const bool plain = 64 * b.n[j] <= h.total;
  if (b.fmt[j] == FOG_E4M3) held_body<FOG_E4M3>(sh, b, ws + j * kJitSlots, j, bid, nb, plain);
  else                      held_body<FOG_E5M2>(sh, b, ws + j * kJitSlots, j, bid, nb, plain);
}

// ---------------------------------------------------------------- several tensors per launch (delayed scaling)
// fog_quantize_delayed for up to kBatchMax contiguous tensors in ONE launch: a workgroup finds its job from the prefix
// sums and does, inside it, exactly what it does in the one-tensor launch (the history update and the scale from the
// previous pass's maxima, the cast, this pass's maxima into the job's own state).
struct DelayedJobs {
  int count;
  int first[kBatchMax + 1];        // first workgroup of each job (prefix sums)
  int prev_off, cur_off, next_off; // word offsets of the three rotating buffers inside a job's state (the same for every job)
  const uint16_t* x[kBatchMax];
  int64_t n[kBatchMax];            // elements, a multiple of 16
  uint8_t* q[kBatchMax];
  int fmt[kBatchMax], margin[kBatchMax];
  float* amax_prev[kBatchMax];
  float* scale[kBatchMax];
  float* scale_inv[kBatchMax];
  float* hist[kBatchMax];
  int hlen[kBatchMax], slot[kBatchMax];
  uint32_t* state[kBatchMax];
};

__global__ __launch_bounds__(kThreads) void quantize_delayed_batch_kernel(DelayedJobs b) {
  int j = 0;
  for (int k = 1; k < b.count; ++k)
    if ((int)blockIdx.x >= b.first[k]) j = k;
  const int bid = (int)blockIdx.x - b.first[j], nb = b.first[j + 1] - b.first[j];
  uint32_t* st = b.state[j];
  const ScaleSource js{st + b.prev_off, kDelayedSlots, b.fmt[j], b.margin[j], b.amax_prev[j], b.scale[j], b.scale_inv[j],
                       b.hist[j], b.hlen[j], b.slot[j], st + b.cur_off, st + b.next_off};
  const int64_t chunks = b.n[j] / 16;
  if (b.fmt[j] == FOG_E4M3) quantize_rows_body<FOG_E4M3, true, false>(b.x[j], 1, chunks, chunks * 16, nullptr, b.q[j], chunks * 16, st + b.cur_off, js, bid, nb);
  else                      quantize_rows_body<FOG_E5M2, true, false>(b.x[j], 1, chunks, chunks * 16, nullptr, b.q[j], chunks * 16, st + b.cur_off, js, bid, nb);
}

// ---------------------------------------------------------------- cast fused with transpose
// One workgroup handles a 128 x 128 element tile.  A thread owns units of 4 rows x 8 columns:
// it loads 16 bytes from each of four consecutive rows, casts, stores 8 code bytes per row to q,
// transposes the 4 x 8 code block in registers (byte permutes) and parks the eight resulting
// dwords (4 rows of one column each) in an LDS tile that is column-major; the tile is then
// streamed out to qT in 16-byte pieces.  LDS 16-byte chunks are XOR-swizzled by column group so
// that neither the dword writes nor the 16-byte reads pile onto the same banks.
constexpr int kTile = 128;

FOG_DEVICE void transpose4x4(uint32_t r0, uint32_t r1, uint32_t r2, uint32_t r3, uint32_t* t) {
  uint32_t lo01 = __builtin_amdgcn_perm(r1, r0, 0x05010400u);  // r0.b0 r1.b0 r0.b1 r1.b1
  uint32_t hi01 = __builtin_amdgcn_perm(r1, r0, 0x07030602u);  // r0.b2 r1.b2 r0.b3 r1.b3
  uint32_t lo23 = __builtin_amdgcn_perm(r3, r2, 0x05010400u);
  uint32_t hi23 = __builtin_amdgcn_perm(r3, r2, 0x07030602u);
  t[0] = __builtin_amdgcn_perm(lo23, lo01, 0x05040100u);
  t[1] = __builtin_amdgcn_perm(lo23, lo01, 0x07060302u);
  t[2] = __builtin_amdgcn_perm(hi23, hi01, 0x05040100u);
  t[3] = __builtin_amdgcn_perm(hi23, hi01, 0x07060302u);
}

template <int FMT, bool AMAX, bool WRITE_Q, bool REREAD, bool THROUGH>
__global__ __launch_bounds__(kThreads) void quantize_transpose_kernel(const uint16_t* __restrict__ x, int64_t rows,
                                                                      int64_t cols, int64_t ldx,
                                                                      const float* __restrict__ scale,
                                                                      uint8_t* __restrict__ q, int64_t ldq,
                                                                      uint8_t* __restrict__ qT, int64_t ldqT,
                                                                      uint32_t* __restrict__ amax_out, int tiles_c, ScaleSource js) {
  __shared__ __attribute__((aligned(16))) uint8_t tile[kTile * kTile];  // [col][row], chunk-swizzled
  const int bid = gridDim.x - 1 - blockIdx.x;   // tiles back to front (see quantize_rows_kernel)
  const int64_t r0 = (int64_t)(bid / tiles_c) * kTile;
  const int64_t c0 = (int64_t)(bid % tiles_c) * kTile;
  // 512 units: 32 row groups x 16 column chunks, two per thread; both are requested before the scale is known
  auto unit_row = [&](int it) { return r0 + ((threadIdx.x + it * kThreads) >> 4) * 4; };
  auto unit_col = [&]() { return c0 + (threadIdx.x & 15) * 8; };
  auto unit_in = [&](int it) { return unit_row(it) < rows && unit_col() < cols; };  // rows % 4 == 0 and cols % 8 == 0 on this path
  uint4 v[2][4];
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    if (unit_in(it)) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint16_t* p = x + (unit_row(it) + k) * ldx + unit_col();
        v[it][k] = REREAD ? *reinterpret_cast<const uint4*>(p) : ld_nt16(p);
      }
    }
  }
  const float rho = js.part ? scale_from_partials(js, blockIdx.x == 0) : *scale;
  uint32_t m = 0;
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const int u = threadIdx.x + it * kThreads;
    const int cc = u & 15, rg = u >> 4;
    const int64_t r = unit_row(it), c = unit_col();
    uint2 code[4];
    if (unit_in(it)) {
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        const uint4 w = v[it][k];
        if (AMAX) m = pkmax_abs_bf16(pkmax_abs_bf16(pkmax_abs_bf16(pkmax_abs_bf16(m, w.x), w.y), w.z), w.w);
        code[k] = cast8<FMT>(w, rho);
        if (WRITE_Q) {
          if (THROUGH) st_through8(q + (r + k) * ldq + c, code[k]);
          else *reinterpret_cast<uint2*>(q + (r + k) * ldq + c) = code[k];
        }
      }
    } else {
#pragma unroll
      for (int k = 0; k < 4; ++k) code[k] = make_uint2(0u, 0u);
    }
    uint32_t t[8];
    transpose4x4(code[0].x, code[1].x, code[2].x, code[3].x, t);
    transpose4x4(code[0].y, code[1].y, code[2].y, code[3].y, t + 4);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int col = cc * 8 + j;
      const int chunk = (rg >> 2) ^ (cc & 7);
      *reinterpret_cast<uint32_t*>(tile + col * kTile + chunk * 16 + (rg & 3) * 4) = t[j];
    }
  }
  __syncthreads();
#pragma unroll
  for (int it = 0; it < 4; ++it) {
    const int idx = threadIdx.x + it * kThreads;  // 1024 pieces: 128 columns x 8 chunks of 16 rows
    const int col = idx >> 3, ch = idx & 7;
    const int64_t c = c0 + col, r = r0 + ch * 16;
    if (c < cols && r < rows) {  // rows % 16 == 0 on this path
      uint4 v = *reinterpret_cast<const uint4*>(tile + col * kTile + ((ch ^ ((col >> 3) & 7)) * 16));
      if (THROUGH) st_through16(qT + c * ldqT + r, v);
      else *reinterpret_cast<uint4*>(qT + c * ldqT + r) = v;
    }
  }
  if (AMAX) {
    uint32_t h = (m >> 16) > (m & 0xFFFFu) ? (m >> 16) : (m & 0xFFFFu);
    h = wave_max_u32(h);
    __shared__ uint32_t part[kThreads / 64];
    if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = h;
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t r = part[0];
#pragma unroll
      for (int w = 1; w < kThreads / 64; ++w) r = r > part[w] ? r : part[w];
      if (r) atomicMax(js.cur ? js.cur + (blockIdx.x & (kDelayedSlots - 1)) : amax_out, r << 16);
    }
  }
}

// The same in one launch with the abs-max, bound by the bytes over the fabric as quantize_held_kernel is: a workgroup takes a run of tiles, keeps the
// first kHeldTiles = 10 of them in registers (one unit of 4 rows x 8 columns a thread and tile, 160 registers; 42 M elements on the chip), reads those
// beyond twice, and transposes one after the other through two LDS tiles in turn, one barrier each.  Loads go through raw buffers over the tile, so that
// those of all ten are in flight at once (their descriptors do not all fit the scalar registers: 55 wait in lanes of
// vector registers).  Back to back, us, with the row-major copy / without, two passes -> this: 21 M elements 27.4 / 24.1 -> 19.5 / 18.5 (with an infinity, or a
// margin that saturates, 20.6 / 19.9; cast again from memory 32 / 30), 34 M 34.3 / 29.5 -> 27.3 / 24.1, 42 M 54.8 / 39.7 -> 31.9 / 26.8, 67 M 86.8 / 64.4 -> 76.2 / 60.3, 117 M 147.7 / 115.5 -> 116.7 / 93.5,
// 151 M 183.4 / 142.6 -> 156.9 / 124.1.  Beside attention forwards of 0 / 16 / 64 / 192 workgroups on another stream, two passes: 34 M 35 / 39 / 42 / 43, 117 M
// 150 / 154 / 157 / 159; this: 27 / 44 / 52 / 71, 117 / 125 / 151-155 / 201.
constexpr int kHeldTiles = 10;
struct HeldTranspose {
  const uint16_t* x; uint8_t* q; uint8_t* qT;
  int64_t rows, cols, ldx, ldq, ldqT;
  int tiles_c, tiles, margin, absent;
  float* amax; float* scale; float* scale_inv;
};
template <int FMT>
__global__ __launch_bounds__(kHeldThreads, 2) void quantize_held_transpose_kernel(HeldTranspose a, uint32_t* __restrict__ words) {
  __shared__ HeldShared sh;
  __shared__ __attribute__((aligned(16))) uint8_t buf[2][kTile * kTile];
  const int tid = threadIdx.x, bid = blockIdx.x, nb = gridDim.x, rg = tid >> 4, cc = tid & 15;
  const int per = (a.tiles + nb - 1) / nb;
  auto begin = [&](int i) { return per * i < a.tiles ? per * i : a.tiles; };
  const int t0 = begin(bid), mine = begin(bid + 1) - t0;
  auto part = [&](int p) { return begin(p / kPieces) + (per + kPieces - 1) / kPieces * (p % kPieces); };   // tile that piece p begins at, if it has any
  auto part_end = [&](int p) { const int end = begin(p / kPieces + 1), to = p % kPieces == kPieces - 1 ? end : part(p + 1); return to < end ? to : end; };
  if (a.absent && bid % (a.absent + 1) != 0) return;
  const uint32_t before = take_share(words, bid);   // (the answer is waited for behind the loads)
  uint32_t m = 0;
  auto take = [&](const uint4* u) __attribute__((always_inline)) {
#pragma unroll
    for (int k = 0; k < 4; ++k) m = pkmax_abs_bf16(pkmax_abs_bf16(pkmax_abs_bf16(pkmax_abs_bf16(m, u[k].x), u[k].y), u[k].z), u[k].w);
  };
  // this thread's unit of tile t: 4 rows x 8 columns, all in or all out, and then zeros, as where there is no tile
  auto fetch = [&](int t, bool there, uint4* u) __attribute__((always_inline)) {
    const int64_t r0 = (int64_t)(t / a.tiles_c) * kTile, c0 = (int64_t)(t % a.tiles_c) * kTile;
    const int64_t rn = a.rows - r0 < kTile ? a.rows - r0 : kTile, cn = a.cols - c0 < kTile ? a.cols - c0 : kTile;
    const __amdgpu_buffer_rsrc_t src = span(a.x + (there ? r0 * a.ldx + c0 : 0), there ? ((rn - 1) * a.ldx + cn) * 2 : 0);
    const bool in = 4 * rg < rn && 8 * cc < cn;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const v4u w = __builtin_amdgcn_raw_buffer_load_b128(src, in ? (int)(((4 * rg + k) * a.ldx + 8 * cc) * 2) : 0x7FFFFFF0, 0, 2);
      u[k] = make_uint4(w.x, w.y, w.z, w.w);
    }
  };
  auto walk = [&](int from, int to, auto ahead) __attribute__((always_inline)) {   // the maximum of tiles from ..< to
    constexpr int N = decltype(ahead)::value;
    for (int t = from; t < to; t += N) {
      uint4 u[N][4];
#pragma unroll
      for (int k = 0; k < N; ++k) fetch(t + k, t + k < to, u[k]);
#pragma unroll
      for (int k = 0; k < N; ++k) take(u[k]);
    }
  };
  walk(t0 + kHeldTiles, t0 + mine, Count<4>{});
  uint4 v[kHeldTiles][4];
#pragma unroll
  for (int i = 0; i < kHeldTiles; ++i)
    fetch(t0 + i, i < mine, v[i]);
#pragma unroll
  for (int i = 0; i < kHeldTiles; ++i)
    take(v[i]);
  int extra;
  note_taken(sh, before);
  const uint32_t own = held_block_max(sh, m);
  if (sh.word == 0u) return;   // taken while this workgroup could not start
  const uint32_t r = gather_maxima(sh, words, bid, nb, before, own, &extra, [&](int p, int q) {
    m = 0u;
    walk(part(p), part_end(q - 1), Count<3>{});   // (what is held leaves registers for three)
    return held_block_max(sh, m);
  });
  const float am = __uint_as_float(r << 16);
  float rho, inv;
  scale_from_amax(am, FMT, a.margin, &rho, &inv);
  if (tid == 0 && publishes(sh, bid, before, extra)) {
    *a.amax = am;
    *a.scale = rho;
    if (a.scale_inv) *a.scale_inv = inv;
  }
  // codes of a unit -> q, and the tile through LDS -> qT (one barrier a tile: the other buffer has been read before it)
  int side = 0;
  auto emit = [&](int t, const uint2* code) __attribute__((always_inline)) {
    const int64_t r0 = (int64_t)(t / a.tiles_c) * kTile, c0 = (int64_t)(t % a.tiles_c) * kTile;
    uint8_t* tile = buf[side];
    side ^= 1;
    if (a.q && r0 + 4 * rg < a.rows && c0 + 8 * cc < a.cols) {
#pragma unroll
      for (int k = 0; k < 4; ++k) st_through8(a.q + (r0 + 4 * rg + k) * a.ldq + c0 + 8 * cc, code[k]);
    }
    uint32_t w[8];
    transpose4x4(code[0].x, code[1].x, code[2].x, code[3].x, w);
    transpose4x4(code[0].y, code[1].y, code[2].y, code[3].y, w + 4);
#pragma unroll
    for (int n = 0; n < 8; ++n) *reinterpret_cast<uint32_t*>(tile + (cc * 8 + n) * kTile + ((rg >> 2) ^ (cc & 7)) * 16 + (rg & 3) * 4) = w[n];
    __syncthreads();
#pragma unroll
    for (int n = 0; n < 2; ++n) {
      const int idx = tid + n * kHeldThreads, col = idx >> 3, ch = idx & 7;   // 1024 pieces: 128 columns x 8 chunks of 16 rows
      if (c0 + col < a.cols && r0 + ch * 16 < a.rows)
        st_through16(a.qT + (c0 + col) * a.ldqT + r0 + ch * 16, *reinterpret_cast<const uint4*>(tile + col * kTile + ((ch ^ ((col >> 3) & 7)) * 16)));
    }
  };
  auto again = [&](int from, int to) __attribute__((always_inline)) {   // tiles that are not held
    uint4 u[4], next[4];
    fetch(from, from < to, u);
    for (int t = from; t < to; ++t) {
      fetch(t + 1, t + 1 < to, next);
      uint2 code[4];
#pragma unroll
      for (int k = 0; k < 4; ++k) code[k] = cast8<FMT>(u[k], rho);
      emit(t, code);
#pragma unroll
      for (int k = 0; k < 4; ++k) u[k] = next[k];
    }
  };
  auto cast_held = [&](auto cast) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kHeldTiles; ++i)
      if (i < mine) {
        uint2 code[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) code[k] = cast(v[i][k]);
        emit(t0 + i, code);
      }
  };
  if (r < 0x7F80u && am * rho <= (FMT == FOG_E4M3 ? 449.0f : 57400.0f))   // finite and within the format, as in held_body
    cast_held([&](uint4 u) __attribute__((always_inline)) {
      return make_uint2(cvt4_fp8_finite<FMT>(bf16lo(u.x) * rho, bf16hi(u.x) * rho, bf16lo(u.y) * rho, bf16hi(u.y) * rho),
                        cvt4_fp8_finite<FMT>(bf16lo(u.z) * rho, bf16hi(u.z) * rho, bf16lo(u.w) * rho, bf16hi(u.w) * rho));
    });
  else
    cast_held([&](uint4 u) __attribute__((always_inline)) { return cast8<FMT>(u, rho); });
  for (int k = -1; k < extra; ++k) again(k < 0 ? t0 + kHeldTiles : part(sh.extra[k]), k < 0 ? t0 + mine : part_end(sh.extra_to[k] - 1));
}

// ---------------------------------------------------------------- general shapes (slow, same results)
template <int FMT>
__global__ __launch_bounds__(kThreads) void quantize_general_kernel(const uint16_t* __restrict__ x, int64_t rows, int64_t cols,
                                                                    int64_t ldx, const float* __restrict__ scale,
                                                                    uint8_t* __restrict__ q, int64_t ldq,
                                                                    uint8_t* __restrict__ qT, int64_t ldqT,
                                                                    uint32_t* __restrict__ amax_out, ScaleSource js) {
  const float rho = js.part ? scale_from_partials(js, blockIdx.x == 0) : *scale;
  const int64_t total = rows * cols;
  uint32_t m = 0;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < total; i += (int64_t)gridDim.x * kThreads) {
    int64_t r = i / cols, c = i - r * cols;
    uint32_t w = x[r * ldx + c];
    uint32_t a = w & 0x7FFFu;
    m = m > a ? m : a;
    float t = bf16lo(w) * rho;
    uint8_t code = (uint8_t)(cvt4_fp8_nan<FMT>(t, t, t, t) & 0xFFu);
    if (q) q[r * ldq + c] = code;
    if (qT) qT[c * ldqT + r] = code;
  }
  if (amax_out) {
    m = wave_max_u32(m);
    if ((threadIdx.x & 63) == 0 && m) atomicMax(js.cur ? js.cur + (blockIdx.x & (kDelayedSlots - 1)) : amax_out, m << 16);
  }
}

// Whether `n` elements of bf16 that the abs-max pass has just read, and their codes, fit the memory-side cache together: the cast then
// reads with ordinary loads, which find more of them there.  Beyond, these keep lines that nobody reads again, at the cost of the codes that
// the products read next.  Linear layers forward + backward, us, three sets of tensors in turn, non-temporal -> ordinary loads: 12 M elements
// cast 46.0 -> 44.8, 16 M 77.2 -> 74.3, 48 M 196.0 -> 196.5, 80 M 349.7 -> 348.5; but 96 M 374.7 -> 379.9, 128 M 652 -> 662, 144 M
// 669 -> 692, 232 M 1102 -> 1140.
// With transposed copies, whose cast takes one tensor of a layer at a time, only up to 8 M elements: layers of 208 x 816 x 5008 62.5 ->
// 59.3, 1456 x 3088 x 1888 89.0 -> 86.5, 2048 x 2048 x 2048 61.3 -> 60.4, 4096 x 2048 x 2048 85.9 -> 85.0; but 4096 x 4096 x 4096
// 210.1 -> 211.0, 4096 x 8192 x 2048 226.5 -> 238.7, 16384 x 4096 x 4096 723 -> 762.
inline bool reread_stays(int64_t n, bool transposed) { return transposed ? n <= (int64_t)8 << 20 : 3 * n <= (int64_t)256 << 20; }

// Workgroups that cast `chunks` chunks of 16 elements (two a thread and trip), `most` at most.
inline int workgroups(int64_t chunks, int most) {
  const int64_t need = (chunks + 2 * kThreads - 1) / (2 * kThreads);
  return (int)(need < 1 ? 1 : need < most ? need : most);
}
// As one of `count` tensors of a just-in-time launch.  Every workgroup waits for the scale before it casts, so up to four tensors get
// what is resident at once (the batch kernel eight a CU, the one-tensor kernel seven), and where each workgroup has several trips to
// make, fewer.  us, 2048 a tensor -> 512: 134 MB in four tensors 58 -> 51.5, 84 MB in three 38 -> 34.4, 268 MB equal (shares of 2048
// by size: 84 MB 37).  One tensor, 2048 -> 1024 -> 512: 16 M elements 16.1 -> 16.0 -> 17.0, 32 M 28.5 -> 28.4 -> 29.5, 112 M
// 113.0 -> 109.7 -> 109.2.
inline int cast_workgroups(int64_t chunks, int count) {
  return workgroups(chunks, count == 1 || (count == 2 && chunks < (int64_t)1 << 20) ? 1024 : 512);
}
// With a scale that is there: nothing to wait for.  us, 2048 -> 512: 16 M elements 10.6 -> 11.4, 32 M 20.0 -> 19.4, 112 M 68.5 -> 62.8.
inline int plain_workgroups(int64_t chunks) { return workgroups(chunks, chunks < (int64_t)2 << 20 ? 2048 : 512); }
// Under delayed scaling, where the maxima a tensor's workgroups leave are the same words in a batch as alone (us, 2048 -> 512:
// batches of 31 MB 15.0 -> 13.5, 84 MB 28.8 -> 25.1, 101 MB 34.7 -> 29.4, 419 MB 118.5 -> 113.7) ...
inline int delayed_workgroups(int64_t chunks) { return workgroups(chunks, 512); }
// ... and where every workgroup raises the one abs-max word when it ends, one after the other (4096 x 4096 29.8 -> 16.4 us).
inline int one_word_workgroups(int64_t chunks) { return workgroups(chunks, 512); }

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

// Just-in-time casts in one launch (quantize_held_kernel) instead of an abs-max and a cast pass: from 18 M elements (70 K a compute unit) to 160 M (625 K).
// Batches back to back, us, two passes -> one launch: 8 M elements 11.7 -> 11.7, 12 M 14.3 -> 13.3, 17 M 18.9 -> 16.1, 20 M 21.8 -> 18.2, 25 M 24.8 -> 20.3
// (in two tensors 22.8 -> 19.9), 42 M in three 39.5 -> 28.6, 67 M in four 63.5 -> 49.7, 82 M 78.8 -> 66.9, 134 M 123 -> 116, 150 M 147 -> 133, 165 M 160 -> 157, 184 M 178 ->
// 168: alone it is level or ahead on either side of both lines.  Below the first it has little to give (with transposed copies nothing: 12.6 M elements 15.2 -> 16.1) and
// more to lose beside another stream's kernel (above); beyond the second three quarters are read again after all.  (Four steps of the shares in LDS besides: a share of 32
// steps 51.3 -> 50, all others up to 4 us slower, the registers spill.)
constexpr int64_t kHeldFrom = 70 << 10, kHeldTo = 625 << 10, kHeldMost = (int64_t)1 << 30;   // elements a compute unit, and in all
constexpr int64_t kHeldStride = 1 << 20;   // of rows where it transposes: a tile's byte offsets stay below 2^31
inline bool held_pays(int64_t n, int64_t cus) {
  return cus <= kHeldShares && n >= kHeldFrom * cus && n <= kHeldTo * cus;
}
// One workgroup per compute unit, dealt to the tensors by their sizes, at least one each.
inline fog_status launch_held(const BatchJobs& b, int64_t total, uint32_t* ws, hipStream_t s, int absent = 0) {
  HeldJobs h;
  h.absent = absent;
  h.total = total;
  h.first[0] = 0;
  int room = fog_compute_units() < kHeldShares ? fog_compute_units() : kHeldShares;
  for (int j = 0; j < kBatchMax; ++j) {
    int nb = 0;
    if (j < b.count) {
      const int most = room - (b.count - 1 - j);      // the others' one each
      nb = (int)((b.n[j] * room + total - 1) / total);
      nb = nb > most ? most : nb < 1 ? 1 : nb;
      total -= b.n[j];
      room -= nb;
    }
    h.first[j + 1] = h.first[j] + nb;
  }
  clear_maxima_kernel<<<b.count, 256, 0, s>>>(h, ws);
  quantize_held_kernel<<<h.first[b.count], kHeldThreads, 0, s>>>(b, h, ws);
  return fog_launch_status();
}
inline int64_t tiles_of(int64_t rows, int64_t cols) { return ((rows + kTile - 1) / kTile) * ((cols + kTile - 1) / kTile); }
// What the tiled transposing kernels take.
inline bool transpose_fits(const void* x, int64_t rows, int64_t cols, int64_t ldx, const void* q, int64_t ldq, const void* qT, int64_t ldqT) {
  return cols % 16 == 0 && rows % 16 == 0 && ldx % 16 == 0 && aligned16(x) && (!q || (ldq % 16 == 0 && aligned16(q))) && qT && ldqT % 16 == 0 &&
         aligned16(qT) && tiles_of(rows, cols) <= 0x7FFFFFFF;
}
// With a transposed copy a workgroup's time goes by tiles, filled or not (the two passes have a workgroup for each), so the same sizes (16.8 M elements 18.7
// us in two passes and 19.4 in one launch, 21 M 27.0 and 21.4; ahead at 151 M still: the figures stand at quantize_held_transpose_kernel) only where all tiles
// are held, eleven sixteenths of the tiles are tensor, or every workgroup's run has its part of full tiles, as in a tall tensor of more than a tile
// column (and not in a wide one of more than a tile row).  With the row-major copy / without, us, two passes -> one launch: 16 columns 20 M 55 / 40 -> 87 / 78, 80 M 189 / 148 ->
// 380 / 303; 64 columns (half filled) 20 M, held, 32 / 25 -> 23 / 22, but 41 M 56 / 39 -> 54 / 50, 77 M 101 / 76 -> 104 / 96; 80 (0.63) 80 M 123 / 85 -> 125 / 88;
// 96 (0.75) 40 M 55 / 39 -> 41 / 36, 80 M 117 / 83 -> 114 / 79; 176 rows (0.69) 70 M 111 / 83 -> 103 / 77; 144 columns (0.56) 40 M 77 / 51 -> 56 / 48, 144 M
// 271 / 178 -> 240 / 173; 144 rows 29 M 41 / 35 -> 39 / 36, 101 M 164 / 125 -> 192 / 152.
inline bool held_transpose_pays(int64_t rows, int64_t cols, int64_t cus) {
  const int64_t n = rows * cols, tiles = tiles_of(rows, cols);
  return held_pays(n, cus) && (tiles <= kHeldTiles * cus || (rows > cols && cols > kTile) || 16 * n >= 11 * tiles * kTile * kTile);
}
inline fog_status launch_held_transpose(HeldTranspose a, int fmt, uint32_t* ws, hipStream_t s) {
  const int cus = fog_compute_units() < kHeldShares ? fog_compute_units() : kHeldShares;
  a.tiles_c = (int)((a.cols + kTile - 1) / kTile);
  a.tiles = (int)tiles_of(a.rows, a.cols);
  const int per = (a.tiles + cus - 1) / cus, nb = (a.tiles + per - 1) / per;
  HeldJobs h{};
  h.first[1] = nb;
  clear_maxima_kernel<<<1, 256, 0, s>>>(h, ws);
  if (fmt == FOG_E4M3) quantize_held_transpose_kernel<FOG_E4M3><<<nb, kHeldThreads, 0, s>>>(a, ws);
  else                 quantize_held_transpose_kernel<FOG_E5M2><<<nb, kHeldThreads, 0, s>>>(a, ws);
  return fog_launch_status();
}

}  // namespace

// ---------------------------------------------------------------- host entry points
extern "C" fog_status fog_amax(const void* x_bf16, int64_t n, float* amax, void* stream) {
  if (!amax || (!x_bf16 && n > 0)) return FOG_ERR_NULL;
  if (n < 0) return FOG_ERR_SHAPE;
  if (n > 0 && !aligned16(x_bf16)) return FOG_ERR_ALIGN;
  hipStream_t s = (hipStream_t)stream;
  zero_u32_kernel<<<1, 1, 0, s>>>(reinterpret_cast<uint32_t*>(amax));
  if (n > 0) {
    const int64_t nvec = n / 8;
    const int ntail = (int)(n - nvec * 8);
    int64_t blocks = (nvec + kThreads * 8 - 1) / (kThreads * 8);
    if (blocks > 1024) blocks = 1024;   // 4 workgroups per CU; one atomic per workgroup
    if (blocks < 1) blocks = 1;
    amax_kernel<false><<<(int)blocks, kThreads, 0, s>>>(reinterpret_cast<const uint4*>(x_bf16), nvec,
                                                        reinterpret_cast<const uint16_t*>(x_bf16) + nvec * 8, ntail,
                                                        reinterpret_cast<uint32_t*>(amax));
  }
  return fog_launch_status();
}

extern "C" fog_status fog_scale(const float* amax, fog_fp8 fmt, int margin, float* scale, float* scale_inv, void* stream) {
  if (!amax || !scale) return FOG_ERR_NULL;
  if (fmt != FOG_E4M3 && fmt != FOG_E5M2) return FOG_ERR_UNSUPPORTED;
  if (margin < -64 || margin > 64) return FOG_ERR_SHAPE;
  scale_kernel<<<1, 1, 0, (hipStream_t)stream>>>(amax, (int)fmt, margin, scale, scale_inv);
  return fog_launch_status();
}

extern "C" fog_status fog_scale_delayed(float* history, int len, const float* new_amax, fog_fp8 fmt, int margin,
                                        float* scale, float* scale_inv, void* stream) {
  if (!history || !new_amax || !scale) return FOG_ERR_NULL;
  if (len < 1 || margin < -64 || margin > 64) return FOG_ERR_SHAPE;
  if (fmt != FOG_E4M3 && fmt != FOG_E5M2) return FOG_ERR_UNSUPPORTED;
  scale_delayed_kernel<<<1, kThreads, 0, (hipStream_t)stream>>>(history, len, new_amax, (int)fmt, margin, scale, scale_inv);
  return fog_launch_status();
}

template <int FMT>
static void launch_quantize(const uint16_t* x, int64_t rows, int64_t cols, int64_t ldx, const float* scale, uint8_t* q,
                            int64_t ldq, uint8_t* qT, int64_t ldqT, uint32_t* amax_out, hipStream_t s, ScaleSource js = ScaleSource{}) {
  const bool base_ok = cols % 16 == 0 && ldx % 16 == 0 && aligned16(x) && (!q || (ldq % 16 == 0 && aligned16(q)));
  if (!qT && base_ok) {
    int64_t r = rows, cpr = cols / 16, lx = ldx, lq = ldq;
    if (ldx == cols && ldq == cols) { cpr = rows * cpr; r = 1; }  // contiguous: one long row
    const int64_t n = r * cpr;
    const int blocks = js.cur ? delayed_workgroups(n) : amax_out ? one_word_workgroups(n) : js.part ? cast_workgroups(n, 1) : plain_workgroups(n);
#define FOG_QR(AM, RE) quantize_rows_kernel<FMT, AM, RE><<<blocks, kThreads, 0, s>>>(x, r, cpr, lx, scale, q, lq, amax_out, js)
    if (amax_out)                                     FOG_QR(true, false);
    else if (js.part && reread_stays(n * 16, false))  FOG_QR(false, true);
    else                                              FOG_QR(false, false);
#undef FOG_QR
    return;
  }
  if (transpose_fits(x, rows, cols, ldx, q, ldq, qT, ldqT)) {
    const int64_t tc = (cols + kTile - 1) / kTile;
    const int grid = (int)tiles_of(rows, cols);
    // Small tensors: writing through takes a microsecond at the end of the launch, more than the lines left dirty cost the next one (layers
    // of 240 x 384 x 320 30.1 -> 32.3 us, 512 x 512 x 512 32.6 -> 34.6; 208 x 816 x 5008 59.1 -> 59.5, 1456 x 3088 x 1888 85.9 -> 85.1).
    const bool through = rows * cols >= (int64_t)2 << 20;
#define FOG_QT(AM, WQ, RE, TH) quantize_transpose_kernel<FMT, AM, WQ, RE, TH><<<grid, kThreads, 0, s>>>(x, rows, cols, ldx, scale, q, ldq, qT, ldqT, amax_out, (int)tc, js)
#define FOG_QT2(AM, WQ, RE) do { if (through) FOG_QT(AM, WQ, RE, true); else FOG_QT(AM, WQ, RE, false); } while (0)
    if (amax_out)                                        { if (q) FOG_QT2(true, true, false);  else FOG_QT2(true, false, false); }
    else if (js.part && reread_stays(rows * cols, true)) { if (q) FOG_QT2(false, true, true);  else FOG_QT2(false, false, true); }
    else                                                 { if (q) FOG_QT2(false, true, false); else FOG_QT2(false, false, false); }
#undef FOG_QT2
#undef FOG_QT
    return;
  }
  int64_t total = rows * cols;
  int64_t blocks = (total + kThreads - 1) / kThreads;
  if (blocks > 8192) blocks = 8192;
  quantize_general_kernel<FMT><<<(int)blocks, kThreads, 0, s>>>(x, rows, cols, ldx, scale, q, ldq, qT, ldqT, amax_out, js);
}

static fog_status quantize_checks(const void* x_bf16, int64_t rows, int64_t cols, int64_t ldx, fog_fp8 fmt,
                                  const uint8_t* q, int64_t ldq, const uint8_t* qT, int64_t ldqT) {
  if (rows < 0 || cols < 0) return FOG_ERR_SHAPE;
  if (fmt != FOG_E4M3 && fmt != FOG_E5M2) return FOG_ERR_UNSUPPORTED;
  if (rows != 0 && cols != 0) {
    if (!x_bf16 || (!q && !qT)) return FOG_ERR_NULL;
    if (ldx < cols || (q && ldq < cols) || (qT && ldqT < rows)) return FOG_ERR_SHAPE;
    if ((reinterpret_cast<uintptr_t>(x_bf16) & 1u) != 0) return FOG_ERR_ALIGN;
  }
  return FOG_OK;
}

extern "C" fog_status fog_quantize(const void* x_bf16, int64_t rows, int64_t cols, int64_t ldx, fog_fp8 fmt,
                                   const float* scale, uint8_t* q, int64_t ldq, uint8_t* qT, int64_t ldqT,
                                   float* amax_out, void* stream) {
  if (!scale) return FOG_ERR_NULL;
  const fog_status st = quantize_checks(x_bf16, rows, cols, ldx, fmt, q, ldq, qT, ldqT);
  if (st != FOG_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  if (amax_out) zero_u32_kernel<<<1, 1, 0, s>>>(reinterpret_cast<uint32_t*>(amax_out));
  if (rows != 0 && cols != 0) {
    const uint16_t* x = reinterpret_cast<const uint16_t*>(x_bf16);
    uint32_t* am = reinterpret_cast<uint32_t*>(amax_out);
    if (fmt == FOG_E4M3) launch_quantize<FOG_E4M3>(x, rows, cols, ldx, scale, q, ldq, qT, ldqT, am, s);
    else                 launch_quantize<FOG_E5M2>(x, rows, cols, ldx, scale, q, ldq, qT, ldqT, am, s);
  }
  return fog_launch_status();
}

constexpr int kJitBlocks = 1024;   // workgroups of the abs-max pass = words of workspace

extern "C" size_t fog_quantize_jit_workspace(void) { return kJitBlocks * sizeof(uint32_t); }

extern "C" fog_status fog_quantize_jit(const void* x_bf16, int64_t rows, int64_t cols, int64_t ldx, fog_fp8 fmt, int margin,
                                       uint8_t* q, int64_t ldq, uint8_t* qT, int64_t ldqT,
                                       float* amax, float* scale, float* scale_inv,
                                       void* workspace, size_t workspace_bytes, void* stream) {
  if (!amax || !scale || !workspace) return FOG_ERR_NULL;
  if (workspace_bytes < fog_quantize_jit_workspace()) return FOG_ERR_WORKSPACE;
  if ((reinterpret_cast<uintptr_t>(workspace) & 3u) != 0) return FOG_ERR_ALIGN;
  if (margin < -64 || margin > 64) return FOG_ERR_SHAPE;
  const fog_status st = quantize_checks(x_bf16, rows, cols, ldx, fmt, q, ldq, qT, ldqT);
  if (st != FOG_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  const uint16_t* x = reinterpret_cast<const uint16_t*>(x_bf16);
  uint32_t* ws = reinterpret_cast<uint32_t*>(workspace);
  const int64_t n = rows * cols;
  if (!qT && (rows == 1 || (ldx == cols && ldq == cols)) && n % 16 == 0 && aligned16(x_bf16) && aligned16(q) && held_pays(n, fog_compute_units())) {
    BatchJobs b{};
    b.count = 1;
    b.x[0] = x; b.n[0] = n; b.q[0] = q; b.fmt[0] = (int)fmt; b.margin[0] = margin; b.amax[0] = amax; b.scale[0] = scale; b.scale_inv[0] = scale_inv;
    return launch_held(b, n, ws, s);
  }
  if (n > 0 && transpose_fits(x, rows, cols, ldx, q, ldq, qT, ldqT) && ldx <= kHeldStride && held_transpose_pays(rows, cols, fog_compute_units()))
    return launch_held_transpose({x, q, qT, rows, cols, ldx, ldq, ldqT, 0, 0, margin, 0, amax, scale, scale_inv}, (int)fmt, ws, s);
  int64_t blocks = 0;   // an empty tensor: no partial maxima, abs-max 0, scale 1
  if (n > 0) {
    if ((ldx == cols || rows == 1) && aligned16(x_bf16)) {
      const int64_t nvec = n / 8;
      const int ntail = (int)(n - nvec * 8);
      blocks = (nvec + kThreads * 8 - 1) / (kThreads * 8);
      if (blocks > kJitBlocks) blocks = kJitBlocks;
      if (blocks < 1) blocks = 1;
      amax_kernel<true><<<(int)blocks, kThreads, 0, s>>>(reinterpret_cast<const uint4*>(x), nvec, x + nvec * 8, ntail, ws);
    } else {
      blocks = (n + kThreads - 1) / kThreads;
      if (blocks > kJitBlocks) blocks = kJitBlocks;
      amax_strided_kernel<true><<<(int)blocks, kThreads, 0, s>>>(x, rows, cols, ldx, ws);
    }
  }
  if (n == 0) {   // nothing to cast: abs-max 0, scale 1
    scale_partials_kernel<<<1, kThreads, 0, s>>>(ws, 0, (int)fmt, margin, amax, scale, scale_inv);
    return fog_launch_status();
  }
  const ScaleSource js{ws, (int)blocks, (int)fmt, margin, amax, scale, scale_inv, nullptr, 0, 0, nullptr, nullptr};
  if (fmt == FOG_E4M3) launch_quantize<FOG_E4M3>(x, rows, cols, ldx, scale, q, ldq, qT, ldqT, nullptr, s, js);
  else                 launch_quantize<FOG_E5M2>(x, rows, cols, ldx, scale, q, ldq, qT, ldqT, nullptr, s, js);
  return fog_launch_status();
}

extern "C" size_t fog_quantize_delayed_state(void) { return 3 * kDelayedSlots * sizeof(uint32_t); }

extern "C" fog_status fog_quantize_delayed(const void* x_bf16, int64_t rows, int64_t cols, int64_t ldx, fog_fp8 fmt, int margin,
                                           float* history, int history_len, int64_t step, void* state, size_t state_bytes,
                                           uint8_t* q, int64_t ldq, uint8_t* qT, int64_t ldqT,
                                           float* amax_prev, float* scale, float* scale_inv, void* stream) {
  if (!history || !state || !scale) return FOG_ERR_NULL;
  if (state_bytes < fog_quantize_delayed_state()) return FOG_ERR_WORKSPACE;
  if ((reinterpret_cast<uintptr_t>(state) & 3u) != 0) return FOG_ERR_ALIGN;
  if (history_len < 1 || step < 0 || margin < -64 || margin > 64) return FOG_ERR_SHAPE;
  const fog_status st = quantize_checks(x_bf16, rows, cols, ldx, fmt, q, ldq, qT, ldqT);
  if (st != FOG_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  uint32_t* base = reinterpret_cast<uint32_t*>(state);
  uint32_t* prev = base + ((step + 2) % 3) * kDelayedSlots;
  uint32_t* cur = base + (step % 3) * kDelayedSlots;
  uint32_t* next = base + ((step + 1) % 3) * kDelayedSlots;
  const ScaleSource js{prev, kDelayedSlots, (int)fmt, margin, amax_prev, scale, scale_inv,
                    history, history_len, (int)(step % history_len), cur, next};
  if (rows == 0 || cols == 0) {   // nothing to cast: the history still advances, this pass's abs-max stays 0
    delayed_scale_only_kernel<<<1, kThreads, 0, s>>>(js);
    return fog_launch_status();
  }
  const uint16_t* x = reinterpret_cast<const uint16_t*>(x_bf16);
  if (fmt == FOG_E4M3) launch_quantize<FOG_E4M3>(x, rows, cols, ldx, scale, q, ldq, qT, ldqT, cur, s, js);
  else                 launch_quantize<FOG_E5M2>(x, rows, cols, ldx, scale, q, ldq, qT, ldqT, cur, s, js);
  return fog_launch_status();
}

extern "C" fog_status fog_delayed_amax(const void* state, int64_t step, float* amax, void* stream) {
  if (!state || !amax) return FOG_ERR_NULL;
  if (step < 0) return FOG_ERR_SHAPE;
  if ((reinterpret_cast<uintptr_t>(state) & 3u) != 0) return FOG_ERR_ALIGN;
  const uint32_t* cur = reinterpret_cast<const uint32_t*>(state) + (step % 3) * kDelayedSlots;
  partials_max_kernel<<<1, kThreads, 0, (hipStream_t)stream>>>(cur, kDelayedSlots, amax);
  return fog_launch_status();
}

extern "C" size_t fog_quantize_jit_batch_workspace(int count) {
  return count > 0 ? (size_t)count * kJitSlots * sizeof(uint32_t) : 0;
}

// Checks of a batch of casts and its description for the kernels (but for the workgroups of the cast pass); *total is its elements.
static fog_status batch_jobs(const fog_cast_job* jobs, int count, void* workspace, size_t workspace_bytes, BatchJobs& b, int64_t* total) {
  if (!jobs || !workspace) return FOG_ERR_NULL;
  if (count < 0 || count > kBatchMax) return FOG_ERR_SHAPE;
  if (workspace_bytes < fog_quantize_jit_batch_workspace(count)) return FOG_ERR_WORKSPACE;
  if ((reinterpret_cast<uintptr_t>(workspace) & 3u) != 0) return FOG_ERR_ALIGN;
  b.count = count;
  b.amax_first[0] = 0;
  *total = 0;
  for (int j = 0; j < count; ++j) {
    const fog_cast_job& t = jobs[j];
    if (!t.x_bf16 || !t.q || !t.amax || !t.scale) return FOG_ERR_NULL;
    if (t.rows <= 0 || t.cols <= 0 || t.margin < -64 || t.margin > 64) return FOG_ERR_SHAPE;
    if (t.fmt != FOG_E4M3 && t.fmt != FOG_E5M2) return FOG_ERR_UNSUPPORTED;
    if (!aligned16(t.x_bf16) || !aligned16(t.q)) return FOG_ERR_ALIGN;
    const int64_t n = t.rows * t.cols;
    if (n % 16 != 0) return FOG_ERR_UNSUPPORTED;
    int64_t ab = (n / 8 + kThreads * 8 - 1) / (kThreads * 8);
    if (ab > kJitSlots) ab = kJitSlots;
    b.amax_first[j + 1] = b.amax_first[j] + (int)ab;
    *total += n;
    b.x[j] = reinterpret_cast<const uint16_t*>(t.x_bf16);
    b.n[j] = n;
    b.q[j] = t.q;
    b.fmt[j] = (int)t.fmt;
    b.margin[j] = t.margin;
    b.amax[j] = t.amax;
    b.scale[j] = t.scale;
    b.scale_inv[j] = t.scale_inv;
  }
  return FOG_OK;
}

extern "C" fog_status fog_quantize_jit_batch(const fog_cast_job* jobs, int count, void* workspace, size_t workspace_bytes,
                                             void* stream) {
  if (count == 0) return FOG_OK;
  BatchJobs b;
  int64_t total;
  const fog_status st = batch_jobs(jobs, count, workspace, workspace_bytes, b, &total);
  if (st != FOG_OK) return st;
  hipStream_t s = (hipStream_t)stream;
  uint32_t* ws = reinterpret_cast<uint32_t*>(workspace);
  if (held_pays(total, fog_compute_units())) return launch_held(b, total, ws, s);
  b.cast_first[0] = 0;
  for (int p = 0; p < count; ++p) {   // launch position p casts job count - 1 - p
    const int64_t chunks = b.n[count - 1 - p] / 16;
    const int cb = cast_workgroups(chunks, count);
    b.cast_first[p + 1] = b.cast_first[p] + cb;
  }
  for (int j = count; j < kBatchMax; ++j) {
    b.amax_first[j + 1] = b.amax_first[count];
    b.cast_first[j + 1] = b.cast_first[count];
    b.x[j] = nullptr; b.n[j] = 0; b.q[j] = nullptr; b.fmt[j] = 0; b.margin[j] = 0;
    b.amax[j] = b.scale[j] = b.scale_inv[j] = nullptr;
  }
  amax_batch_kernel<<<b.amax_first[count], kThreads, 0, s>>>(b, ws);
  if (reread_stays(total, false)) quantize_batch_kernel<true><<<b.cast_first[count], kThreads, 0, s>>>(b, ws);
  else                     quantize_batch_kernel<false><<<b.cast_first[count], kThreads, 0, s>>>(b, ws);
  return fog_launch_status();
}

extern "C" fog_status fog_probe_quantize_held(const fog_cast_job* jobs, int count, void* workspace, size_t workspace_bytes, int64_t absent,
                                              void* stream) {
  if (count == 0) return FOG_OK;
  BatchJobs b;
  int64_t total;
  const fog_status st = batch_jobs(jobs, count, workspace, workspace_bytes, b, &total);
  if (st != FOG_OK) return st;
  if (absent < 0 || absent > 0xFFFF || total > kHeldMost) return FOG_ERR_SHAPE;
  return launch_held(b, total, reinterpret_cast<uint32_t*>(workspace), (hipStream_t)stream, (int)absent);
}

// Host-only helper (include/fog_probe.h): the choice above without a launch.
extern "C" fog_status fog_probe_cast_plan(int64_t rows, int64_t cols, int with_transpose, int compute_units_or_0, int* one_launch) {
  if (!one_launch) return FOG_ERR_NULL;
  if (rows < 1 || cols < 1 || rows > INT64_MAX / 32 / cols || compute_units_or_0 < 0) return FOG_ERR_SHAPE;
  const int cus = compute_units_or_0 > 0 ? compute_units_or_0 : fog_compute_units();
  *one_launch = with_transpose ? rows % 16 == 0 && cols % 16 == 0 && cols <= kHeldStride && held_transpose_pays(rows, cols, cus)
                               : rows * cols % 16 == 0 && held_pays(rows * cols, cus);
  return FOG_OK;
}

extern "C" fog_status fog_probe_quantize_held_transpose(const void* x_bf16, int64_t rows, int64_t cols, int64_t ldx, fog_fp8 fmt, int margin,
                                                        uint8_t* q, int64_t ldq, uint8_t* qT, int64_t ldqT, float* amax, float* scale,
                                                        float* scale_inv, void* workspace, size_t workspace_bytes, int64_t absent, void* stream) {
  if (!amax || !scale || !workspace || !qT) return FOG_ERR_NULL;
  if (workspace_bytes < fog_quantize_jit_workspace()) return FOG_ERR_WORKSPACE;
  if ((reinterpret_cast<uintptr_t>(workspace) & 3u) != 0) return FOG_ERR_ALIGN;
  if (margin < -64 || margin > 64 || absent < 0 || absent > 0xFFFF || rows < 1 || cols < 1) return FOG_ERR_SHAPE;
  const fog_status st = quantize_checks(x_bf16, rows, cols, ldx, fmt, q, ldq, qT, ldqT);
  if (st != FOG_OK) return st;
  if (!transpose_fits(x_bf16, rows, cols, ldx, q, ldq, qT, ldqT)) return FOG_ERR_ALIGN;
  if (rows > kHeldMost / cols || ldx > kHeldStride) return FOG_ERR_SHAPE;
  return launch_held_transpose({reinterpret_cast<const uint16_t*>(x_bf16), q, qT, rows, cols, ldx, ldq, ldqT, 0, 0, margin, (int)absent, amax, scale, scale_inv},
                               (int)fmt, reinterpret_cast<uint32_t*>(workspace), (hipStream_t)stream);
}

extern "C" fog_status fog_quantize_delayed_batch(const fog_delayed_job* jobs, int count, int64_t step, void* stream) {
  if (count == 0) return FOG_OK;
  if (!jobs) return FOG_ERR_NULL;
  if (count < 0 || count > kBatchMax || step < 0) return FOG_ERR_SHAPE;
  DelayedJobs b;
  b.count = count;
  b.first[0] = 0;
  b.prev_off = (int)((step + 2) % 3) * kDelayedSlots;
  b.cur_off = (int)(step % 3) * kDelayedSlots;
  b.next_off = (int)((step + 1) % 3) * kDelayedSlots;
  for (int j = 0; j < count; ++j) {
    const fog_delayed_job& t = jobs[j];
    if (!t.x_bf16 || !t.q || !t.history || !t.state || !t.scale) return FOG_ERR_NULL;
    if (t.rows <= 0 || t.cols <= 0 || t.history_len < 1 || t.margin < -64 || t.margin > 64) return FOG_ERR_SHAPE;
    if (t.fmt != FOG_E4M3 && t.fmt != FOG_E5M2) return FOG_ERR_UNSUPPORTED;
    if (!aligned16(t.x_bf16) || !aligned16(t.q) || (reinterpret_cast<uintptr_t>(t.state) & 3u) != 0) return FOG_ERR_ALIGN;
    if (t.state_bytes < fog_quantize_delayed_state()) return FOG_ERR_WORKSPACE;
    const int64_t n = t.rows * t.cols;
    if (n % 16 != 0) return FOG_ERR_UNSUPPORTED;
    const int cb = delayed_workgroups(n / 16);
    b.first[j + 1] = b.first[j] + cb;
    b.x[j] = reinterpret_cast<const uint16_t*>(t.x_bf16);
    b.n[j] = n;
    b.q[j] = t.q;
    b.fmt[j] = (int)t.fmt;
    b.margin[j] = t.margin;
    b.amax_prev[j] = t.amax_prev;
    b.scale[j] = t.scale;
    b.scale_inv[j] = t.scale_inv;
    b.hist[j] = t.history;
    b.hlen[j] = t.history_len;
    b.slot[j] = (int)(step % t.history_len);
    b.state[j] = reinterpret_cast<uint32_t*>(t.state);
  }
  for (int j = count; j < kBatchMax; ++j) {
    b.first[j + 1] = b.first[count];
    b.x[j] = nullptr; b.n[j] = 0; b.q[j] = nullptr; b.fmt[j] = 0; b.margin[j] = 0;
    b.amax_prev[j] = b.scale[j] = b.scale_inv[j] = b.hist[j] = nullptr;
    b.hlen[j] = 1; b.slot[j] = 0; b.state[j] = nullptr;
  }
  quantize_delayed_batch_kernel<<<b.first[count], kThreads, 0, (hipStream_t)stream>>>(b);
  return fog_launch_status();
}
