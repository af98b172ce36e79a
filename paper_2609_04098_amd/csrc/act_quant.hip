// Dynamic activation quantization to NVFP4 on gfx950 (paper, section 2
// "NVFP4"; the run-time "A4" half of W4A4).
//
// Two launches on the caller's stream (one for activations of at most
// kSmallMaxBlocks blocks, see act_quant_small_kernel), no atomics and no memset:
//   1. amax_partial: each workgroup reduces |x| over a grid-strided share of
//      X and writes one partial maximum to the workspace.  bf16 magnitudes
//      order like unsigned integers, so the reduction is packed u16 max.
//   2. quantize: every workgroup first reduces the partials to amax_X and
//      forms G = fl32(2688 / amax_X) (workgroup 0 writes it out), then each
//      thread quantizes 16-element blocks: 32 bytes of bf16 in, 8 bytes of
//      packed E2M1 codes and 1 byte of E4M3 scale out.
// In static mode pass 1 is skipped and G is read from the caller's scalar.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "launch.h"
#include "quant_device.h"

// Scratch memory of the allocation-free entry point
// (nvfp4_quantize_act_noalloc): the dynamic global scale's partial maxima,
// kActScratchBytes per device, held until the process ends.  Host code never
// uses this name as an address (it names a host-side stand-in); it takes the
// device address from hipGetSymbolAddress, once per device (act_scratch).
static __device__ __align__(256) float scratch[nvfp4::kActPartials];
static_assert(sizeof(scratch) == nvfp4::kActScratchBytes, "scratch size");

namespace nvfp4 {

constexpr int kThreads = 256;

__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    uint32_t o = __shfl_xor(v, off, 64);
    v = v > o ? v : o;
  }
  return v;
}

__device__ __forceinline__ uint32_t block_max_u32(uint32_t v, uint32_t* lds) {
  v = wave_max_u32(v);
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) lds[wave] = v;
  __syncthreads();
  uint32_t r = lds[0];
#pragma unroll
  for (int w = 1; w < kThreads / 64; ++w) r = r > lds[w] ? r : lds[w];
  __syncthreads();
  return r;
}

// Address of 16-byte vector `v` (8 bf16) of X: contiguous rows or stride ldx.
template <bool kContig>
__device__ __forceinline__ const uint4* vec_ptr(const uint16_t* x, uint32_t v, uint32_t vec_per_row,
                                                uint32_t ldx) {
  if (kContig) return reinterpret_cast<const uint4*>(x) + v;
  uint32_t row = v / vec_per_row, col = v - row * vec_per_row;
  return reinterpret_cast<const uint4*>(x + (size_t)row * ldx) + col;
}

template <bool kContig>
__global__ __launch_bounds__(kThreads) void amax_partial_kernel(const uint16_t* __restrict__ x,
                                                                uint32_t n_vec, uint32_t vec_per_row,
                                                                uint32_t ldx, float* __restrict__ partial) {
  __shared__ uint32_t lds[kThreads / 64];
  typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
  u16x2 m = {0, 0};
  const uint32_t stride = gridDim.x * kThreads;
  uint32_t v = blockIdx.x * kThreads + threadIdx.x;
  // Four independent 16-byte loads in flight per thread.
  for (; v + 3 * stride < n_vec; v += 4 * stride) {
    uint4 d[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) d[u] = *vec_ptr<kContig>(x, v + u * stride, vec_per_row, ldx);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, d[u].x & 0x7FFF7FFFu));
      m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, d[u].y & 0x7FFF7FFFu));
      m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, d[u].z & 0x7FFF7FFFu));
      m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, d[u].w & 0x7FFF7FFFu));
    }
  }
  for (; v < n_vec; v += stride) {
    uint4 d = *vec_ptr<kContig>(x, v, vec_per_row, ldx);
    m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, d.x & 0x7FFF7FFFu));
    m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, d.y & 0x7FFF7FFFu));
    m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, d.z & 0x7FFF7FFFu));
    m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, d.w & 0x7FFF7FFFu));
  }
  uint32_t mx = m[0] > m[1] ? m[0] : m[1];
  mx = block_max_u32(mx, lds);
  if (threadIdx.x == 0) partial[blockIdx.x] = __uint_as_float(mx << 16);
}

// Address of 16-element block b of X.
template <bool kContig>
__device__ __forceinline__ const uint4* block_ptr(const uint16_t* x, uint32_t b, uint32_t blocks_per_row,
                                                  uint32_t ldx) {
  if (kContig) return reinterpret_cast<const uint4*>(x) + 2 * (size_t)b;
  const uint32_t row = b / blocks_per_row, col = b - row * blocks_per_row;
  return reinterpret_cast<const uint4*>(x + (size_t)row * ldx) + 2 * col;
}

// Grid-strided loop over 16-element blocks: 32 bytes of bf16 in, 8 bytes of
// packed codes and 1 scale byte out per block.  The next block's loads are
// issued before the current block is quantized (two blocks in flight per
// thread).  (Walking the blocks from the end of X to its start after the
// amax pass, so as to meet the most recently read part of X in the MALL,
// measured 2% slower on a 335 MB activation and is not done.)
// d0, d1: the thread's first block.
template <bool kContig, QuantForm kForm>
__device__ __forceinline__ void quantize_blocks(const uint16_t* __restrict__ x, uint32_t n_blocks,
                                                uint32_t blocks_per_row, uint32_t ldx,
                                                uint8_t* __restrict__ codes, uint8_t* __restrict__ scales,
                                                float g, float gf4, uint4 d0, uint4 d1) {
  const float gd6 = g * (1.0f / 6.0f);
  const uint32_t stride = gridDim.x * kThreads;
  for (uint32_t i = blockIdx.x * kThreads + threadIdx.x; i < n_blocks; i += stride) {
    const uint32_t b = i;
    uint4 e0 = d0, e1 = d1;
    if (i + stride < n_blocks) {
      const uint4* nxt = block_ptr<kContig>(x, i + stride, blocks_per_row, ldx);
      e0 = nxt[0];
      e1 = nxt[1];
    }
    const uint32_t v[8] = {d0.x, d0.y, d0.z, d0.w, d1.x, d1.y, d1.z, d1.w};
    uint32_t c0, c1;
    const uint32_t sc = quantize_block_as<kForm>(v, g, gd6, gf4, c0, c1);
    reinterpret_cast<uint2*>(codes)[b] = make_uint2(c0, c1);
    scales[b] = (uint8_t)sc;
    d0 = e0;
    d1 = e1;
  }
}

template <bool kDynamic, bool kContig>
__global__ __launch_bounds__(kThreads) void act_quant_kernel(
    const uint16_t* __restrict__ x, uint32_t n_blocks, uint32_t blocks_per_row, uint32_t ldx,
    uint8_t* __restrict__ codes, uint8_t* __restrict__ scales, float* __restrict__ g_enc,
    const float* __restrict__ partial, uint32_t n_partial) {
  __shared__ uint32_t lds[kThreads / 64];
  // The first block is on its way while G is formed (the last block again past
  // the end).
  const uint32_t first = blockIdx.x * kThreads + threadIdx.x;
  const uint4* src = block_ptr<kContig>(x, first < n_blocks ? first : n_blocks - 1, blocks_per_row, ldx);
  const uint4 d0 = src[0], d1 = src[1];
  float g;
  if (kDynamic) {
    uint32_t m = 0;
    for (uint32_t i = threadIdx.x; i < n_partial; i += kThreads) {
      uint32_t p = __float_as_uint(partial[i]);
      m = m > p ? m : p;                       // non-negative floats order as integers
    }
    g = global_scale(__uint_as_float(block_max_u32(m, lds)));
    if (blockIdx.x == 0 && threadIdx.x == 0) *g_enc = g;
  } else {
    g = *g_enc;
  }
  // The form is chosen per tensor, uniformly across the launch.
  const QuantMode q = quant_mode(g);
  with_quant_form(q, [&](auto form) {
    quantize_blocks<kContig, decltype(form)::value>(x, n_blocks, blocks_per_row, ldx, codes, scales, g, 0.25f * q.gf,
                                                    d0, d1);
  });
}

__global__ void write_zero_scale_kernel(float* g_enc) { *g_enc = 0.0f; }

// Small activations (decode-shaped calls, up to some tens of tokens): one
// launch.  Every workgroup takes the maximum over the whole of X itself (the
// maximum is order-free, so all form the same G; workgroup 0 writes it), then
// quantizes its share of the blocks, one per thread, with the same code.  What
// bounds it is latency and the 64 bytes a clock a CU reads from L2.  GPU time
// per call, same box: one workgroup that walks all blocks 4.8 us at 2560
// blocks and 6.1 at 3840, this 3.9 and 4.0; two launches 4.8 us from 4352 to
// 16384 blocks, this 4.3 at 4352, 4.5 at 5120, 5.0 at 8000 (and one launch,
// 3.5 us of host time, less), 5.8 at 10240.
constexpr int kSmallThreads = 1024;
constexpr int kSmallLoads = 4;           // 16-byte loads in flight per thread
constexpr uint32_t kSmallMaxBlocks = 8192;

// 16-byte vectors first, first + kSmallThreads, ... of X (past the end: vector 0
// again).  Strided rows: row and column are carried along, two divisions for
// the walk instead of one per vector (4 x 5120, ldx = 2 K: 5.0 us with those, 4.2).
template <bool kContig>
struct SmallWalk {
  const uint16_t* x;
  uint32_t v, n_vec, vec_per_row, ldx, row, col, d_row, d_col;
  __device__ __forceinline__ SmallWalk(const uint16_t* x_, uint32_t first, uint32_t n_vec_, uint32_t vec_per_row_,
                                       uint32_t ldx_)
      : x(x_), v(first), n_vec(n_vec_), vec_per_row(vec_per_row_), ldx(ldx_), row(0), col(0), d_row(0), d_col(0) {
    if (kContig) return;
    row = first / vec_per_row, col = first - row * vec_per_row;
    d_row = (uint32_t)kSmallThreads / vec_per_row, d_col = (uint32_t)kSmallThreads - d_row * vec_per_row;
  }
  __device__ __forceinline__ const uint4* next() {
    const uint4* p;
    if (kContig) {
      p = reinterpret_cast<const uint4*>(x) + (v < n_vec ? v : 0);
    } else {
      const bool in = v < n_vec;
      p = reinterpret_cast<const uint4*>(x + (size_t)(in ? row : 0) * ldx) + (in ? col : 0);
      row += d_row;
      col += d_col;
      if (col >= vec_per_row) col -= vec_per_row, row += 1;
    }
    v += kSmallThreads;
    return p;
  }
};

template <bool kDynamic, bool kContig>
__global__ __launch_bounds__(kSmallThreads) void act_quant_small_kernel(
    const uint16_t* __restrict__ x, uint32_t n_blocks, uint32_t blocks_per_row, uint32_t ldx,
    uint8_t* __restrict__ codes, uint8_t* __restrict__ scales, float* __restrict__ g_enc) {
  __shared__ uint32_t lds[kSmallThreads / 64];
  const uint32_t b = blockIdx.x * kSmallThreads + threadIdx.x;
  const uint32_t bq = b < n_blocks ? b : n_blocks - 1;
  const uint4* src = block_ptr<kContig>(x, bq, blocks_per_row, ldx);
  const uint4 d0 = src[0], d1 = src[1];
  float g;
  if (kDynamic) {
    typedef unsigned short u16x2 __attribute__((ext_vector_type(2)));
    auto amax = [](u16x2 m, const uint4& d) {
      m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, d.x & 0x7FFF7FFFu));
      m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, d.y & 0x7FFF7FFFu));
      m = __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, d.z & 0x7FFF7FFFu));
      return __builtin_elementwise_max(m, __builtin_bit_cast(u16x2, d.w & 0x7FFF7FFFu));
    };
    // The thread's own block; in a single workgroup these are all of X.
    u16x2 mp = amax(amax(u16x2{0, 0}, d0), d1);
    const uint32_t n_vec = gridDim.x == 1 ? 0 : 2 * n_blocks, vec_per_row = 2 * blocks_per_row;
    SmallWalk<kContig> at(x, threadIdx.x, n_vec, vec_per_row, ldx);
    for (uint32_t v = threadIdx.x; v < n_vec; v += kSmallLoads * kSmallThreads) {
      uint4 d[kSmallLoads];
#pragma unroll
      for (int u = 0; u < kSmallLoads; ++u) d[u] = *at.next();
#pragma unroll
      for (int u = 0; u < kSmallLoads; ++u) mp = amax(mp, d[u]);
    }
    // Workgroup maximum (16 waves); bf16 magnitudes order like integers.
    uint32_t m = wave_max_u32(mp[0] > mp[1] ? mp[0] : mp[1]);
    if ((threadIdx.x & 63) == 0) lds[threadIdx.x >> 6] = m;
    __syncthreads();
    m = lds[0];
#pragma unroll
    for (int w = 1; w < kSmallThreads / 64; ++w) m = m > lds[w] ? m : lds[w];
    g = global_scale(__uint_as_float(m << 16));
    if (b == 0) *g_enc = g;
  } else {
    g = *g_enc;
  }
  const QuantMode q = quant_mode(g);                           // before any lane leaves
  if (b >= n_blocks) return;
  const uint32_t v[8] = {d0.x, d0.y, d0.z, d0.w, d1.x, d1.y, d1.z, d1.w};
  uint32_t c0, c1, sc;
  with_quant_form(q, [&](auto form) {
    sc = quantize_block_as<decltype(form)::value>(v, g, g * (1.0f / 6.0f), 0.25f * q.gf, c0, c1);
  });
  reinterpret_cast<uint2*>(codes)[b] = make_uint2(c0, c1);
  scales[b] = (uint8_t)sc;
}

static int grid_for(uint64_t work_items, int cap) {
  uint64_t g = (work_items + kThreads - 1) / kThreads;
  if (g > (uint64_t)cap) g = cap;
  return g < 1 ? 1 : (int)g;
}

hipError_t launch_act_amax(const void* x, int64_t M, int64_t K, int64_t ldx, float* partial, int* n_partial,
                           hipStream_t stream) {
  const bool contig = (ldx == K);
  const uint16_t* xp = static_cast<const uint16_t*>(x);
  const uint32_t n_vec = (uint32_t)(M * K / 8), vec_per_row = (uint32_t)(K / 8);
  *n_partial = grid_for(n_vec / 4, kActPartials);
  if (contig)
    hipLaunchKernelGGL(amax_partial_kernel<true>, dim3(*n_partial), dim3(kThreads), 0, stream, xp, n_vec,
                       vec_per_row, (uint32_t)ldx, partial);
  else
    hipLaunchKernelGGL(amax_partial_kernel<false>, dim3(*n_partial), dim3(kThreads), 0, stream, xp, n_vec,
                       vec_per_row, (uint32_t)ldx, partial);
  return hipGetLastError();
}

namespace {
constexpr int kMaxDevices = 64;
std::once_flag g_scratch_once[kMaxDevices];
float* g_scratch_ptr[kMaxDevices];
hipError_t g_scratch_err[kMaxDevices];
}  // namespace

hipError_t act_scratch(float** ptr) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  // Once per device, with that device current (the calling thread's).
  std::call_once(g_scratch_once[dev], [dev]() {
    void* p = nullptr;
    g_scratch_err[dev] = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    g_scratch_ptr[dev] = static_cast<float*>(p);
  });
  if (g_scratch_err[dev] != hipSuccess) return g_scratch_err[dev];
  *ptr = g_scratch_ptr[dev];
  return hipSuccess;
}

hipError_t launch_act_quant(const void* x, int64_t M, int64_t K, int64_t ldx, uint8_t* codes,
                            uint8_t* scales, float* g_enc, bool dynamic, float* partial,
                            hipStream_t stream) {
  if (M == 0 || K == 0) {
    if (dynamic) hipLaunchKernelGGL(write_zero_scale_kernel, dim3(1), dim3(1), 0, stream, g_enc);
    return hipGetLastError();
  }
  const bool contig = (ldx == K);
  const uint16_t* xp = static_cast<const uint16_t*>(x);
  const uint32_t n_vec = (uint32_t)(M * K / 8), vec_per_row = (uint32_t)(K / 8);
  const uint32_t n_blocks = (uint32_t)(M * K / 16), blocks_per_row = (uint32_t)(K / 16);
  if (n_blocks <= kSmallMaxBlocks) {
    const uint32_t grid = (n_blocks + kSmallThreads - 1) / kSmallThreads;
#define NVFP4_AQS(D, C)                                                                             \
  hipLaunchKernelGGL((act_quant_small_kernel<D, C>), dim3(grid), dim3(kSmallThreads), 0, stream, xp, n_blocks, \
                     blocks_per_row, (uint32_t)ldx, codes, scales, g_enc)
    if (dynamic) {
      if (contig) NVFP4_AQS(true, true); else NVFP4_AQS(true, false);
    } else {
      if (contig) NVFP4_AQS(false, true); else NVFP4_AQS(false, false);
    }
#undef NVFP4_AQS
    return hipGetLastError();
  }
  int n_partial = 0;
  if (dynamic) {
    hipError_t e = launch_act_amax(x, M, K, ldx, partial, &n_partial, stream);
    if (e != hipSuccess) return e;
  }
  const int grid = grid_for(n_blocks, kActQuantGridCap);
#define NVFP4_AQ(D, C)                                                                          \
  hipLaunchKernelGGL((act_quant_kernel<D, C>), dim3(grid), dim3(kThreads), 0, stream, xp, n_blocks, \
                     blocks_per_row, (uint32_t)ldx, codes, scales, g_enc, partial, (uint32_t)n_partial)
  if (dynamic) {
    if (contig) NVFP4_AQ(true, true); else NVFP4_AQ(true, false);
  } else {
    if (contig) NVFP4_AQ(false, true); else NVFP4_AQ(false, false);
  }
#undef NVFP4_AQ
  return hipGetLastError();
}

}  // namespace nvfp4
