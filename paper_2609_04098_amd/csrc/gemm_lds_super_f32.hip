// Prefill GEMM instantiation: LdsSquareSuper, FP32 output (see gemm_lds.h),
// its K-parts form, and the pass that sums K parts.
#include "gemm_lds.h"

namespace nvfp4 {

hipError_t launch_lds_super_f32(const GemmOperands& o, GemmParams p, uint32_t n_begin, uint32_t n_end,
                                hipStream_t stream) {
  return launch_lds_as<LdsSquareSuper, true>(o, p, n_begin, n_end, stream);
}

hipError_t launch_lds_super_parts(const GemmOperands& o, const GemmParams& p, uint32_t n_begin, uint32_t n_end,
                                  uint32_t k_parts, float* parts, hipStream_t stream) {
  return launch_lds_parts<LdsSquareSuper>(o, p, n_begin, n_end, k_parts, parts, stream);
}

// Scales of columns col .. col + 3 of Y (col + 3 may lie past N).
__device__ __forceinline__ float4 column_scales(const GemmParams& p, const float* __restrict__ a_g,
                                                const float* __restrict__ w_g, uint32_t col) {
  int s[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) s[j] = segment_of(p, col + j);
  const float first = segment_scale(a_g, w_g, s[0]);
  if (s[0] == s[3]) return make_float4(first, first, first, first);
  return make_float4(first, segment_scale(a_g, w_g, s[1]), segment_scale(a_g, w_g, s[2]), segment_scale(a_g, w_g, s[3]));
}

// The sum of a group of four columns over the parts (q: its part 0, n4 groups per
// part), in part order, times the columns' scales.  The loads of the first four
// parts are in flight while the scales are formed.
__device__ __forceinline__ float4 scaled_sum(const float4* __restrict__ q, uint32_t n4, const GemmParams& p,
                                             const float* __restrict__ a_g, const float* __restrict__ w_g,
                                             uint32_t col) {
  float4 first[4];
#pragma unroll
  for (uint32_t j = 0; j < 4; ++j)
    if (j < p.k_parts) first[j] = q[(size_t)j * n4];
  const float4 alpha = column_scales(p, a_g, w_g, col);
  float4 a = first[0];
  auto add = [&a](const float4& b) {
    a.x += b.x;
    a.y += b.y;
    a.z += b.z;
    a.w += b.w;
  };
#pragma unroll
  for (uint32_t j = 1; j < 4; ++j)
    if (j < p.k_parts) add(first[j]);
#pragma unroll 4
  for (uint32_t j = 4; j < p.k_parts; ++j) add(q[(size_t)j * n4]);
  return make_float4(a.x * alpha.x, a.y * alpha.y, a.z * alpha.z, a.w * alpha.w);
}

// Y[row, col0 + c] = (part0[row, c] + part1[row, c] + ...) * scale for c < width
// (FP32 additions in part order, one multiplication, then RNE to bf16 for bf16
// output); four columns per thread (partial rows are parts_row(width) floats;
// the padding is never stored).  y_vec: bf16 outputs whose groups of four columns
// start on 8-byte boundaries are stored 8 bytes at a time.
template <bool kF32Out>
__global__ __launch_bounds__(256) void sum_parts_kernel(const float4* __restrict__ parts, GemmParams p, uint32_t n4,
                                                        uint32_t w4, uint32_t width, const float* __restrict__ a_g,
                                                        const float* __restrict__ w_g, void* __restrict__ y,
                                                        uint32_t col0, bool y_vec) {
  for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < n4; i += gridDim.x * 256u) {
    const uint32_t row = i / w4, c = (i - row * w4) * 4u;
    const float4 sum = scaled_sum(parts + i, n4, p, a_g, w_g, col0 + c);
    const float v[4] = {sum.x, sum.y, sum.z, sum.w};
    if (kF32Out) {
      float* d = static_cast<float*>(y) + (size_t)row * p.ldy + col0 + c;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (c + j < width) d[j] = v[j];
    } else {
      uint16_t* d = static_cast<uint16_t*>(y) + (size_t)row * p.ldy + col0 + c;
      if (y_vec && c + 4 <= width) {
        *reinterpret_cast<uint2*>(d) = make_uint2(pack_bf16_rne(v[0], v[1]), pack_bf16_rne(v[2], v[3]));
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (c + j < width) d[j] = f32_to_bf16_rne(v[j]);
      }
    }
  }
}

hipError_t launch_lds_super_tile_parts(const GemmOperands& o, const GemmParams& p, uint32_t tile_begin,
                                       uint32_t tile_end, uint32_t k_parts, float* parts, hipStream_t stream) {
  GemmParams q = p;
  q.tile_begin = tile_begin;
  q.tile_count = tile_end - tile_begin;
  q.k_parts = k_parts;
  q.ldy = kSquareTile;
  GemmOperands r = o;
  r.y = parts;
  return launch_lds_as<LdsSquareSuper, true>(r, q, 0, p.N, stream);
}

// The same sum over partial tiles [k_parts][tile_count][kSquareTile][kSquareTile].
template <bool kF32Out>
__global__ __launch_bounds__(256) void sum_tiles_kernel(const float4* __restrict__ parts, GemmParams p, uint32_t n4,
                                                        const float* __restrict__ a_g, const float* __restrict__ w_g,
                                                        void* __restrict__ y, bool y_vec) {
  constexpr uint32_t kTile4 = kSquareTile * kSquareTile / 4, kRow4 = kSquareTile / 4;
  for (uint32_t i = blockIdx.x * 256u + threadIdx.x; i < n4; i += gridDim.x * 256u) {
    uint32_t tm, tn;
    tile_at<LdsSquareSuper::kGroupM>(p, p.tile_begin + i / kTile4, tm, tn);
    const uint32_t row = tm * kSquareTile + i % kTile4 / kRow4, col = tn * kSquareTile + i % kRow4 * 4u;
    if (row >= p.M || col >= p.N) continue;
    const float4 sum = scaled_sum(parts + i, n4, p, a_g, w_g, col);
    const float v[4] = {sum.x, sum.y, sum.z, sum.w};
    if (kF32Out) {
      float* d = static_cast<float*>(y) + (size_t)row * p.ldy + col;
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (col + j < p.N) d[j] = v[j];
    } else {
      uint16_t* d = static_cast<uint16_t*>(y) + (size_t)row * p.ldy + col;
      if (y_vec && col + 4 <= p.N) {
        *reinterpret_cast<uint2*>(d) = make_uint2(pack_bf16_rne(v[0], v[1]), pack_bf16_rne(v[2], v[3]));
      } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if (col + j < p.N) d[j] = f32_to_bf16_rne(v[j]);
      }
    }
  }
}

hipError_t launch_sum_tiles(const float* parts, const GemmOperands& o, const GemmParams& p, uint32_t tile_begin,
                            uint32_t tile_end, uint32_t k_parts, bool out_f32, hipStream_t stream) {
  GemmParams q = p;
  q.tiles_m = (p.M + kSquareTile - 1) / kSquareTile;
  q.tiles_n = (p.N + kSquareTile - 1) / kSquareTile;
  q.tile_begin = tile_begin;
  q.k_parts = k_parts;
  const uint32_t n4 = (tile_end - tile_begin) * (kSquareTile * kSquareTile / 4);
  const dim3 grid(n4 / 256 < 2048 ? n4 / 256 : 2048), block(256);
  const float4* p4 = reinterpret_cast<const float4*>(parts);
  const bool y_vec = p.ldy % 4 == 0 && reinterpret_cast<uintptr_t>(o.y) % 8 == 0;
  if (out_f32)
    hipLaunchKernelGGL(sum_tiles_kernel<true>, grid, block, 0, stream, p4, q, n4, o.a_g, o.w_g, o.y, false);
  else
    hipLaunchKernelGGL(sum_tiles_kernel<false>, grid, block, 0, stream, p4, q, n4, o.a_g, o.w_g, o.y, y_vec);
  return hipGetLastError();
}

hipError_t launch_sum_parts(const float* parts, const GemmOperands& o, const GemmParams& p, uint32_t k_parts,
                            uint32_t col0, bool out_f32, hipStream_t stream) {
  GemmParams q = p;
  q.k_parts = k_parts;
  const uint32_t width = p.N - col0, w4 = parts_row(width) / 4, n4 = p.M * w4;
  const uint32_t blocks = (n4 + 255) / 256;
  const dim3 grid(blocks < 2048 ? blocks : 2048), block(256);
  const float4* p4 = reinterpret_cast<const float4*>(parts);
  const bool y_vec = p.ldy % 4 == 0 && (reinterpret_cast<uintptr_t>(o.y) + col0 * 2u) % 8 == 0;
  if (out_f32)
    hipLaunchKernelGGL(sum_parts_kernel<true>, grid, block, 0, stream, p4, q, n4, w4, width, o.a_g, o.w_g, o.y, col0,
                       false);
  else
    hipLaunchKernelGGL(sum_parts_kernel<false>, grid, block, 0, stream, p4, q, n4, w4, width, o.a_g, o.w_g, o.y, col0,
                       y_vec);
  return hipGetLastError();
}

}  // namespace nvfp4
