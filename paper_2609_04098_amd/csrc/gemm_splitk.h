// Device code shared by the split-K kernels (gemm_splitk.hip, gemm_rows16.hip):
// the activation quantizer fused in front of a decode GEMM, and waits.
#pragma once

#include "gemm_common.h"

namespace nvfp4 {

// Activation quantization fused in front of the split-K GEMM, one launch,
// for decode shapes whose whole activation fits in LDS (kQuant = 1 with a
// given G, 2 with the dynamic G).  Every workgroup reads all of X (a few KB
// to a few tens of KB, from L2 after the first workgroup), takes the global
// maximum itself in dynamic mode (the maximum is order-free, so every
// workgroup forms the same G), quantizes every block with the stand-alone
// quantizer's device code into LDS, and the GEMM then reads its activation
// fragments from LDS instead of streaming them: one launch, no hand-off
// between workgroups, and the results of nvfp4_quantize_act + nvfp4_gemm
// bit for bit (same codes, same summation order).  Workgroup 0 also writes
// G and, when asked for, the codes and scales.

// Workgroup barrier for LDS data only: waits for this wave's LDS accesses,
// not for its outstanding global loads (__syncthreads' fence would also wait
// for the weight ring's DMA issued before the activation is quantized).
__device__ __forceinline__ void lds_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(lds::kWaitLgkm0);
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Maximum over the workgroup (kThreads threads) of a non-negative value.
template <int kThreads>
__device__ __forceinline__ uint32_t wg_max_u32(uint32_t v, uint32_t* red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const uint32_t o = __shfl_xor(v, off, 64);
    v = v > o ? v : o;
  }
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  lds_barrier();
  uint32_t r = red[0];
#pragma unroll
  for (int w = 1; w < kThreads / 64; ++w) r = r > red[w] ? r : red[w];
  lds_barrier();
  return r;
}

// The 8 dwords (16 bf16) of block b of X (row-major blocks, bpr per row).
__device__ __forceinline__ void load_x_block(const DecodeQuantArgs& q, uint32_t b, uint32_t bpr, uint32_t v[8]) {
  const uint32_t row = b / bpr, col = b - row * bpr;
  const uint4* src = reinterpret_cast<const uint4*>(q.x + (size_t)row * q.ldx) + 2 * col;
  const uint4 d0 = src[0], d1 = src[1];
  v[0] = d0.x; v[1] = d0.y; v[2] = d0.z; v[3] = d0.w;
  v[4] = d1.x; v[5] = d1.y; v[6] = d1.z; v[7] = d1.w;
}

// Quantize all of X into the LDS activation (codes [M][K/2], then scales
// [M][K/16]); returns G.  X has at most kDecodeFuseMaxBlocks blocks (the
// launcher's bound): each thread loads its blocks once (load_x_slots, issued
// before the weight's first ring stages, so that waiting for X does not
// wait for them too: the memory counter counts loads in issue order) and
// keeps them in registers from the maximum to the quantization.
template <int kThreads>
struct XSlots {
  static constexpr int kSlots = kDecodeFuseMaxBlocks / kThreads;
  static_assert(kSlots * kThreads == kDecodeFuseMaxBlocks, "blocks per thread");
  uint32_t v[kSlots][8];
};

template <int kThreads>
__device__ __forceinline__ void load_x_slots(const DecodeQuantArgs& q, const GemmParams& p, XSlots<kThreads>& xs) {
  const uint32_t bpr = p.K >> 4, n_blocks = p.M * bpr;
#pragma unroll
  for (int t = 0; t < XSlots<kThreads>::kSlots; ++t) {
    const uint32_t b = threadIdx.x + t * kThreads;
    if (b < n_blocks) load_x_block(q, b, bpr, xs.v[t]);
  }
}

template <int kThreads, bool kDynamic>
__device__ float quantize_into_lds(const DecodeQuantArgs& q, const GemmParams& p, XSlots<kThreads>& xs,
                                   uint8_t* lds_codes, uint8_t* lds_scales, uint32_t* red) {
  constexpr int kSlots = XSlots<kThreads>::kSlots;
  const uint32_t bpr = p.K >> 4, n_blocks = p.M * bpr;
  uint32_t (&v)[kSlots][8] = xs.v;
  uint32_t m = 0;
#pragma unroll
  for (int t = 0; t < kSlots; ++t) {
    const uint32_t b = threadIdx.x + t * kThreads;
    if (kDynamic && b < n_blocks) {
      const uint32_t a = __float_as_uint(block_amax(v[t]));
      m = m > a ? m : a;                     // non-negative floats order as integers
    }
  }
  float g;
  if (kDynamic) {
    g = global_scale(__uint_as_float(wg_max_u32<kThreads>(m, red)));
    if (blockIdx.x == 0 && threadIdx.x == 0) *q.g_enc = g;
  } else {
    g = *q.g_enc;
  }
  const float gd6 = g * (1.0f / 6.0f);
  const QuantMode qm = quant_mode(g);
  const bool out = q.codes != nullptr && blockIdx.x == 0;
  // All blocks first, then the LDS writes: a write to LDS waits for the
  // weight ring's direct-to-LDS loads issued before it (the compiler cannot
  // tell the addresses apart), so the quantization runs before that wait.
  uint32_t c[kSlots][3];
  with_quant_form(qm, [&](auto form) {
#pragma unroll
    for (int t = 0; t < kSlots; ++t)
      if (threadIdx.x + t * kThreads < n_blocks)
        c[t][2] = quantize_block_as<decltype(form)::value>(v[t], g, gd6, 0.25f * qm.gf, c[t][0], c[t][1]);
  });
#pragma unroll
  for (int t = 0; t < kSlots; ++t) {
    const uint32_t b = threadIdx.x + t * kThreads;
    if (b < n_blocks) {
      reinterpret_cast<uint2*>(lds_codes)[b] = make_uint2(c[t][0], c[t][1]);
      lds_scales[b] = (uint8_t)c[t][2];
      if (out) {
        reinterpret_cast<uint2*>(q.codes)[b] = make_uint2(c[t][0], c[t][1]);
        q.scales[b] = (uint8_t)c[t][2];
      }
    }
  }
  lds_barrier();
  return g;
}

// Wait until at most rem * kL loads of this wave are outstanding (rem <= R;
// rem < 0 waits for all).
template <int kL, int R>
__device__ __forceinline__ void wait_rem(int rem) {
  if constexpr (R <= 0) {
    __builtin_amdgcn_s_waitcnt(lds::vmcnt_imm(0));
  } else {
    if (rem >= R)
      __builtin_amdgcn_s_waitcnt(lds::vmcnt_imm(R * kL));
    else
      wait_rem<kL, R - 1>(rem);
  }
}

}  // namespace nvfp4
