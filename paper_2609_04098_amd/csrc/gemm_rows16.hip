// Decode GEMM for at most 16 activation rows.
#include "gemm_splitk.h"

namespace nvfp4 {

// As the split-K kernel with per-wave rings (gemm_splitk.hip): the KS waves of
// a workgroup share FN 32-column weight tiles and split the reduction, wave w
// taking chunks w, w + KS, ...; each streams its weight (and activation) chunks
// through a private LDS ring and the partial sums meet in LDS.  What bounded
// that kernel at few rows was not the weight stream but the work per CU: a 32 x
// 32 MFMA step costs 32 cycles whatever the rows, and the activation of a chunk
// as much decode as a weight tile (4 x 5120 x 17408 ran at 18 GB/s per CU with
// 60 KB in flight).  Here the products are 16 x 16 x 32 MFMAs: lane (g, c) = 16
// g + c supplies block g of the chunk (8 bytes of codes, one scale) of row c
// and of weight columns c and 16 + c, so a chunk costs 17 + 34 FN decode VALU
// and 64 FN MFMA cycles instead of 33 + 33 FN and 128 FN.
//
// kQuant: the activation is quantized into LDS by every workgroup (1: given G,
// 2: dynamic), see gemm_splitk.h.
template <int KS, int FN, int kStages, bool kF32Out, int kQuant>
__global__ __launch_bounds__(KS * 64, KS < 8 ? 2 : KS / 4) void gemm_rows16_kernel(
    const uint8_t* __restrict__ a_codes, const uint8_t* __restrict__ a_scales, const float* __restrict__ a_g,
    const uint8_t* __restrict__ w_packed, const float* __restrict__ w_g, void* __restrict__ y, GemmParams p,
    DecodeQuantArgs q) {
  constexpr bool kALds = kQuant != 0;
  using L = SplitkStage<kALds ? 0 : 1, FN>;
  constexpr int kWOff = kALds ? 0 : 1;                       // first weight slot of a stage
  constexpr int kStageBytes = L::kBytes, kLw = L::kLoads;
  constexpr int kItems = FN * 128, kPerThread = (kItems + KS * 64 - 1) / (KS * 64);
  static_assert(kStages >= 2 && kStages <= 4 && (kStages - 1) * kLw < 64, "ring depth, memory counter range");
  static_assert(KS * kStages * kStageBytes >= FN * 2 * KS * 1024, "the reduction reuses the rings");
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  __shared__ __attribute__((aligned(16))) uint8_t a_static[kALds ? 9 * kDecodeFuseMaxBlocks : 16];
  const uint32_t lane = threadIdx.x & 63, wave = wave_index();
  const uint32_t r = lane & 31, h = lane >> 5;               // of a 32-row tile (DMA)
  const uint32_t c16 = lane & 15, g4 = lane >> 4;            // of a 16 x 16 x 32 product
  const uint32_t n0 = xcd_contiguous(p.tiles_n) * (FN * 32);
  uint8_t* ring = smem + wave * (kStages * kStageBytes);

  const uint32_t ap_off = r < p.M ? r * (p.K >> 1) + h * 16u : kOOB;
  const uint32_t aps_off = lane < p.M ? lane * (p.K >> 4) : kOOB;    // M <= 16: lanes 0..15 load a scale dword
  uint32_t b_off[FN], bs_off[L::kPairsB];
#pragma unroll
  for (int f = 0; f < FN; ++f) {
    const uint32_t nt = (n0 >> 5) + f;
    b_off[f] = nt < p.w_tiles ? nt * p.w_kc * 1024u + lane * 16u : kOOB;
  }
#pragma unroll
  for (int j = 0; j < L::kPairsB; ++j) {
    const uint32_t nt = (n0 >> 5) + 2 * j + h;
    bs_off[j] = (2 * j + h < (uint32_t)FN && nt < p.w_tiles) ? nt * p.w_kc * 128u + r * 4u : kOOB;
  }
  const __amdgpu_buffer_rsrc_t ra = rsrc(a_codes, p.a_code_bytes);
  const __amdgpu_buffer_rsrc_t rs = rsrc(a_scales, p.a_scale_bytes);
  const __amdgpu_buffer_rsrc_t rb = rsrc(w_packed, p.w_scale_offset);
  const __amdgpu_buffer_rsrc_t rbs = rsrc(w_packed + p.w_scale_offset, p.w_bytes - p.w_scale_offset);
  // DMA of the wave's chunk i (K index wave + KS i) into stage i % kStages;
  // chunks past the end of K re-load the last one and are never read.
  auto issue = [&](uint32_t i) {
    const uint32_t kc = wave + KS * i;
    const uint32_t kq = kc < p.chunks ? kc : p.chunks - 1;
    uint8_t* st = ring + (i % kStages) * kStageBytes;
    if constexpr (!kALds) {
      dma16(ra, st, ap_off, kq * 32u);
      dma4(rs, st + L::kScaleA, aps_off, kq * 4u);
    }
#pragma unroll
    for (int f = 0; f < FN; ++f) dma16(rb, st + (kWOff + f) * 1024, b_off[f], kq * 1024u);
#pragma unroll
    for (int j = 0; j < L::kPairsB; ++j) dma4(rbs, st + L::kScaleB + j * 256, bs_off[j], kq * 128u);
  };

  struct Regs {
    uint2 a, b[FN][2];
    uint32_t sa, sb[FN][2];
  };
  const uint8_t* as_lds = a_static + p.M * (p.K >> 1);
  // Lane (g, c): bytes [8 (g % 2), + 8) of the 16 bytes of half g / 2 of its row.
  const uint32_t rd = (g4 >> 1) * 512u + c16 * 16u + (g4 & 1u) * 8u;
  auto read_stage = [&](Regs& R, uint32_t i) {
    const uint8_t* st = ring + (i % kStages) * kStageBytes;
    if constexpr (kALds) {
      const uint32_t kc = wave + KS * i;
      const bool ok = c16 < p.M && kc < p.chunks;
      R.a = ok ? *(const uint2*)(a_static + c16 * (p.K >> 1) + kc * 32 + g4 * 8) : make_uint2(0u, 0u);
      R.sa = ok ? as_lds[c16 * (p.K >> 4) + kc * 4 + g4] : 0u;
    } else {
      R.a = *(const uint2*)(st + rd);
      R.sa = st[L::kScaleA + c16 * 4 + g4];
    }
#pragma unroll
    for (int f = 0; f < FN; ++f)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        R.b[f][j] = *(const uint2*)(st + (kWOff + f) * 1024 + j * 256 + rd);
        R.sb[f][j] = st[L::kScaleB + f * 128 + j * 64 + c16 * 4 + g4];
      }
  };

  typedef float floatx4 __attribute__((ext_vector_type(4)));
  floatx4 acc[FN][2];
#pragma unroll
  for (int f = 0; f < FN; ++f) acc[f][0] = acc[f][1] = floatx4{};
  auto scale2 = [](uint32_t s) {
    const half2v v = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(s, 1.0f, false);
    return __builtin_shufflevector(v, v, 0, 0);
  };
  auto compute = [&](const Regs& R) {
    const half2v sa = scale2(R.sa);
    const half8 a0 = decode8(R.a.x, sa), a1 = decode8(R.a.y, sa);
#pragma unroll
    for (int f = 0; f < FN; ++f)
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        const half2v sb = scale2(R.sb[f][j]);
        acc[f][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a0, decode8(R.b[f][j].x, sb), acc[f][j], 0, 0, 0);
        acc[f][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(a1, decode8(R.b[f][j].y, sb), acc[f][j], 0, 0, 0);
      }
  };

  XSlots<KS * 64> xs;
  if constexpr (kALds) {
    load_x_slots<KS * 64>(q, p, xs);
    __builtin_amdgcn_sched_barrier(0);                   // X's loads first
  }
#pragma unroll
  for (int s = 0; s < kStages; ++s) issue(s);
  float ga;
  if constexpr (kALds) {
    __shared__ uint32_t red[KS];
    ga = quantize_into_lds<KS * 64, kQuant == 2>(q, p, xs, a_static, a_static + p.M * (p.K >> 1), red);
  } else {
    ga = *a_g;
  }
  // Column scales of the sums this thread stores (item it: fragment column
  // it / 64 of 16, lane it % 64 of it).
  float alpha[kPerThread];
#pragma unroll
  for (int t = 0; t < kPerThread; ++t) {
    const uint32_t it = threadIdx.x + t * (KS * 64), col = n0 + (it >> 6) * 16u + (it & 15u);
    int s = 0;
#pragma unroll
    for (int i = 1; i < NVFP4_SEG_TABLE - 1; ++i) s += (i < p.n_seg && col >= p.seg_off[i]) ? 1 : 0;
    const float prod = ga * w_g[s];
    alpha[t] = prod == 0.0f ? 0.0f : 1.0f / prod;
  }
  Regs cur, nxt;
  __builtin_amdgcn_s_waitcnt(lds::vmcnt_imm((kStages - 1) * kLw));
  const uint32_t n_mine = wave < p.chunks ? (p.chunks - 1 - wave) / KS + 1 : 0;
  read_stage(cur, 0);
  for (uint32_t i = 0; i < n_mine; ++i) {
    __builtin_amdgcn_s_waitcnt(lds::kWaitLgkm0);         // cur read from its stage
    if (i + kStages < n_mine) {
      issue(i + kStages);                                 // refills cur's stage
      __builtin_amdgcn_s_waitcnt(lds::vmcnt_imm((kStages - 1) * kLw));   // chunk i + 1 landed
    } else {
      wait_rem<kLw, kStages - 2>((int)n_mine - 2 - (int)i);             // chunks after i + 1 stay in flight
    }
    read_stage(nxt, i + 1);
    compute(cur);
    cur = nxt;
  }
  __builtin_amdgcn_s_waitcnt(0x0F70);                     // drain this wave's DMA before the ring is reused
  __syncthreads();

  floatx4* part = reinterpret_cast<floatx4*>(smem);       // [2 FN][KS][64]
#pragma unroll
  for (int f = 0; f < FN; ++f)
#pragma unroll
    for (int j = 0; j < 2; ++j) part[((2 * f + j) * KS + wave) * 64 + lane] = acc[f][j];
  __syncthreads();
#pragma unroll
  for (int t = 0; t < kPerThread; ++t) {
    const uint32_t it = threadIdx.x + t * (KS * 64), l = it & 63u, col = n0 + (it >> 6) * 16u + (it & 15u);
    if (it >= (uint32_t)kItems || col >= p.N) continue;
    const floatx4* pi = part + (it >> 6) * (KS * 64) + l;   // its fragment column's KS partial sums
    floatx4 sum = pi[0];
#pragma unroll
    for (int w = 1; w < KS; ++w) sum += pi[w * 64];       // in wave order
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t row = (l >> 4) * 4u + i;
      if (row >= p.M) continue;
      const float v = sum[i] * alpha[t];
      if (kF32Out)
        static_cast<float*>(y)[(size_t)row * p.ldy + col] = v;
      else
        static_cast<uint16_t*>(y)[(size_t)row * p.ldy + col] = f32_to_bf16_rne(v);
    }
  }
}

template <int KS, int FN, int kStages, int kQuant>
static hipError_t launch_rows16_as(const GemmOperands& o, GemmParams p, const DecodeQuantArgs& q, bool out_f32,
                                   hipStream_t stream) {
  constexpr int kLds = KS * kStages * SplitkStage<kQuant ? 0 : 1, FN>::kBytes;
  static_assert(kLds + (kQuant ? 9 * (int)kDecodeFuseMaxBlocks : 16) + 64 <= 160 * 1024, "LDS");
  p.tiles_m = 1;
  p.tiles_n = (p.N + FN * 32 - 1) / (FN * 32);
  const dim3 grid(p.tiles_n), block(KS * 64);
  if (out_f32)
    hipLaunchKernelGGL((gemm_rows16_kernel<KS, FN, kStages, true, kQuant>), grid, block, kLds, stream, o.a_codes,
                       o.a_scales, o.a_g, o.w_packed, o.w_g, o.y, p, q);
  else
    hipLaunchKernelGGL((gemm_rows16_kernel<KS, FN, kStages, false, kQuant>), grid, block, kLds, stream, o.a_codes,
                       o.a_scales, o.a_g, o.w_packed, o.w_g, o.y, p, q);
  return hipGetLastError();
}

template <int kQuant>
static hipError_t launch_rows16_shape(DecodeShape shape, const GemmOperands& o, const GemmParams& p,
                                      const DecodeQuantArgs& q, bool out_f32, hipStream_t stream) {
  switch (shape) {
    case DecodeShape::kRows16w1: return launch_rows16_as<16, 1, 2, kQuant>(o, p, q, out_f32, stream);
    case DecodeShape::kRows8w2: return launch_rows16_as<8, 2, 2, kQuant>(o, p, q, out_f32, stream);
    case DecodeShape::kRows8w3: return launch_rows16_as<8, 3, 2, kQuant>(o, p, q, out_f32, stream);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_rows16(DecodeShape shape, const GemmOperands& o, const GemmParams& p, bool out_f32,
                         hipStream_t stream) {
  if (shape == DecodeShape::kRows4w2) return launch_rows16_as<4, 2, 3, 0>(o, p, DecodeQuantArgs{}, out_f32, stream);
  return launch_rows16_shape<0>(shape, o, p, DecodeQuantArgs{}, out_f32, stream);
}

hipError_t launch_rows16_quant(DecodeShape shape, const GemmOperands& o, const GemmParams& p, const DecodeQuantArgs& q,
                               bool dynamic, bool out_f32, hipStream_t stream) {
  return dynamic ? launch_rows16_shape<2>(shape, o, p, q, out_f32, stream)
                 : launch_rows16_shape<1>(shape, o, p, q, out_f32, stream);
}

}  // namespace nvfp4
