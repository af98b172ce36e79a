// Split-K NVFP4 GEMM for outputs with few 32 x 32 tiles (tall-skinny gate
// projections, decode-shaped calls).
#include "gemm_splitk.h"

namespace nvfp4 {

// ----------------------------------------------------------- split-K path
//
// Shapes whose output has too few 32 x 32 tiles to give every SIMD two waves
// (N <= 96: the tall-skinny gate projections; M <= 32: decode-shaped calls;
// small outputs of plan_gemm): the KS = 4 or 8 waves of a workgroup share one FM
// x FN fragment tile and split its reduction, wave w taking chunks w, w + KS,
// ..., so that at step i the workgroup consumes chunks KS i .. KS i + KS - 1.
// The weight fragments of a wave's chunk go through a private LDS ring
// (direct-to-LDS loads, refilled as soon as the wave has read a stage).
// The activation of a step is, for each group of four waves, one 128-byte line
// group per row (4 chunks x 32 bytes of codes, 16 bytes of scales), which the
// four load together, a quarter each, into a ring they share: a wave-wide load then covers 8 whole rows instead of 32
// rows x 16 bytes, and a row's line is fetched once per group instead of
// once per wave (the per-chunk loads of 32-byte row pieces took 3-4 times
// as many memory requests as the weight).  One barrier per step: after it
// every wave's share of the next step has landed and every wave has read
// the stage about to be refilled.  Each wave reads the next chunk's raw
// fragments from LDS while it decodes and multiplies the current one, and
// the partial sums meet in LDS at the end, summed in wave order
// (deterministic).  Requires K % 64 == 0.

template <int KS, int FM, int FN, int kStages, bool kF32Out, bool kGate, int kQuant = 0, bool kShareA = true>
__global__ __launch_bounds__(KS * 64, KS < 8 ? 2 : KS / 4) void gemm_splitk_kernel(const uint8_t* __restrict__ a_codes,
                                                             const uint8_t* __restrict__ a_scales,
                                                             const float* __restrict__ a_g,
                                                             const uint8_t* __restrict__ w_packed,
                                                             const float* __restrict__ w_g,
                                                             void* __restrict__ y, GemmParams p,
                                                             DecodeQuantArgs q) {
  constexpr int BM = FM * 32, BN = FN * 32;
  // With the fused quantizer the activation sits in LDS; otherwise it is
  // streamed through the workgroup's shared ring (kShareA), or, for
  // activations of a few rows (whose loads are nearly all past the rows and
  // read nothing), through each wave's private ring beside the weight, with
  // no barrier in the loop.
  constexpr bool kALds = kQuant != 0;
  constexpr bool kAShared = !kALds && kShareA;
  constexpr bool kAPrivate = !kALds && !kShareA;
  static_assert(!kALds || FM == 1, "LDS-resident activation: one 32-row fragment");
  static_assert(KS % 4 == 0, "a step is KS / 4 128-byte line groups (4 chunks each) of every activation row");
  constexpr int G = KS / 4;                                  // groups of 4 waves, one line group each
  using L = SplitkStage<kAPrivate ? FM : 0, FN>;
  constexpr int kWOff = kAPrivate ? FM : 0;                  // first weight slot of a private stage
  using AG = SplitkAGroup<FM>;
  constexpr int kFrags = FM + FN;
  constexpr int kScaleA = L::kScaleA, kScaleB = L::kScaleB, kStageBytes = L::kBytes;
  constexpr int kLw = L::kLoads;                             // private-ring DMA loads per step and wave
  constexpr int kLa = kAShared ? AG::kLoadsPerWave : 0;      // activation DMA loads per step and wave
  constexpr int kLoads = kLw + kLa;
  constexpr int kWaitFirst = lds::vmcnt_imm((kStages - 1) * kLoads);
  static_assert(kStages >= 2 && kStages <= 4 && (kStages - 1) * kLoads + kLw < 64, "ring depth, memory counter range");
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  // The wave index is uniform: taking it through readfirstlane keeps the
  // chunk index, buffer descriptors and LDS addresses in scalar registers.
  const uint32_t lane = threadIdx.x & 63, wave = wave_index();
  const uint32_t r = lane & 31, h = lane >> 5;
  const uint32_t grp = wave >> 2, gw = wave & 3u;            // group of 4 waves, wave in the group
  uint32_t tm, tn;
  tile_of<8>(p, tm, tn);
  const uint32_t m0 = tm * BM, n0 = tn * BN;
  constexpr int kRingBytes = splitk_ring_bytes<KS, FM, FN, kStages, kAShared>() +
                             (kAPrivate ? KS * kStages * (L::kBytes - SplitkStage<0, FN>::kBytes) : 0);
  uint8_t* ring = smem + wave * (kStages * kStageBytes);
  uint8_t* a_ring = smem + KS * kStages * kStageBytes + grp * (kStages * AG::kBytes);   // the group's (kAShared)
  const uint32_t n_steps = (p.chunks + KS - 1) / KS;

  const uint32_t n_groups = (p.chunks + 3) / 4;              // line groups
  // Activation DMA of a step i: group g takes line group i G + g, wave w of
  // the group its slices q = w FM + t.
  // Codes, slice q: rows 8q .. 8q + 7 of the tile, 128 bytes each; lane l
  // takes 16-byte piece (l % 8) ^ (l / 8) ^ (q % 8) of row 8q + l / 8 and
  // lands at slot l (16 l) of the slice's 1 KB image, so that the 16 lanes
  // of one LDS read (rows r, the same piece) hit distinct banks.  Scales,
  // slice q: lane l < 32 takes dword l % 4 (chunk l % 4 of the line group) of row
  // 8q + l / 4 (4 l in the slice's 260-byte slot; lanes >= 32 read zeros).
  uint32_t ac_off[AG::kSlicesPerWave], as_off[AG::kSlicesPerWave];
#pragma unroll
  for (int t = 0; t < AG::kSlicesPerWave; ++t) {
    const uint32_t q = gw * AG::kSlicesPerWave + t;
    const uint32_t row_c = m0 + 8 * q + (lane >> 3), piece = (lane & 7) ^ (lane >> 3) ^ (q & 7);
    ac_off[t] = (kAShared && row_c < p.M) ? row_c * (p.K >> 1) + piece * 16u : kOOB;
    const uint32_t row_s = m0 + 8 * q + (lane >> 2);
    as_off[t] = (kAShared && lane < 32 && row_s < p.M) ? row_s * (p.K >> 4) + (lane & 3) * 4u : kOOB;
  }
  // Where lane (h, r) finds its activation fragment f in a shared stage:
  // row 32 f + r, piece 2 w + h (chunk w of the line group, bytes 16 h ..
  // 16 h + 15).
  uint32_t ar_code[FM], ar_scale[FM];
#pragma unroll
  for (int f = 0; f < FM; ++f) {
    const uint32_t q = 4 * f + (r >> 3), rr = r & 7;
    ar_code[f] = q * 1024u + (rr * 8u + ((2 * gw + h) ^ rr ^ (q & 7))) * 16u;
    ar_scale[f] = AG::kScaleBase + q * AG::kScaleSlot + rr * 16u + gw * 4u;
  }
  // Private-ring activation: fragment f's codes, lane (h, r) the 16 bytes
  // of row r for its chunk; scale DMA of fragment pair j, lane l the scale
  // dword of row l of the pair (the missing second fragment of an odd count
  // reads zeros).
  uint32_t ap_off[FM], aps_off[L::kPairsA > 0 ? L::kPairsA : 1];
#pragma unroll
  for (int f = 0; f < FM; ++f) {
    const uint32_t row = m0 + f * 32 + r;
    ap_off[f] = row < p.M ? row * (p.K >> 1) + h * 16u : kOOB;
  }
#pragma unroll
  for (int j = 0; j < L::kPairsA; ++j) {
    const uint32_t row = m0 + 2 * j * 32 + lane;
    aps_off[j] = (2 * j + h < (uint32_t)FM && row < p.M) ? row * (p.K >> 4) : kOOB;
  }
  // Scale DMA of weight fragment pair j: lane l loads the scale dword of row
  // l % 32 of weight tile l / 32 of the pair; the missing second fragment of
  // an odd count reads zeros.
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
  const uint8_t* w_scales = w_packed + p.w_scale_offset;
  const uint32_t w_scale_bytes = p.w_bytes - p.w_scale_offset;
  const __amdgpu_buffer_rsrc_t ra = rsrc(a_codes, p.a_code_bytes);
  const __amdgpu_buffer_rsrc_t rs = rsrc(a_scales, p.a_scale_bytes);
  const __amdgpu_buffer_rsrc_t rb = rsrc(w_packed, p.w_scale_offset);
  const __amdgpu_buffer_rsrc_t rbs = rsrc(w_scales, w_scale_bytes);
  // DMA of step i into stage i % kStages: this wave's share of its group's
  // activation line group, and the weight fragments of its chunk KS i + w.
  // (Loads of chunks past the end of K -- prologue loads when K is short, a
  // wave without a chunk in the last step -- re-load the last chunk or step
  // so that every address stays inside its tensor; they are never read.)
  auto issue_a = [&](uint32_t i) {
    if constexpr (kAShared) {
      const uint32_t lg = i * G + grp, lq = lg < n_groups ? lg : n_groups - 1;
      uint8_t* st = a_ring + (i % kStages) * AG::kBytes;
#pragma unroll
      for (int t = 0; t < AG::kSlicesPerWave; ++t) {
        const uint32_t q = gw * AG::kSlicesPerWave + t;
        dma16(ra, st + q * 1024, ac_off[t], lq * 128u);
        // Scales of chunks past the end of K read zeros: a wave without a
        // chunk in the last step then multiplies zeros into its sums.
        dma4(rs, st + AG::kScaleBase + q * AG::kScaleSlot, 4 * lg + (lane & 3) < p.chunks ? as_off[t] : kOOB,
             lq * 16u);
      }
    }
  };
  auto issue_w = [&](uint32_t i) {
    const uint32_t kc = wave + KS * i;
    const uint32_t kq = kc < p.chunks ? kc : p.chunks - 1;
    uint8_t* st = ring + (i % kStages) * kStageBytes;
    if constexpr (kAPrivate) {
#pragma unroll
      for (int f = 0; f < FM; ++f) dma16(ra, st + f * 1024, ap_off[f], kq * 32u);
#pragma unroll
      for (int j = 0; j < L::kPairsA; ++j) dma4(rs, st + kScaleA + j * 256, aps_off[j], kq * 4u);
    }
#pragma unroll
    for (int f = 0; f < FN; ++f) dma16(rb, st + (kWOff + f) * 1024, b_off[f], kq * 1024u);
#pragma unroll
    for (int j = 0; j < L::kPairsB; ++j) dma4(rbs, st + kScaleB + j * 256, bs_off[j], kq * 128u);
  };

  struct Regs {
    int4v c[kFrags];
    uint32_t s[kFrags];
  };
  // LDS-resident activation (fused quantizer): codes [M][K/2], then scales
  // [M][K/16], in a static array apart from the rings (so that its writes
  // need not wait for the ring's direct-to-LDS loads); rows >= M are zero
  // operands.
  __shared__ __attribute__((aligned(16))) uint8_t a_static[kALds ? 9 * kDecodeFuseMaxBlocks : 16];
  const uint8_t* a_lds = a_static;
  const uint8_t* as_lds = a_lds + p.M * (p.K >> 1);
  auto read_stage = [&](Regs& R, uint32_t i) {
    const uint8_t* st = ring + (i % kStages) * kStageBytes;
#pragma unroll
    for (int f = 0; f < FM; ++f) {
      if constexpr (kALds) {
        const uint32_t kc = wave + KS * i;
        const bool ok = r < p.M && kc < p.chunks;
        R.c[f] = ok ? *(const int4v*)(a_lds + r * (p.K >> 1) + kc * 32 + h * 16) : int4v{0, 0, 0, 0};
        R.s[f] = ok ? *(const uint32_t*)(as_lds + r * (p.K >> 4) + kc * 4) : 0u;
      } else if constexpr (kAPrivate) {
        R.c[f] = *(const int4v*)(st + f * 1024 + lane * 16);
        R.s[f] = *(const uint32_t*)(st + kScaleA + f * 128 + r * 4);
      } else {
        const uint8_t* as = a_ring + (i % kStages) * AG::kBytes;
        R.c[f] = *(const int4v*)(as + ar_code[f]);
        R.s[f] = *(const uint32_t*)(as + ar_scale[f]);
      }
    }
#pragma unroll
    for (int f = 0; f < FN; ++f) {
      R.c[FM + f] = *(const int4v*)(st + (kWOff + f) * 1024 + lane * 16);
      R.s[FM + f] = *(const uint32_t*)(st + kScaleB + f * 128 + r * 4);
    }
  };

  floatx16 acc[FM][FN];
#pragma unroll
  for (int fa = 0; fa < FM; ++fa)
#pragma unroll
    for (int fb = 0; fb < FN; ++fb) acc[fa][fb] = floatx16{};

  // Decode + MFMA of one chunk whose raw fragments are in cur.
  auto compute = [&](const Regs& cur) {
    half2v sc[kFrags];
#pragma unroll
    for (int f = 0; f < kFrags; ++f) sc[f] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(cur.s[f] >> (16 * h), 1.0f, false);
    half8 v[2][kFrags];
#pragma unroll
    for (int f = 0; f < kFrags; ++f) v[0][f] = decode8((uint32_t)cur.c[f][0], __builtin_shufflevector(sc[f], sc[f], 0, 0));
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int u = j & 1;
      if (j < 3) {
        const int t = (j + 1) >> 1;
#pragma unroll
        for (int f = 0; f < kFrags; ++f)
          v[u ^ 1][f] = decode8((uint32_t)cur.c[f][j + 1], t ? __builtin_shufflevector(sc[f], sc[f], 1, 1)
                                                            : __builtin_shufflevector(sc[f], sc[f], 0, 0));
      }
#pragma unroll
      for (int fa = 0; fa < FM; ++fa)
#pragma unroll
        for (int fb = 0; fb < FN; ++fb)
          acc[fa][fb] = __builtin_amdgcn_mfma_f32_32x32x16_f16(v[u][fa], v[u][FM + fb], acc[fa][fb], 0, 0, 0);
    }
  };
  // Interleave of one step: MFMAs, decode VALU, the DMA and LDS reads issued
  // after the last wait of the step.
  auto schedule = [&](auto dma_tag) {
    constexpr int kDma = decltype(dma_tag)::value;
    constexpr int kMfma = 4 * FM * FN;
    constexpr int kValu = (4 * 8 * kFrags + 2 * kFrags + kMfma - 1) / kMfma;
#pragma unroll
    for (int q = 0; q < kMfma; ++q) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                   // MFMA
      __builtin_amdgcn_sched_group_barrier(0x002, kValu, 0);                               // VALU
      if (q < kDma) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);                     // VMEM (DMA)
      if (q < 2 * kFrags) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);               // LDS read
    }
  };

  float alpha[FN];
  Regs cur, nxt;
  if constexpr (!kAShared) {
    // Private rings only, no barrier: cur's stage is free once cur is in
    // registers, so it is refilled before the wait for chunk i + 1 and
    // kStages - 1 chunks stay in flight through it.  Near the end nothing
    // is refilled, and the wait for chunk i + 1 lets exactly the chunks
    // after it stay in flight (loads land in order).  With the fused
    // quantizer the weight's first stages do not depend on the activation:
    // their loads fly while the workgroup quantizes X into LDS.
    XSlots<KS * 64> xs;
    if constexpr (kALds) {
      load_x_slots<KS * 64>(q, p, xs);
      __builtin_amdgcn_sched_barrier(0);                 // X's loads first
    }
#pragma unroll
    for (int s = 0; s < kStages; ++s) issue_w(s);
    if constexpr (kALds) {
      __shared__ uint32_t red[KS];
      uint8_t* a_dst = a_static;
      const float ga = quantize_into_lds<KS * 64, kQuant == 2>(q, p, xs, a_dst, a_dst + p.M * (p.K >> 1), red);
      segment_alpha<FN>(p, ga, w_g, n0, r, alpha);
    } else {
      segment_alpha<FN>(p, *a_g, w_g, n0, r, alpha);
    }
    __builtin_amdgcn_s_waitcnt(kWaitFirst);
    const uint32_t n_mine = wave < p.chunks ? (p.chunks - 1 - wave) / KS + 1 : 0;
    read_stage(cur, 0);
    for (uint32_t i = 0; i < n_mine; ++i) {
      __builtin_amdgcn_s_waitcnt(lds::kWaitLgkm0);       // cur read from its stage
      if (i + kStages < n_mine) {
        issue_w(i + kStages);                             // refills cur's stage
        __builtin_amdgcn_s_waitcnt(lds::vmcnt_imm((kStages - 1) * kLw));   // chunk i + 1 landed
      } else {
        wait_rem<kLw, kStages - 2>((int)n_mine - 2 - (int)i);             // chunks after i + 1
      }
      read_stage(nxt, i + 1);
      compute(cur);
      schedule(std::integral_constant<int, kLw>{});
      cur = nxt;
    }
  } else {
    // Loads are issued in the order W(0), A(0), W(1), A(1), ...: W(j) (this
    // wave's weight of step j) as soon as the wave has read the stage it
    // refills, A(j) (its share of step j's activation) after the barrier
    // that says every wave has read that stage.  Every step refills (past
    // the last step with re-loads of the last chunk, into stages nobody
    // reads again), so waiting for step i + 1 always leaves in flight the
    // loads of steps i + 2 .. i + kStages - 1 and W(i + kStages).
    constexpr int kWaitStep = lds::vmcnt_imm((kStages - 2) * kLoads + kLw);
    segment_alpha<FN>(p, *a_g, w_g, n0, r, alpha);
#pragma unroll
    for (int s = 0; s < kStages; ++s) {
      issue_w(s);
      issue_a(s);
    }
    __builtin_amdgcn_s_waitcnt(kWaitFirst);
    __builtin_amdgcn_s_barrier();                          // every wave's share of step 0 landed
    read_stage(cur, 0);
    for (uint32_t i = 0; i < n_steps; ++i) {
      __builtin_amdgcn_s_waitcnt(lds::kWaitLgkm0);       // cur read from its stages
      issue_w(i + kStages);                               // this wave's weight stage is free
      __builtin_amdgcn_s_waitcnt(kWaitStep);              // this wave's loads of step i + 1 landed
      __builtin_amdgcn_s_barrier();                       // ... everyone's; every wave has read stage i
      issue_a(i + kStages);
      read_stage(nxt, i + 1);
      compute(cur);
      schedule(std::integral_constant<int, kLa>{});
      cur = nxt;
    }
  }
  // Drain this wave's DMA (prologue loads past a short K) before the ring
  // is reused for the partial sums.
  __builtin_amdgcn_s_waitcnt(0x0F70);
  __syncthreads();

  constexpr int kFit = kRingBytes / (KS * 64 * 64);            // fragments whose partials fit the rings
  constexpr int kGroup = kFit < FM * FN ? kFit : FM * FN;
  static_assert(kGroup >= 1, "partial sums of one fragment fit the ring");
  splitk_epilogue<KS, FM, FN, kGroup, kF32Out, kGate>(acc, reinterpret_cast<float*>(smem), p, alpha, y, m0, n0,
                                                      wave, lane);
}

template <int KS, int FM, int FN, int kStages, bool kShareA>
constexpr int splitk_lds() {
  return kShareA ? splitk_ring_bytes<KS, FM, FN, kStages, true>() : KS * kStages * SplitkStage<FM, FN>::kBytes;
}

template <int KS, int FM, int FN, int kStages, bool kShareA, bool kGate>
static hipError_t launch_splitk(const GemmOperands& o, GemmParams p, bool out_f32, hipStream_t stream) {
  constexpr int BM = FM * 32, BN = FN * 32;
  constexpr int kLds = splitk_lds<KS, FM, FN, kStages, kShareA>();
  static_assert(kLds >= KS * 64 * 64 && kLds <= 160 * 1024 - 64, "the reduction reuses the rings; LDS per CU");
  p.tiles_m = (p.M + BM - 1) / BM;
  p.tiles_n = (p.N + BN - 1) / BN;
  const dim3 grid(p.tiles_m * p.tiles_n), block(KS * 64);
#define NVFP4_SK(F32)                                                                                         \
  hipLaunchKernelGGL((gemm_splitk_kernel<KS, FM, FN, kStages, F32, kGate, 0, kShareA>), grid, block, kLds, stream, \
                     o.a_codes, o.a_scales, o.a_g, o.w_packed, o.w_g, o.y, p, DecodeQuantArgs{})
  if (out_f32) NVFP4_SK(true); else NVFP4_SK(false);
#undef NVFP4_SK
  return hipGetLastError();
}

// Tall-skinny outputs (N <= 96).  While 32-row tiles leave CUs idle, eight
// waves share the reduction of a 32-row tile of as few fragments as still
// give every tile its own CU (gates at N = 96, K = 5120, same box: 1000 rows
// 33.5 -> 10.4 us, 4000 rows 34.3 -> 14.8, 8000 rows 34.5 -> 20.6 against
// 64 x 96 tiles of four waves, which keep 16 to 125 CUs busy).  Up to twice as
// many rows 32 x 96 tiles of four waves where a tile's first loads and epilogue
// weigh more than the weight's decode, which two row fragments share: with the
// quantizer in the workgroup (8300 rows 63 -> 49 us), with the gates at its end up
// to K = 8192 (16384 x 96 x 5120 33.9 -> 31.6; x 17408 71.6 against 75.5), in the
// plain product below 2048 (8300 x 96 x 64 6.7 -> 5.8, x 320 7.5 -> 6.9, x 2560 14.1
// against 14.2, 16384 x 96 x 17408 62.5 against 70.6).  Else, and beyond: 64 x 96
// tiles (32768 rows: 53.8 us, 77.8 with 32 x 96 of eight waves).  Four waves either
// way: the same order of the sums.
int narrow_fragments(int64_t M, int64_t N, int64_t K, uint32_t n_cu, NarrowUse use) {
  const uint64_t rows = (uint64_t)((M + 31) / 32), frags = (uint64_t)((N + 31) / 32);
  for (uint64_t f = 1; f <= 3; ++f)
    if (rows * ((frags + f - 1) / f) <= n_cu) return (int)f;
  const bool small = use == NarrowUse::kQuantize || K <= (use == NarrowUse::kGates ? 8192 : 2047);
  return small && rows <= 2 * (uint64_t)n_cu ? 4 : 0;
}

template <bool kGate>
static hipError_t launch_narrow(const GemmOperands& o, const GemmParams& p, bool out_f32, hipStream_t stream) {
  switch (narrow_fragments(p.M, p.N, p.K, cu_count(), kGate ? NarrowUse::kGates : NarrowUse::kProduct)) {
    case 1: return launch_splitk<8, 1, 1, 3, true, kGate>(o, p, out_f32, stream);
    case 2: return launch_splitk<8, 1, 2, 3, true, kGate>(o, p, out_f32, stream);
    case 3: return launch_splitk<8, 1, 3, 3, true, kGate>(o, p, out_f32, stream);
    case 4: return launch_splitk<4, 1, 3, 3, true, kGate>(o, p, out_f32, stream);
    default: return launch_splitk<4, 2, 3, 3, true, kGate>(o, p, out_f32, stream);
  }
}

hipError_t launch_splitk_narrow(const GemmOperands& o, GemmParams p, bool out_f32, bool gate, hipStream_t stream) {
  return gate ? launch_narrow<true>(o, p, out_f32, stream) : launch_narrow<false>(o, p, out_f32, stream);
}

constexpr int64_t kRowsMaxElems = 12 * 16384, kLongNarrowK = 2048;
// Decode shapes (M <= 32).  The order of an output column's sum follows from
// the number of waves that share it, so the fused quantize + GEMM launch
// (M * K <= 16 * kDecodeFuseMaxBlocks) takes the same form as the plain one.
// Measured, same box, W cycled through copies larger than the last-level cache:
//  * up to 16 rows (gemm_rows16_kernel).  At most one 32-column tile per CU: 16
//    waves (1 x 8192 x 5120 fused 9.1 us with 8-wave 32 x 32 tiles, 7.7 with
//    this; 4 x 5120 x 17408 18.8 with 16-wave 32 x 32 tiles, 16.1).  More: 8
//    waves and two tiles (1 x 8704 x 5120 fused 13.1 -> 10.1), three while that
//    makes no more workgroups than CUs (1 x 17408 x 5120 fused 19.1 -> 13.5, 16 x
//    17408 x 5120 18.2 -> 14.0).  Beyond, by how full the last round of workgroups
//    is: up to four tiles per CU 8 waves and two (two full rounds; 1 x 24600 x 5120
//    18.1 us, 21.9 with 4 waves and two), up to six 4 waves and two, or where every
//    workgroup quantizes X (the fused launch) 8 waves and three (4 and 16 x 34816
//    x 5120 25.1 -> 22.0 and 28.6 -> 24.3; 1 x 34816 x 5120 fused 27.4 -> 22.7, 23.8
//    with 4 waves and two), more again 8 waves and two (1 x 50000 x 17408 96 us; 124
//    with 4 waves and two).  With more X than kRowsMaxElems every 8-wave form
//    loads it more slowly: 4 waves and two tiles up to six tiles per CU (16 x 24600
//    x 17408 56.5 us; 49.7 with W in the last-level cache on 32-row tiles, 40.6
//    with this), 32-row tiles past it (16 x 50000 x 17408 123 -> 115).
//  * 17 to 32 rows, at most one tile per CU: 4 waves with per-wave rings
//    (32 x 8192 x 5120: two tiles per workgroup and a shared activation ring
//    13.7 us, this 9.7), for long K 8 waves with a shared ring (32 x 5120 x
//    17408 35.5 -> 21.2).
//  * more tiles: a shared activation ring and as many tiles per workgroup as
//    bring the workgroups to between 0.6 of the CUs and one each: the
//    activation's decode and loads are shared by them (32 x 17408 x 5120, 8
//    waves and three tiles: 15.1 us against 16.6 with 4 waves and three and
//    18.1 with two; 32 x 34816 x 5120, 4 waves and five tiles: 22.3 against 25.8
//    with three and 26.2 with two).  Up to four tiles per CU two tiles make two
//    full rounds (17 x 24600 x 17408 53.3 us; 59.1 with five).
//  * N <= 128 (97 .. 128 here) with M * K past the one-launch limit: the waves of
//    the fused launch at these sizes, quant_gemm_kernel, which has no 16-row form:
//    eight from K = kLongNarrowK on (7 x 128 x 5120 8 waves 7.9 us, 4 waves 8.6; x
//    17408 18.3 and 23.5; 16 waves of the 16-row form would take 6.4 and 12.9).
DecodeShape decode_shape(int64_t M, int64_t N, int64_t K, uint32_t n_cu) {
  const uint64_t tiles = (uint64_t)((N + 31) / 32);
  if (N <= 128 && M * K > 16 * (int64_t)kDecodeFuseMaxBlocks)
    return K >= kLongNarrowK ? DecodeShape::k8Shared : DecodeShape::k4Private;
  if (M <= 16) {
    if (tiles <= n_cu) return DecodeShape::kRows16w1;
    if (5 * tiles < 9 * (uint64_t)n_cu) return DecodeShape::kRows8w2;        // three: under 0.6 of the CUs
    if (tiles <= 3 * (uint64_t)n_cu) return DecodeShape::kRows8w3;
    const bool past_six = tiles > 6 * (uint64_t)n_cu;
    if (M * K > kRowsMaxElems) return past_six ? DecodeShape::k4SharedPair : DecodeShape::kRows4w2;
    if (past_six || tiles <= 4 * (uint64_t)n_cu) return DecodeShape::kRows8w2;
    return M * K <= 16 * (int64_t)kDecodeFuseMaxBlocks ? DecodeShape::kRows8w3 : DecodeShape::kRows4w2;
  }
  if (tiles <= n_cu) return K >= 8192 ? DecodeShape::k8Shared : DecodeShape::k4Private;
  if (5 * tiles < 9 * (uint64_t)n_cu) return DecodeShape::k8SharedPair;
  if (tiles <= 3 * (uint64_t)n_cu) return DecodeShape::k8Shared3;
  return tiles > 4 * (uint64_t)n_cu && tiles <= 5 * (uint64_t)n_cu ? DecodeShape::k4Shared5 : DecodeShape::k4SharedPair;
}

hipError_t launch_splitk_decode(const GemmOperands& o, GemmParams p, bool out_f32, hipStream_t stream) {
  const DecodeShape shape = decode_shape(p.M, p.N, p.K, cu_count());
  switch (shape) {
    case DecodeShape::k4Private: return launch_splitk<4, 1, 1, 3, false, false>(o, p, out_f32, stream);
    case DecodeShape::k8SharedPair: return launch_splitk<8, 1, 2, 3, true, false>(o, p, out_f32, stream);
    case DecodeShape::k8Shared3: return launch_splitk<8, 1, 3, 3, true, false>(o, p, out_f32, stream);
    case DecodeShape::k4Shared5: return launch_splitk<4, 1, 5, 2, true, false>(o, p, out_f32, stream);
    case DecodeShape::k8Shared: return launch_splitk<8, 1, 1, 4, true, false>(o, p, out_f32, stream);
    case DecodeShape::k4SharedPair: return launch_splitk<4, 1, 2, 3, true, false>(o, p, out_f32, stream);
    default: return launch_rows16(shape, o, p, out_f32, stream);
  }
}

// Small outputs with M > 32 (see plan_gemm): four or eight waves share the
// reduction of a tile.  64 x 96: two ring stages (100 x 34816 x 5120 49.9 us,
// 55.5 with three).
hipError_t launch_splitk_tile(const GemmOperands& o, const GemmParams& p, int kind, bool out_f32, hipStream_t stream) {
  switch (kind) {
    case GemmPlan::kSplitk32x32: return launch_splitk<4, 1, 1, 3, false, false>(o, p, out_f32, stream);
    case GemmPlan::kSplitk32x64: return launch_splitk<4, 1, 2, 3, true, false>(o, p, out_f32, stream);
    case GemmPlan::kSplitk64x64: return launch_splitk<4, 2, 2, 3, true, false>(o, p, out_f32, stream);
    case GemmPlan::kSplitk32x96: return launch_splitk<8, 1, 3, 3, true, false>(o, p, out_f32, stream);
    case GemmPlan::kSplitk32x160: return launch_splitk<4, 1, 5, 2, true, false>(o, p, out_f32, stream);
    default: return launch_splitk<4, 2, 3, 2, true, false>(o, p, out_f32, stream);
  }
}

// The fused decode launch, with the waves of decode_shape.  Above 16 rows (K
// below 1024) two weight tiles (eight waves: one) per workgroup, a ring one
// stage deeper than the plain kernel's: more of the weight in flight while the
// workgroup quantizes X.
template <int KS, int FN, int kStages>
static hipError_t launch_decode_quant(const GemmOperands& o, GemmParams p, const DecodeQuantArgs& q, bool dynamic,
                                      bool out_f32, hipStream_t stream) {
  constexpr int kRing = splitk_ring_bytes<KS, 1, FN, kStages, false>();
  static_assert(kRing >= KS * 64 * 64, "the reduction reuses the rings");
  p.tiles_m = 1;
  p.tiles_n = (p.N + FN * 32 - 1) / (FN * 32);
  const dim3 grid(p.tiles_n), block(KS * 64);
#define NVFP4_DQ(F32, Q)                                                                                   \
  hipLaunchKernelGGL((gemm_splitk_kernel<KS, 1, FN, kStages, F32, false, Q>), grid, block, kRing, stream, \
                     o.a_codes, o.a_scales, o.a_g, o.w_packed, o.w_g, o.y, p, q)
  if (dynamic) {
    if (out_f32) NVFP4_DQ(true, 2); else NVFP4_DQ(false, 2);
  } else {
    if (out_f32) NVFP4_DQ(true, 1); else NVFP4_DQ(false, 1);
  }
#undef NVFP4_DQ
  return hipGetLastError();
}

hipError_t launch_decode_quant_gemm(const GemmOperands& o, GemmParams p, const DecodeQuantArgs& q, bool dynamic,
                                    bool out_f32, hipStream_t stream) {
  if (p.M <= 16)
    return launch_rows16_quant(decode_shape(p.M, p.N, p.K, cu_count()), o, p, q, dynamic, out_f32, stream);
  switch (decode_shape(p.M, p.N, p.K, cu_count())) {         // K < 1024 here: no k8Shared
    case DecodeShape::k8SharedPair:
    case DecodeShape::k8Shared3: return launch_decode_quant<8, 1, 4>(o, p, q, dynamic, out_f32, stream);
    default: return launch_decode_quant<4, 2, 4>(o, p, q, dynamic, out_f32, stream);
  }
}

}  // namespace nvfp4
