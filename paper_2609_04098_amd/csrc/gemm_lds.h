// The prefill GEMM kernel (gemm_lds_kernel) and its launcher template; each
// launched configuration is instantiated in its own translation unit
// (gemm_lds_square.hip, gemm_lds_tall.hip; the super-stage kernel, whose
// schedule takes minutes to compile, one output type per unit:
// gemm_lds_super.hip, gemm_lds_super_f32.hip).
#pragma once

#include "gemm_common.h"

namespace nvfp4 {

// Workgroup shape of the LDS kernel: WM x WN waves, each owning an
// FM x FN block of 32 x 32 accumulator fragments; kOcc workgroups per CU.
template <int WM_, int WN_, int FM_, int FN_, int kOcc_, int kValu_, int kStages_, bool kSuper_ = false>
struct LdsCfg {
  static constexpr int WM = WM_, WN = WN_, FM = FM_, FN = FN_, kOcc = kOcc_;
  // kSuper (K % 256 == 0): the scales of 4 consecutive chunks move together,
  // one 16-byte DMA per fragment pair (a row's 4 scale dwords are
  // contiguous), into two alternating scale "super-stages" beside the ring.
  static constexpr bool kSuper = kSuper_;
  static constexpr int kWaves = WM * WN, kThreads = kWaves * 64;
  static constexpr int BM = WM * FM * 32, BN = WN * FN * 32;
  static constexpr int NFA = WM * FM, NFB = WN * FN;         // fragments per workgroup
  // Each wave moves the same number of A and B fragments (codes + scales);
  // with fewer fragments than waves, several waves move the same one (the
  // same bytes to the same place).
  static constexpr int kAPerWave = NFA >= kWaves ? NFA / kWaves : 1;
  static constexpr int kBPerWave = NFB >= kWaves ? NFB / kWaves : 1;
  // Scales: one dword of 4 block scales per fragment row and chunk.  With an
  // even count per wave, one DMA moves the scales of two fragments (64
  // distinct rows, 128 B per fragment slot); with an odd count, one DMA per
  // fragment (both half-waves load the same 32 rows; 256 B slots).
  static constexpr bool kPairA = kAPerWave % 2 == 0, kPairB = kBPerWave % 2 == 0;
  static constexpr int kSFA = kPairA ? 128 : 256, kSFB = kPairB ? 128 : 256;
  static constexpr int kSDmaA = kPairA ? kAPerWave / 2 : kAPerWave, kSDmaB = kPairB ? kBPerWave / 2 : kBPerWave;
  // One stage of the ring: raw codes (1 KB per fragment), then the scale
  // slots, of one 64-deep chunk.
  static constexpr int kA = 0, kB = NFA * 1024, kSA = kB + NFB * 1024, kSB = kSA + NFA * kSFA;
  static constexpr int kStageBytes = kSuper ? kSA : kSB + NFB * kSFB;
  // A super-stage: per A fragment [32 rows][4 chunks][4 B] (512 B), then per
  // W fragment [4 chunks][32 rows][4 B] (512 B, the packed order).
  static constexpr int kSuperB = NFA * 512, kSuperBytes = kSuperB + NFB * 512;
  // kStages 64-deep stages in the ring; iteration c refills the stage of
  // chunk c (consumed by every wave before the barrier that opens the
  // iteration) with chunk c + kStages.
  static constexpr int kStages = kStages_;
  static constexpr int kSuperBase = kStages * kStageBytes;
  static constexpr int kLdsBytes = kSuperBase + (kSuper ? 2 * kSuperBytes : 0);
  // BF16 epilogue staging, beyond the ring (so that no wave waits for the
  // others to leave the ring): per wave 32 output rows of its FN fragment
  // columns, rows padded by 16 bytes, then a scale per column.
  static constexpr int kEpiPitch = FN * 32 * 2 + 16;
  static constexpr int kEpiWave = 32 * kEpiPitch + FN * 32 * 4;
  static constexpr int kEpiBytes = kWaves * kEpiWave;
  static constexpr int kLdsTotal = kLdsBytes + kEpiBytes;     // bf16 output
  // DMA loads per chunk and wave (without the super-stage loads).
  static constexpr int kLoadsPerWave = kAPerWave + kBPerWave + (kSuper ? 0 : kSDmaA + kSDmaB);
  static constexpr int kSuperLoads = 2;          // per 4 chunks: one A pair, one W pair
  static_assert(!kSuper || (kAPerWave <= 2 && kBPerWave <= 2 && NFA % 2 == 0 && NFB % 2 == 0 && kStages == 4),
                "super-stage layout");
  static constexpr int kGroupM = 4;
  static constexpr int kMfma = 4 * FM * FN;                   // MFMAs per chunk and wave
  static constexpr int kValuPerMfma = kValu_;                 // schedule: VALU slots after each MFMA
  static constexpr int kLdsReads = 2 * (FM + FN);             // LDS reads per chunk and wave
  static constexpr int kWaitFirst = lds::vmcnt_imm((kStages - 1) * kLoadsPerWave);   // chunk 0 landed
  static constexpr int kWaitNext = lds::vmcnt_imm((kStages - 2) * kLoadsPerWave);    // chunk c + 1 landed
  // With super-stages: at chunk c the loads issued after everything chunk
  // c + 1 needs are those of chunks c - 2 and c - 1, plus the super-stage
  // loads issued with chunk c - 2 or c - 1 when that is a multiple of 4.
  static constexpr int kWaitSuper0 = lds::vmcnt_imm(2 * kLoadsPerWave);                // c % 4 in {0, 3}
  static constexpr int kWaitSuper1 = lds::vmcnt_imm(2 * kLoadsPerWave + kSuperLoads);  // c % 4 in {1, 2}
  static_assert(kStages >= 2 && (kStages - 1) * kLoadsPerWave < 64, "ring depth");
  static_assert((NFA % kWaves == 0 || kWaves % NFA == 0) && (NFB % kWaves == 0 || kWaves % NFB == 0), "load split");
  static_assert(kLdsReads <= kMfma / 2 && kLoadsPerWave <= kMfma, "schedule slots");
  static_assert(kOcc * kLdsTotal <= 160 * 1024, "LDS per CU");
};

// The launched shape: 256 x 256 workgroups of 2 x 2 waves, each wave a
// 128 x 128 block (4 x 4 fragments, 256 accumulator registers), one
// workgroup per CU.  Per chunk a wave decodes 8 fragments for 64 MFMAs
// (4 VALU per MFMA); with 4 x 2 fragments and two waves per SIMD it was
// 6 per MFMA and measured 4-10% slower on the prefill shapes, as did rings
// of 3 or 6 stages.  Its own VALU co-issues with its MFMAs.
typedef LdsCfg<2, 2, 4, 4, 1, 6, 4> LdsSquare;
// The same with scale super-stages (K % 256 == 0).
typedef LdsCfg<2, 2, 4, 4, 1, 5, 4, true> LdsSquareSuper;
// 256 x 128 workgroups of 2 x 2 waves with 4 x 2 fragments, two per CU: the
// tail of a launch whose last round of square tiles would be at most half
// full (see launch_gemm).
typedef LdsCfg<2, 2, 4, 2, 2, 5, 4> LdsTall;
// Small tiles, two workgroups per CU, for outputs with too few 256 x 256
// tiles (see plan_gemm): 128 x 128 workgroups of 2 x 2 waves, and 64 x 256
// workgroups of 1 x 4 waves for up to 64 rows and ragged row counts; both
// have 2 x 2 fragments per wave (8 decode VALU per MFMA, which with two
// waves per SIMD costs 21 ns per MFMA against 16.3 ns for the MFMA alone).
// 128 x 256 (2 x 4 fragments per wave, 6 VALU per MFMA) measured the same
// per MFMA and balances worse.
typedef LdsCfg<2, 2, 2, 2, 2, 9, 4> LdsMid;
typedef LdsCfg<2, 2, 2, 2, 2, 9, 4, true> LdsMidSuper;
typedef LdsCfg<1, 4, 2, 2, 2, 9, 4> LdsLow;
typedef LdsCfg<1, 4, 2, 2, 2, 9, 4, true> LdsLowSuper;
static_assert(LdsSquare::BM == kSquareTile && LdsSquare::BN == kSquareTile && LdsSquareSuper::BN == kSquareTile,
              "square tile of the dispatch");

// BF16 epilogue of the LDS kernel: y = RNE_bf16(acc / (G_A G_W[s])) for the
// segment s of each column.  Accumulator fragment (fa, fb) is transposed:
// lane (h, r) holds output row m0 + 32 fa + r and, in entries 4 q .. 4 q + 3,
// the adjacent columns n0 + 32 fb + 8 q + 4 h + (0..3).  A whole wave block
// (all rows < M, all columns < N, one segment) with rows starting on 16-byte
// boundaries moves through the wave's own LDS staging area 32 rows at a time:
// each lane writes 8 bytes (4 columns) of one row, then every global store
// writes 16 bytes of one row, 4 lanes covering the 32 columns of a fragment
// and 16 rows per instruction (a dword per column pair spread over 4 rows
// per instruction took 3 times as long per tile in isolation, and the
// epilogue 4.8 instead of 3.3 us per tile on mlp_gate_up).  Other blocks
// (partial, unaligned, or with a segment boundary inside the wave's columns)
// are staged too, with a scale per column and narrower or fewer stores.  The
// staged stores of whole blocks are non-temporal when
// the output is at least as large as the MALL (p.y_stream), each
// instruction then writing 4 whole rows of the wave block (256 bytes each):
// with ordinary stores, the dirty lines of mlp_gate_up's 570 MB output were
// written back during the next step's activation amax pass (dynamic
// act-quant 47.3 -> 36.4 us in the step, the GEMM and the step 0.5-0.9%
// shorter, same box).
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
constexpr int kCachePolicyNonTemporal = 2;   // the "nt" bit of a gfx950 buffer instruction

// Fast-path test and column scale of the BF16 epilogue, taken before the K
// loop so that the scale loads stay off the epilogue's path.
struct EpiPlan {
  bool whole;     // stage the wave block through LDS with one column scale
  float alpha;    // that scale
};

__device__ __forceinline__ int segment_of(const GemmParams& p, uint32_t col) {
  int s = 0;
#pragma unroll
  for (int i = 1; i < NVFP4_SEG_TABLE - 1; ++i) s += (i < p.n_seg && col >= p.seg_off[i]) ? 1 : 0;
  return s;
}

__device__ __forceinline__ float segment_scale(const float* __restrict__ a_g, const float* __restrict__ w_g, int s) {
  const float prod = *a_g * w_g[s];
  return prod == 0.0f ? 0.0f : 1.0f / prod;
}

template <int FM, int FN>
__device__ __forceinline__ EpiPlan epi_plan(const GemmParams& p, const float* __restrict__ a_g,
                                            const float* __restrict__ w_g, const void* y, uint32_t m0, uint32_t n0) {
  const uint32_t n_last = (n0 + FN * 32u < p.N ? n0 + FN * 32u : p.N) - 1u;
  const int s0 = segment_of(p, n0);
  EpiPlan e;
  e.whole = m0 + FM * 32u <= p.M && n0 + FN * 32u <= p.N && ((p.ldy * 2u) & 15u) == 0 &&
            (reinterpret_cast<uintptr_t>(y) & 15u) == 0 && s0 == segment_of(p, n_last);
  e.alpha = segment_scale(a_g, w_g, s0);
  return e;
}

template <int FM, int FN, int kPitch>
__device__ __forceinline__ void store_tile_t(const floatx16 (&acc)[FM][FN], const GemmParams& p, EpiPlan ep,
                                             const float* __restrict__ a_g, const float* __restrict__ w_g,
                                             void* __restrict__ y, uint32_t m0, uint32_t n0, uint8_t* stage) {
  constexpr uint32_t E = 2u;                      // bytes per output element
  // The lane again (not from a register that would be kept through the K loop).
  const uint32_t lane = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
  const uint32_t r = lane & 31u, h = lane >> 5;
  if (ep.whole) {
    const float alpha = ep.alpha;
    constexpr uint32_t kPieces = 2u * E;          // 16-byte pieces per fragment row
    constexpr uint32_t kRows = 64u / kPieces;     // rows per store instruction
    const uint32_t rr = lane / kPieces, pc = lane % kPieces;
    constexpr uint32_t kLanesWide = FN * kPieces, kRowsWide = 64u / kLanesWide;   // whole wave-block rows
    const uint32_t rw = lane / kLanesWide, pw = lane % kLanesWide;
    // Non-temporal stores go through a buffer descriptor: a plain store in
    // the other branch would be merged with a non-temporal one (dropping
    // the hint).
    const __amdgpu_buffer_rsrc_t ry = rsrc(y, p.M * p.ldy * E);
#pragma unroll
    for (int fa = 0; fa < FM; ++fa) {
#pragma unroll
      for (int fb = 0; fb < FN; ++fb)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const floatx16& v = acc[fa][fb];
          const uint32_t lo = pack_bf16_rne(v[4 * q] * alpha, v[4 * q + 1] * alpha);
          const uint32_t hi = pack_bf16_rne(v[4 * q + 2] * alpha, v[4 * q + 3] * alpha);
          *reinterpret_cast<u32x2*>(stage + r * kPitch + (fb * 32u + q * 8u + h * 4u) * E) = u32x2{lo, hi};
        }
      // Lanes read what other lanes wrote, and the next fragment row
      // overwrites what they read: keep the LDS accesses in program order.
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      // Byte offsets in y stay below 2^32 (the API bounds M * ldy by 2^31).
      if (p.y_stream) {
        // Non-temporal: whole 128-byte lines per instruction (a row of the
        // wave block per FN * 4 lanes); 64-byte pieces wrote 1.38 times the
        // output bytes to HBM this way.
#pragma unroll
        for (uint32_t k = 0; k < 32u / kRowsWide; ++k) {
          const uint32_t row = k * kRowsWide + rw;
          const int4v v = *reinterpret_cast<const int4v*>(stage + row * kPitch + pw * 16u);
          const uint32_t off = ((m0 + fa * 32u + row) * p.ldy + n0) * E + pw * 16u;
          __builtin_amdgcn_raw_buffer_store_b128(v, ry, off, 0, kCachePolicyNonTemporal);
        }
      } else {
#pragma unroll
        for (uint32_t k = 0; k < 32u / kRows; ++k)
#pragma unroll
          for (int fb = 0; fb < FN; ++fb) {
            const uint32_t row = k * kRows + rr;
            const int4v v = *reinterpret_cast<const int4v*>(stage + row * kPitch + fb * 32u * E + pc * 16u);
            const uint32_t off = ((m0 + fa * 32u + row) * p.ldy + n0 + fb * 32u) * E + pc * 16u;
            *reinterpret_cast<int4v*>(static_cast<uint8_t*>(y) + off) = v;
          }
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    }
    return;
  }
  // Blocks past M or N, of several segments, or in outputs whose rows allow no
  // 16-byte stores: staged the same way, with a scale per column, and stored in
  // pieces of 16, 8 or 4 bytes as the rows allow (a wave's store takes 16 cycles
  // whatever its width: 5 us more per 256 x 256 tile with 8 bytes, 11 with 4).
  // Element by element from the accumulators (64 lanes on 32 rows, a store per
  // element) such a block took 20 to 30 us, most of a short-K call: 8000 x 1300 x
  // 128 48.2 us on 256 x 256 tiles and 46.7 on 128 x 128, with this 16.6.
  if (m0 >= p.M || n0 >= p.N) return;
  float* scale = reinterpret_cast<float*>(stage + 32 * kPitch);
  const uint32_t cols = p.N - n0 < FN * 32u ? p.N - n0 : FN * 32u;
#pragma unroll
  for (uint32_t c = 0; c < FN * 32u; c += 64)
    scale[c + lane] = c + lane < cols ? segment_scale(a_g, w_g, segment_of(p, n0 + c + lane)) : 0.0f;
  const uint32_t align = (p.ldy * E | (uint32_t)reinterpret_cast<uintptr_t>(y)) & 15u;   // of the rows, 0: 16 bytes
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
  for (int fa = 0; fa < FM; ++fa) {
    const uint32_t row0 = m0 + fa * 32u;
    if (row0 >= p.M) return;
    const uint32_t rows = p.M - row0 < 32u ? p.M - row0 : 32u;
    // One fragment row at a time is copied out of the accumulators: all of them
    // ahead of the branch need more registers than there are.
    floatx16 part[FN];
#pragma unroll
    for (int fb = 0; fb < FN; ++fb) {
      part[fb] = acc[fa][fb];
      asm volatile("" : "+v"(part[fb]));
    }
#pragma unroll
    for (int fb = 0; fb < FN; ++fb)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const floatx16& v = part[fb];
        const uint32_t c = fb * 32u + q * 8u + h * 4u;
        const float4 a = *reinterpret_cast<const float4*>(scale + c);
        const uint32_t lo = pack_bf16_rne(v[4 * q] * a.x, v[4 * q + 1] * a.y);
        const uint32_t hi = pack_bf16_rne(v[4 * q + 2] * a.z, v[4 * q + 3] * a.w);
        *reinterpret_cast<u32x2*>(stage + r * kPitch + c * E) = u32x2{lo, hi};
      }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    uint16_t* y0 = static_cast<uint16_t*>(y) + (size_t)row0 * p.ldy + n0;
    // Pieces of `bytes`; what reaches past N, and pieces that rows don't align,
    // element by element.
    auto store = [&](auto bytes_tag, bool aligned) {
      constexpr uint32_t kBytes = decltype(bytes_tag)::value, kElems = kBytes / E;
      typedef uint32_t piece __attribute__((ext_vector_type(kBytes / 4)));
      constexpr uint32_t kLanes = FN * 32u / kElems, kRows = 64u / kLanes;
      const uint32_t c = lane % kLanes * kElems;
#pragma unroll 4
      for (uint32_t row = lane / kLanes; row < rows; row += kRows) {
        const uint8_t* src = stage + row * kPitch + c * E;
        uint16_t* dst = y0 + (size_t)row * p.ldy + c;
        if (aligned && c + kElems <= cols) {
          *reinterpret_cast<piece*>(dst) = *reinterpret_cast<const piece*>(src);
        } else if constexpr (kElems == 2) {
          const uint32_t v = *reinterpret_cast<const uint32_t*>(src);
          if (c < cols) dst[0] = (uint16_t)v;
          if (c + 1u < cols) dst[1] = (uint16_t)(v >> 16);
        } else {
          for (uint32_t i = 0; i < kElems && c + i < cols; ++i) dst[i] = reinterpret_cast<const uint16_t*>(src)[i];
        }
      }
    };
    if (align == 0)
      store(std::integral_constant<uint32_t, 16>{}, true);
    else if ((align & 7u) == 0)
      store(std::integral_constant<uint32_t, 8>{}, true);
    else
      store(std::integral_constant<uint32_t, 4>{}, (align & 3u) == 0);
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  }
}

template <class C, bool kF32Out>
__global__ __launch_bounds__(C::kThreads, C::kOcc) void gemm_lds_kernel(const uint8_t* __restrict__ a_codes,
                                                                   const uint8_t* __restrict__ a_scales,
                                                                   const float* __restrict__ a_g,
                                                                   const uint8_t* __restrict__ w_packed,
                                                                   const float* __restrict__ w_g,
                                                                   void* __restrict__ y, GemmParams p) {
  constexpr int WN = C::WN, FM = C::FM, FN = C::FN, BM = C::BM, BN = C::BN;
  constexpr int kA = C::kA, kB = C::kB, kSA = C::kSA, kSB = C::kSB, kStages = C::kStages;
  constexpr int kStageBytes = C::kStageBytes, kAPerWave = C::kAPerWave, kBPerWave = C::kBPerWave;
  extern __shared__ __attribute__((aligned(16))) uint8_t smem[];
  const uint32_t lane = threadIdx.x & 63, wave = wave_index();
  const uint32_t r = lane & 31, h = lane >> 5;
  // K split (FP32 partial sums): part j of a tile takes the j-th of k_parts
  // nearly equal runs of whole groups of kUnit chunks; the descriptors' bases
  // move to its first chunk, the row strides stay those of the whole K.
  // Consecutive workgroups of an XCD take different tiles of one part (they
  // read the same K range of A and W, and so share them in the XCD's L2).
  constexpr uint32_t kUnit = C::kSuper ? 4 : 1;
  uint32_t part = 0, kc0 = 0, chunks = p.chunks, tm, tn;
  uint32_t tile_out = 0;                     // partial tile (tile runs with K parts)
  if (kF32Out && p.k_parts > 1) {
    const uint32_t tiles = p.tile_count ? p.tile_count : p.tiles_m * p.tiles_n, units = p.chunks / kUnit;
    const uint32_t pid = xcd_contiguous(tiles * p.k_parts);
    // (The divisions run in vector registers.  Descriptors made from their
    // results as they are cost every load of the K loop a loop over the lanes,
    // in the launches without K parts too: FP32 outputs took 4 to 8% more,
    // 5000 x 5120 x 1088 72.8 -> 77.0 us.)
    part = __builtin_amdgcn_readfirstlane(pid / tiles);
    kc0 = __builtin_amdgcn_readfirstlane(part * units / p.k_parts * kUnit);
    chunks = __builtin_amdgcn_readfirstlane((part + 1) * units / p.k_parts * kUnit) - kc0;
    tile_at<C::kGroupM>(p, p.tile_begin + pid - part * tiles, tm, tn);
    tile_out = pid;
  } else {
    tile_at<C::kGroupM>(p, p.tile_begin + xcd_contiguous(p.tile_count ? p.tile_count : p.tiles_m * p.tiles_n), tm, tn);
  }
  const uint32_t wm = wave / WN, wn = wave % WN;

  // Per-lane offsets are fixed; the chunk advances the descriptors' base
  // (and shrinks their size) in scalar registers.  Rows >= M and tiles past
  // the packed weight get offsets beyond every descriptor: zeros.
  // Scale DMA j: lane (h, r) loads the scale dword of row r of fragment
  // j * 2 + h of the wave's pair (paired), or of fragment j (single).
  uint32_t a_off[kAPerWave], as_off[C::kSDmaA], b_off[kBPerWave], bs_off[C::kSDmaB];
  const uint32_t fa0 = kAPerWave * wave % C::NFA, fb0 = kBPerWave * wave % C::NFB;   // first fragment this wave loads
  const uint32_t nt0 = (p.n_off >> 5) + tn * (BN / 32);             // first weight tile of the tile
#pragma unroll
  for (int i = 0; i < kAPerWave; ++i) {
    const uint32_t row = tm * BM + (fa0 + i) * 32 + r;
    a_off[i] = row < p.M ? row * (p.K >> 1) + h * 16u : kOOB;
  }
#pragma unroll
  for (int j = 0; j < C::kSDmaA; ++j) {
    const uint32_t row = tm * BM + (fa0 + (C::kPairA ? 2 * j + h : j)) * 32 + r;
    as_off[j] = row < p.M ? row * (p.K >> 4) : kOOB;
  }
#pragma unroll
  for (int i = 0; i < kBPerWave; ++i) {
    const uint32_t nt = nt0 + fb0 + i;
    b_off[i] = nt < p.w_tiles ? nt * p.w_kc * 1024u + lane * 16u : kOOB;
  }
#pragma unroll
  for (int j = 0; j < C::kSDmaB; ++j) {
    const uint32_t nt = nt0 + fb0 + (C::kPairB ? 2 * j + h : j);
    bs_off[j] = nt < p.w_tiles ? nt * p.w_kc * 128u + r * 4u : kOOB;
  }
  const uint8_t* w_scales = w_packed + p.w_scale_offset;
  const uint32_t w_scale_bytes = p.w_bytes - p.w_scale_offset;

  const __amdgpu_buffer_rsrc_t ra = rsrc(a_codes + kc0 * 32u, p.a_code_bytes - kc0 * 32u);
  const __amdgpu_buffer_rsrc_t rs = rsrc(a_scales + kc0 * 4u, p.a_scale_bytes - kc0 * 4u);
  const __amdgpu_buffer_rsrc_t rb = rsrc(w_packed + kc0 * 1024u, p.w_scale_offset - kc0 * 1024u);
  const __amdgpu_buffer_rsrc_t rbs = rsrc(w_scales + kc0 * 128u, w_scale_bytes - kc0 * 128u);
  // DMA of chunk kc into stage kc % kStages.  The ring runs kStages - 1
  // chunks past the end of K; those stages are never read, and re-load the
  // last chunk so that every address stays inside its tensor.
  auto issue = [&](uint32_t kc) {
    uint8_t* st = smem + (kc % kStages) * kStageBytes;
    const uint32_t kq = kc < chunks ? kc : chunks - 1;
#pragma unroll
    for (int i = 0; i < kAPerWave; ++i) dma16(ra, st + kA + (fa0 + i) * 1024, a_off[i], kq * 32u);
    if constexpr (!C::kSuper) {
#pragma unroll
      for (int j = 0; j < C::kSDmaA; ++j)
        dma4(rs, st + kSA + (fa0 + (C::kPairA ? 2 * j : j)) * C::kSFA, as_off[j], kq * 4u);
    }
#pragma unroll
    for (int i = 0; i < kBPerWave; ++i) dma16(rb, st + kB + (fb0 + i) * 1024, b_off[i], kq * 1024u);
    if constexpr (!C::kSuper) {
#pragma unroll
      for (int j = 0; j < C::kSDmaB; ++j)
        dma4(rbs, st + kSB + (fb0 + (C::kPairB ? 2 * j : j)) * C::kSFB, bs_off[j], kq * 128u);
    }
  };
  // Super-stage sg (the scales of chunks 4 sg .. 4 sg + 3) into buffer
  // sg % 2: lane (h, r) loads row r of A fragment fap + h of the wave's pair
  // (16 bytes: 4 chunks of one row) and 16 bytes (rows 4 (r % 8) .., chunk
  // r / 8) of the 512-byte group of weight tile fbp + h.  Groups past the end
  // of K re-load the last one.
  const uint32_t fap = fa0 & ~1u, fbp = fb0 & ~1u;
  const uint32_t a_sup_off = [&]() {
    const uint32_t row = tm * BM + (fap + h) * 32 + r;
    return row < p.M ? row * (p.K >> 4) : kOOB;
  }();
  const uint32_t b_sup_off = [&]() {
    const uint32_t nt = nt0 + fbp + h;
    return nt < p.w_tiles ? nt * p.w_kc * 128u + r * 16u : kOOB;
  }();
  auto issue_super = [&](uint32_t sg) {
    uint8_t* sb = smem + C::kSuperBase + (sg & 1u) * C::kSuperBytes;
    const uint32_t last = (chunks >> 2) - 1;
    const uint32_t sq = sg < last ? sg : last;
    dma16(rs, sb + fap * 512, a_sup_off, sq * 16u);
    dma16(rbs, sb + C::kSuperB + fbp * 512, b_sup_off, sq * 512u);
  };

  struct Regs {
    int4v ca[FM], cb[FN];
    uint32_t sa[FM], sb[FN];   // low 16 bits: the lane's two block scales
  };
  // Lane (h, r) takes the half h of row r's scale dword (blocks 2h, 2h + 1
  // of the chunk).
  auto read_stage = [&](Regs& R, uint32_t kc) {
    const uint8_t* st = smem + (kc % kStages) * kStageBytes;
    const uint8_t* sb = smem + C::kSuperBase + ((kc >> 2) & 1u) * C::kSuperBytes;
    const uint32_t j = kc & 3u;
#pragma unroll
    for (int f = 0; f < FM; ++f) {
      R.ca[f] = *(const int4v*)(st + kA + (wm * FM + f) * 1024 + lane * 16);
      if constexpr (C::kSuper)
        R.sa[f] = *(const uint16_t*)(sb + (wm * FM + f) * 512 + r * 16 + j * 4 + h * 2);
      else
        R.sa[f] = *(const uint16_t*)(st + kSA + (wm * FM + f) * C::kSFA + r * 4 + h * 2);
    }
#pragma unroll
    for (int f = 0; f < FN; ++f) {
      R.cb[f] = *(const int4v*)(st + kB + (wn * FN + f) * 1024 + lane * 16);
      if constexpr (C::kSuper)
        R.sb[f] = *(const uint16_t*)(sb + C::kSuperB + (wn * FN + f) * 512 + j * 128 + r * 4 + h * 2);
      else
        R.sb[f] = *(const uint16_t*)(st + kSB + (wn * FN + f) * C::kSFB + r * 4 + h * 2);
    }
  };

  // BF16 output: acc[fa][fb] holds the transposed output block of fragments
  // (fa, fb) (the MFMAs take the weight fragment as their first operand),
  // for the staged epilogue.  FP32 output keeps the direct orientation and
  // per-element stores, whose 32 lanes write 128 contiguous bytes of a row
  // (the staged form measured 3% slower there, and its instantiation's
  // main loop compiled worse).
  constexpr bool kTransposed = !kF32Out;
  const uint32_t m0_wave = tm * BM + wm * FM * 32, n0_wave = p.n_off + tn * BN + wn * FN * 32;
  EpiPlan ep{};
  if constexpr (kTransposed) ep = epi_plan<FM, FN>(p, a_g, w_g, y, m0_wave, n0_wave);
  floatx16 acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = floatx16{};

  // The decode of MFMA step 0 of chunk c + 1 runs beside the MFMAs of step 3
  // of chunk c, so no iteration starts with a run of VALU work in front of
  // its first MFMA (one wave per SIMD: nothing else would cover it).
  half2v sA[FM], sB[FN];
  half8 av[2][FM], bv[2][FN];
  auto scales = [&](const Regs& R) {
#pragma unroll
    for (int f = 0; f < FM; ++f) sA[f] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(R.sa[f], 1.0f, false);
#pragma unroll
    for (int f = 0; f < FN; ++f) sB[f] = __builtin_amdgcn_cvt_scalef32_pk_f16_fp8(R.sb[f], 1.0f, false);
  };
  // Decode MFMA step j (0..3) of R into buffer u; steps 0, 1 use the first
  // block scale of the lane, steps 2, 3 the second.
  auto decode_step = [&](const Regs& R, int j, int u) {
#pragma unroll
    for (int f = 0; f < FM; ++f)
      av[u][f] = decode8((uint32_t)R.ca[f][j], j >> 1 ? __builtin_shufflevector(sA[f], sA[f], 1, 1)
                                                      : __builtin_shufflevector(sA[f], sA[f], 0, 0));
#pragma unroll
    for (int f = 0; f < FN; ++f)
      bv[u][f] = decode8((uint32_t)R.cb[f][j], j >> 1 ? __builtin_shufflevector(sB[f], sB[f], 1, 1)
                                                      : __builtin_shufflevector(sB[f], sB[f], 0, 0));
  };
  // One chunk: wait until chunk c + 1 has landed, barrier, DMA of chunk
  // c + kStages into the stage of chunk c (and, with super-stages, at
  // c % 4 == 0 the scales of chunks c + 4 .. c + 7 into the buffer that held
  // those of chunks c - 4 .. c - 1), LDS reads of chunk c + 1 into `next`,
  // decode + MFMA of `cur`.  pos_tag: c % 4 (super-stages) or 0.
  auto step = [&](uint32_t c, const Regs& cur, Regs& next, auto pos_tag) {
    constexpr int kPos = decltype(pos_tag)::value;
    constexpr bool kIssueSuper = C::kSuper && kPos == 0;
    // Wait for chunk c + 1's DMA and for this wave's LDS reads (those of
    // stage c were issued in the previous iteration), so that after the
    // barrier the stage of chunk c may be refilled.  The MFMAs and decode of
    // the previous chunk may still sink past the barrier; they read only
    // registers.
    if constexpr (C::kSuper)
      __builtin_amdgcn_s_waitcnt((kPos == 1 || kPos == 2 ? C::kWaitSuper1 : C::kWaitSuper0) & lds::kLgkm0Mask);
    else
      __builtin_amdgcn_s_waitcnt(C::kWaitNext & lds::kLgkm0Mask);
    __builtin_amdgcn_s_barrier();
    issue(c + kStages);
    if constexpr (kIssueSuper) issue_super((c >> 2) + 1);
    read_stage(next, c + 1);
    // Square tiles: all LDS reads of chunk c + 1 go out before this chunk's
    // MFMAs.  Left to the scheduler, half of them sank to just ahead of
    // their decode at the end of the chunk, each then waited on within one
    // MFMA (mlp_gate_up 2.17 -> 2.13 ms with the fence).
    if constexpr (C::kMfma >= 64) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int u = j & 1;
      if (j < 3) {
        decode_step(cur, j + 1, u ^ 1);
      } else {
        scales(next);
        decode_step(next, 0, 0);
      }
#pragma unroll
      for (int fa = 0; fa < FM; ++fa)
#pragma unroll
        for (int fb = 0; fb < FN; ++fb)
          acc[fa][fb] = kTransposed
                            ? __builtin_amdgcn_mfma_f32_32x32x16_f16(bv[u][fb], av[u][fa], acc[fa][fb], 0, 0, 0)
                            : __builtin_amdgcn_mfma_f32_32x32x16_f16(av[u][fa], bv[u][fb], acc[fa][fb], 0, 0, 0);
    }
    // LDS reads spread over the first half of the chunk, DMA issues over the
    // first three quarters.
    constexpr int kDma = C::kLoadsPerWave + (kIssueSuper ? C::kSuperLoads : 0);
    constexpr int kLdsEvery = (C::kMfma / 2) / C::kLdsReads;
    constexpr int kDmaEvery = (3 * C::kMfma / 4) / kDma;
#pragma unroll
    for (int i = 0; i < C::kMfma; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                       // MFMA
      __builtin_amdgcn_sched_group_barrier(0x002, C::kValuPerMfma, 0);         // VALU
      if (i % kLdsEvery == kLdsEvery - 1 && i / kLdsEvery < C::kLdsReads)
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);                     // LDS read
      if (i % kDmaEvery == 0 && i / kDmaEvery < kDma)
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);                     // VMEM (DMA)
    }
  };
  using Pos0 = std::integral_constant<int, 0>;
  using Pos1 = std::integral_constant<int, 1>;
  using Pos2 = std::integral_constant<int, 2>;
  using Pos3 = std::integral_constant<int, 3>;

  if constexpr (C::kSuper) {
    issue_super(0);                          // before chunk 0's codes: landed with them
    __builtin_amdgcn_sched_barrier(0);       // keep that order (the waits count loads in issue order)
  }
#pragma unroll
  for (int s = 0; s < kStages; ++s) issue(s);
  __builtin_amdgcn_s_waitcnt(C::kWaitFirst);
  __builtin_amdgcn_s_barrier();
  Regs cur, nxt;
  read_stage(cur, 0);
  scales(cur);
  decode_step(cur, 0, 0);
  if constexpr (C::kSuper) {
    // chunks % 4 == 0 (K % 256 == 0, parts of whole groups).
    for (uint32_t c = 0; c < chunks; c += 4) {
      step(c, cur, nxt, Pos0{});
      step(c + 1, nxt, cur, Pos1{});
      step(c + 2, cur, nxt, Pos2{});
      step(c + 3, nxt, cur, Pos3{});
    }
  } else {
    for (uint32_t c = 0; c < chunks; ++c) {
      step(c, cur, nxt, Pos0{});
      cur = nxt;
    }
  }
  // Drain the DMA of the chunks past the end before the workgroup exits.
  __builtin_amdgcn_s_waitcnt(0x0F70);
  void* yo = y;
  if constexpr (kF32Out) {
    // A partial tile's element (row, col) sits at row * ldy + col of the whole
    // output's rows (ldy = kSquareTile for a tile of its own).
    ptrdiff_t off = (ptrdiff_t)part * p.part_stride;
    if (p.k_parts > 1 && p.tile_count)
      off = (ptrdiff_t)tile_out * (BM * BN) - ((ptrdiff_t)tm * BM * p.ldy + (ptrdiff_t)tn * BN);
    yo = reinterpret_cast<void*>(reinterpret_cast<intptr_t>(y) + off * (ptrdiff_t)sizeof(float));
  }
  if constexpr (kTransposed) {
    constexpr int kPitch = C::kEpiPitch;
    store_tile_t<FM, FN, kPitch>(acc, p, ep, a_g, w_g, yo, m0_wave, n0_wave,
                                 smem + C::kLdsBytes + wave * C::kEpiWave);
  } else {
    store_tile<FM, FN, kF32Out>(acc, p, a_g, w_g, yo, m0_wave, n0_wave, r, h);
  }
}

// Output columns [n_begin, n_end) (n_begin a multiple of 32).
template <class C, bool kF32Out>
static hipError_t launch_lds_as(const GemmOperands& o, GemmParams p, uint32_t n_begin, uint32_t n_end,
                                hipStream_t stream) {
  p.n_off = n_begin;
  p.tiles_m = (p.M + C::BM - 1) / C::BM;
  p.tiles_n = (n_end - n_begin + C::BN - 1) / C::BN;
  const dim3 grid((p.tile_count ? p.tile_count : p.tiles_m * p.tiles_n) * p.k_parts), block(C::kThreads);
  const uint32_t lds = kF32Out ? C::kLdsBytes : C::kLdsTotal;
  hipLaunchKernelGGL((gemm_lds_kernel<C, kF32Out>), grid, block, lds, stream, o.a_codes, o.a_scales, o.a_g,
                     o.w_packed, o.w_g, o.y, p);
  return hipGetLastError();
}

// Output columns [n_begin, n_end) as k_parts runs of K per tile (whole groups
// of 4 chunks with super-stages): unscaled FP32 partial sums into
// parts[k_parts][M][parts_row(n_end - n_begin)], for sum_parts_kernel.
template <class C>
static hipError_t launch_lds_parts(const GemmOperands& o, GemmParams p, uint32_t n_begin, uint32_t n_end,
                                   uint32_t k_parts, float* parts, hipStream_t stream) {
  const uint32_t ldp = parts_row(n_end - n_begin);
  p.k_parts = k_parts;
  p.part_stride = p.M * ldp;
  p.ldy = ldp;
  GemmOperands q = o;
  // The kernel stores column c at y[row * ldy + c]: shift the base so that
  // column n_begin lands at parts[row * ldp].
  q.y = reinterpret_cast<void*>(reinterpret_cast<uintptr_t>(parts) - (uintptr_t)n_begin * sizeof(float));
  return launch_lds_as<C, true>(q, p, n_begin, n_end, stream);
}

template <class C>
static hipError_t launch_lds(const GemmOperands& o, GemmParams p, uint32_t n_begin, uint32_t n_end, bool out_f32,
                             hipStream_t stream) {
  return out_f32 ? launch_lds_as<C, true>(o, p, n_begin, n_end, stream)
                 : launch_lds_as<C, false>(o, p, n_begin, n_end, stream);
}

}  // namespace nvfp4
