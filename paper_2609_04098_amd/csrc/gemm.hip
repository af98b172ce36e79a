// Host dispatch of the NVFP4 GEMM (nvfp4_gemm, nvfp4_gemm_gdn_gates): picks
// the kernel family for a shape.  The kernels and the numerics are described
// in gemm_common.h.
#include <mutex>

#include "gemm_common.h"

namespace nvfp4 {

namespace {
constexpr int kMaxDevices = 64;
std::once_flag g_cu_once[kMaxDevices];
int g_cu_count[kMaxDevices];
}  // namespace

uint32_t cu_count() {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return 0;
  std::call_once(g_cu_once[dev], [dev]() {
    int n = 0;
    g_cu_count[dev] = hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess ? n : 0;
  });
  return (uint32_t)g_cu_count[dev];
}

// Estimated time of one tile shape on n_cu compute units, in us, for the
// choice between tile shapes and numbers of K parts.  A workgroup alone on a
// CU and two that share it take the same time per chunk and workgroup
// (measured: 240 workgroups of 91 chunks and 480 of 45 both 50 us), so the
// work is counted in rounds of one workgroup per CU whatever the occupancy.
// The clock is held by power, so a round that leaves CUs idle runs faster: a
// partly filled last round of square tiles takes 0.74 to 0.8 of a full one (320
// and 384 tiles at K = 5120, 400 at K = 17408: 240, 242 and 699 us against 138
// and 389 for one round), a lone round of up to 0.85 of the CUs 0.9 (128 to 204
// tiles); at K = 2048, where M and N reach no further than whole tiles, of up to
// 0.6 of them 0.72 (64 to 160 tiles 41 to 45 us, 192 48, 256 57).  Smaller tiles,
// several to a CU, gain less (`last`, `lone`), and split-K tiles, whose waves wait
// more, need a second workgroup on the CU to reach their rate (lone 1.1).
static float rounds_of(uint64_t workgroups, uint32_t n_cu, float last, float lone) {
  const float frac = (float)(workgroups % n_cu) / (float)n_cu, knee = lone < 0.8f ? 0.6f : 0.85f;
  if (workgroups < n_cu) return lone >= 1.0f || frac <= knee ? lone : lone + (1.0f - lone) * (frac - knee) / (1.0f - knee);
  return (float)(workgroups / n_cu) + (frac == 0.0f ? 0.0f : frac > last ? frac : last);
}

struct TileCost {
  int kind, super_kind;
  uint32_t bm, bn;
  float chunk_us, chunk_us_super;   // one 64-deep chunk of a tile
  float fixed_us;                   // first loads, epilogue, launch
  float round_us;                   // first loads and epilogue of a further round, at short K
  float last, lone;                 // see rounds_of
  uint32_t max_parts;               // K parts the launcher offers (with super-stages; square: only with them)
};
// Fitted to M = 50 .. 1000 against N = 4352 .. 34816 at K = 5120 and to N = 5120
// at K = 2176 .. 17408, the square tile also to larger M, and checked at M = 64 ..
// 3000, N = 256 .. 8192, K = 64 .. 5120 (below N of about 1000 and K of 2000 the
// estimates order the tiles, their times are off by up to a third).  The
// split-K tiles (four or eight waves share a tile's reduction and meet in LDS) have
// the cheaper small tile, the LDS tiles the cheaper large one and K parts.
// round_us: below kShortK the chunks of a split-K tile don't cover the first
// loads and the epilogue of the next round's tile (1024 x 5120 with 64 x 64 tiles,
// five rounds: 14.9 us at K = 64 and at K = 256; 128 x 128 tiles 7.2 and 9.5).
constexpr TileCost kTileCosts[] = {
    {GemmPlan::kLdsSquare, GemmPlan::kLdsSuper, 256, 256, 1.65f, 1.55f, 7.5f, 0.0f, 0.75f, 0.9f, 32},
    {GemmPlan::kLdsMid, GemmPlan::kLdsMidSuper, 128, 128, 0.53f, 0.465f, 6.5f, 0.0f, 0.92f, 0.95f, 32},
    {GemmPlan::kLdsLow, GemmPlan::kLdsLowSuper, 64, 256, 0.57f, 0.515f, 7.0f, 0.0f, 0.92f, 0.95f, 32},
    {GemmPlan::kSplitk64x96, GemmPlan::kSplitk64x96, 64, 96, 0.175f, 0.175f, 6.5f, 1.8f, 1.0f, 1.1f, 1},
    {GemmPlan::kSplitk64x64, GemmPlan::kSplitk64x64, 64, 64, 0.15f, 0.15f, 5.5f, 1.5f, 1.0f, 1.1f, 1},
    {GemmPlan::kSplitk32x160, GemmPlan::kSplitk32x160, 32, 160, 0.185f, 0.185f, 6.0f, 1.5f, 1.0f, 1.1f, 1},
    {GemmPlan::kSplitk32x96, GemmPlan::kSplitk32x96, 32, 96, 0.12f, 0.12f, 0.0f, 0.0f, 1.0f, 1.0f, 1},
    {GemmPlan::kSplitk32x64, GemmPlan::kSplitk32x64, 32, 64, 0.08f, 0.08f, 5.5f, 0.5f, 1.0f, 1.1f, 1},
    {GemmPlan::kSplitk32x32, GemmPlan::kSplitk32x32, 32, 32, 0.06f, 0.06f, 4.0f, 0.0f, 1.0f, 1.1f, 1},
};
constexpr int64_t kShortK = 2048;
// The square tile at K <= kShortK.
constexpr TileCost kSquareShort = {GemmPlan::kLdsSquare, GemmPlan::kLdsSuper, 256, 256, 1.65f, 1.55f, 9.0f, 0.0f, 0.75f, 0.72f, 32};

// Where the costs of short K hold.  Rows that are no multiple of 16 bytes are
// stored in narrower pieces, which costs the tiled kernels' staged stores 2 us a
// tile and more but not the split-K tiles': with N % 8 != 0 their rounds go without
// the extra cost (bf16, 1024 x 2601 x 1024 12.0 us on split-K tiles, 17.6 on 128 x
// 128; 777 x 1998 x 128 6.9 and 9.2).
static bool short_k(int64_t N, int64_t K) { return K <= kShortK && N % 8 == 0; }
static const TileCost& square_cost(int64_t N, int64_t K) { return short_k(N, K) ? kSquareShort : kTileCosts[0]; }
// The summing pass: a launch, and every partial sum written and read once
// (they stay in the last-level cache).
constexpr float kSumLaunchUs = 2.5f, kPartBytesPerUs = 6.0e6f;
// Bound on the partial sums of one call.
constexpr uint64_t kMaxPartBytes = 128ull << 20;
constexpr uint32_t kMinPartChunks = 4;   // one group of chunks with super-stages

// The split-K tiles are offered where their costs were fitted: a batch of up
// to 1024 rows, or a K below 2048, where the longer first loads of the LDS tiles
// weigh more (1300 x 1300 x 1088: 24 us with 128 x 128 tiles; 1000 rows 10 us
// with split-K tiles); at most 6 rounds of tiles (100 x 34816 x 5120 with 32 x 64
// tiles, 9 rounds, took 75 us for an estimate of 70; the LDS tiles, which share
// each operand between their waves, are the better ones there), 5 below K =
// 1024, where the estimates are mostly fixed cost.
constexpr int64_t kSplitkMaxRows = 1024;
constexpr uint64_t kSplitkMaxRounds = 6, kSplitkMaxRoundsShort = 5;

// Below this K the K-halves / tall-tile form of the last round is kept as
// it is: the cost of a tile is then mostly its first loads and epilogue.
constexpr int64_t kTailMinK = 2048;

// K parts of the last round's tiles: at most kMaxTailParts.
constexpr uint32_t kMaxTailParts = 8;
// Another plan replaces whole square tiles only for an estimated gain beyond
// the estimate's own error.
constexpr float kPlanGain = 0.96f;

// The cheapest single launch over all columns: tile shape and K parts.
static GemmPlan plan_tiles(int64_t M, int64_t N, int64_t K, uint32_t n_cu, bool with_ws, float* cost) {
  const bool super = K % 256 == 0;
  const uint32_t unit = super ? 4 : 1, units = (uint32_t)(K / 64) / unit;
  // Among the split-K tiles the plain costs decide, which fit their order; their
  // extra cost per round (TileCost::round_us) counts against the tiled kernels.
  GemmPlan best{}, best_splitk{};
  float splitk_cost = 0.0f, splitk_round_cost = 0.0f;
  *cost = 0.0f;
  for (const TileCost& row : kTileCosts) {
    const bool square = row.kind == GemmPlan::kLdsSquare;
    const TileCost& t = square ? square_cost(N, K) : row;
    const uint64_t tiles = (uint64_t)((M + t.bm - 1) / t.bm) * (uint64_t)((N + t.bn - 1) / t.bn);
    const bool splitk = t.kind == t.super_kind;
    const uint64_t max_rounds = K < 1024 ? kSplitkMaxRoundsShort : kSplitkMaxRounds;
    if (splitk && ((M > kSplitkMaxRows && K >= kShortK) || tiles > max_rounds * n_cu)) continue;
    for (uint32_t parts = 1; parts <= t.max_parts; ++parts) {
      const uint64_t part_bytes = (uint64_t)parts * (uint64_t)M * parts_row((uint32_t)N) * sizeof(float);
      if (parts > 1 && (!with_ws || units * unit < parts * kMinPartChunks || part_bytes > kMaxPartBytes ||
                        (square && !super)))
        break;
      // 32 x 96 tiles of eight waves fill a CU's LDS: a round's first loads and
      // epilogue (5 us, 42 chunks' worth) are not covered by another workgroup.
      const uint32_t chunks = (units + parts - 1) / parts * unit + (t.kind == GemmPlan::kSplitk32x96 ? 42 : 0);
      const float rounds = rounds_of(tiles * parts, n_cu, t.last, t.lone);
      float c = rounds * (float)chunks * (super ? t.chunk_us_super : t.chunk_us) + t.fixed_us;
      if (parts > 1) c += kSumLaunchUs + 2.0f * (float)part_bytes / kPartBytesPerUs;
      GemmPlan& b = splitk ? best_splitk : best;
      float& b_cost = splitk ? splitk_cost : *cost;
      if (b.first != GemmPlan::kNone && c >= b_cost) continue;
      b.first = super ? t.super_kind : t.kind;
      b.k_parts = parts;
      b_cost = c;
      if (splitk) splitk_round_cost = rounds > 1.0f ? (rounds - 1.0f) * t.round_us : 0.0f;
    }
  }
  if (best_splitk.first != GemmPlan::kNone) {
    const float fade = 2.0f - 2.0f * (float)K / (float)kShortK;      // from kShortK / 2 on
    if (short_k(N, K)) splitk_cost += (fade < 1.0f ? fade : 1.0f) * splitk_round_cost;
    if (splitk_cost < *cost) {
      best = best_splitk;
      *cost = splitk_cost;
    }
  }
  best.n_split = (uint32_t)N;
  return best;
}

// Square tiles fill whole rounds of one workgroup per CU.  When the last
// round would be at most half full and its tiles make whole tile columns,
// those columns run as a second launch: with a workspace and K % 512 == 0, the
// same square tiles as two K halves on twice the CUs (FP32 partial sums, then
// a summing pass: about 0.55 of a round plus the pass); otherwise as 256 x 128
// tiles (two per CU), about 0.7 of a round.  Scale super-stages need
// K % 256 == 0 (whole groups of 4 chunks).
static GemmPlan plan_square(int64_t M, int64_t N, int64_t K, uint32_t n_cu, bool with_ws) {
  GemmPlan g{};
  g.first = (K % 256) == 0 ? GemmPlan::kLdsSuper : GemmPlan::kLdsSquare;
  g.n_split = (uint32_t)N;
  g.k_parts = 1;
  const uint32_t tiles_m = (uint32_t)((M + kSquareTile - 1) / kSquareTile);
  const uint32_t tiles_n = (uint32_t)((N + kSquareTile - 1) / kSquareTile);
  const uint32_t rem = n_cu ? (tiles_m * tiles_n) % n_cu : 0;
  if (rem != 0 && rem <= n_cu / 2 && rem % tiles_m == 0 && rem / tiles_m < tiles_n) {
    g.n_split = (tiles_n - rem / tiles_m) * kSquareTile;
    g.second = (with_ws && K % 512 == 0) ? GemmPlan::kLdsSuperHalves : GemmPlan::kLdsTall;
  }
  return g;
}

// Full rounds of square tiles, then the tiles of the last round in K parts
// that spread them over all CUs: for last rounds more than half full (or not
// whole tile columns), which K halves would not shorten.  FP32 partial tiles,
// then a summing pass.  K % 256 == 0.
static GemmPlan plan_square_tiles(int64_t M, int64_t N, int64_t K, uint32_t n_cu, float* cost) {
  GemmPlan best{};
  const TileCost& sq = square_cost(N, K);
  const uint64_t tiles = (uint64_t)((M + kSquareTile - 1) / kSquareTile) * ((N + kSquareTile - 1) / kSquareTile);
  const uint64_t rem = tiles % n_cu;
  const uint32_t units = (uint32_t)(K / 256);
  for (uint32_t parts = 2; parts <= kMaxTailParts && parts <= units && rem != 0 && tiles > n_cu; ++parts) {
    const uint64_t part_bytes = (uint64_t)parts * rem * kSquareTile * kSquareTile * sizeof(float);
    if (part_bytes > kMaxPartBytes) break;
    const float tail_rounds = rounds_of(rem * parts, n_cu, sq.last, sq.lone);
    const float c = ((float)(tiles / n_cu) * (float)units + tail_rounds * (float)((units + parts - 1) / parts)) *
                        4.0f * sq.chunk_us_super + (1.0f + tail_rounds) * sq.fixed_us + kSumLaunchUs +
                    2.0f * (float)part_bytes / kPartBytesPerUs;
    if (best.first == GemmPlan::kNone || c < *cost) {
      *cost = c;
      best.first = GemmPlan::kLdsSuper;
      best.second = GemmPlan::kLdsSuperTiles;
      best.n_full = (uint32_t)(tiles - rem);
      best.tail_parts = parts;
    }
  }
  best.n_split = (uint32_t)N;
  best.k_parts = 1;
  return best;
}

// The kernels one nvfp4_gemm call launches for a shape (n_cu: compute units
// of the device).
GemmPlan plan_gemm(int64_t M, int64_t N, int64_t K, uint32_t n_cu, bool with_ws) {
  const bool aligned = (K % 64) == 0;
  GemmPlan g{};
  g.n_split = (uint32_t)N;
  g.k_parts = 1;
  if (M == 0) return g;
  if (aligned && N <= 96) {
    g.first = GemmPlan::kSplitkNarrow;
  } else if (aligned && M <= 32) {
    g.first = GemmPlan::kSplitkDecode;
  } else if (aligned) {
    // Square tiles, unless another tile shape or K parts are estimated to be
    // faster.
    g = plan_square(M, N, K, n_cu, with_ws);
    const bool tail = g.second != GemmPlan::kNone;
    if (n_cu != 0 && (!tail || K >= kTailMinK)) {
      const TileCost& sq = square_cost(N, K);
      const uint64_t tiles = (uint64_t)((M + kSquareTile - 1) / kSquareTile) * ((N + kSquareTile - 1) / kSquareTile);
      const float last = g.second == GemmPlan::kLdsSuperHalves ? 0.55f : sq.last;
      const float rounds = tail ? (float)(tiles / n_cu) + last : rounds_of(tiles, n_cu, sq.last, sq.lone);
      const float base = rounds * (float)(K / 64) * (K % 256 == 0 ? sq.chunk_us_super : sq.chunk_us) + sq.fixed_us;
      float cost, tail_cost;
      const GemmPlan t = plan_tiles(M, N, K, n_cu, with_ws, &cost);
      if (cost < kPlanGain * base) g = t; else cost = base;
      if (with_ws && K % 256 == 0) {
        const GemmPlan q = plan_square_tiles(M, N, K, n_cu, &tail_cost);
        if (q.first != GemmPlan::kNone && tail_cost < kPlanGain * cost) g = q;
      }
    }
  } else {
    const int64_t k_pad = (K + 63) / 64 * 64;
    if (with_ws && M * k_pad < ((int64_t)1 << 31)) {
      g = plan_gemm(M, N, k_pad, n_cu, true);
      g.k_pad = (uint32_t)k_pad;
    } else {
      g.first = GemmPlan::kReg;
    }
  }
  return g;
}

// K % 64 != 0 with a workspace: the shapes that stay on the register path.  It
// has no pass over the activation in front (2 us and a launch) and 256 x 256 tiles
// of 2 us per chunk; rows that allow no 16-byte stores it stores as fast as the
// tiled kernels.  It wins where the latter have to store such rows (bf16) of half
// a round of tiles or more and K is short, or of 0.4 of one up to three chunks, or
// of a quarter up to two.  Register path and padded: 8000 x 1300 (192 tiles) K = 16
// 13.5 and 15.8 us, 144 17.7 and 18.5, 528 29.5 and 31.8, 784 38 and 39; 8000 x
// 4004 x 208 36.1 and 43; 2200 x 3998 (144 tiles) x 336 21.9 and 31.3; 2200 x 3004
// (108) x 144 16.5 and 19.9; 1500 x 4004 (96 tiles) x 112 16.7 and 19, x 144 18.1
// and 16.9; 777 x 4004 (64) x 48 12.3 and 13.5; but 1500 x 1300 (36) x 16 13.2 and
// 9.0, and with 16-byte stores 3000 x 4000 x 144 17.7 and 14.
static bool keeps_register_path(int64_t M, int64_t N, int64_t K, uint32_t n_cu, bool wide_stores) {
  const uint64_t tiles = (uint64_t)((M + kSquareTile - 1) / kSquareTile) * (uint64_t)((N + kSquareTile - 1) / kSquareTile);
  if (K % 64 == 0 || wide_stores) return false;
  const uint64_t n = n_cu;
  return (K <= 9 * 64 && 2 * tiles >= n) || (K <= 3 * 64 && 5 * tiles >= 2 * n) || (K <= 2 * 64 && 4 * tiles >= n);
}

size_t plan_workspace_bytes(const GemmPlan& g, int64_t M, int64_t N) {
  const size_t pad = g.k_pad ? pad_bytes(M, g.k_pad) : 0;
  if (g.second == GemmPlan::kLdsSuperHalves)
    return pad + (size_t)2 * (size_t)M * (size_t)parts_row((uint32_t)N - g.n_split) * sizeof(float);
  if (g.second == GemmPlan::kLdsSuperTiles) {
    const size_t tiles = (size_t)((M + kSquareTile - 1) / kSquareTile) * (size_t)((N + kSquareTile - 1) / kSquareTile);
    return pad + (size_t)g.tail_parts * (tiles - g.n_full) * kSquareTile * kSquareTile * sizeof(float);
  }
  if (g.k_parts > 1) return pad + (size_t)g.k_parts * (size_t)M * (size_t)parts_row((uint32_t)N) * sizeof(float);
  return pad;
}

const char* gemm_kernel_name(int kind, bool parts) {
  switch (kind) {
    case GemmPlan::kLdsSquare: return "gemm_lds_kernel<LdsSquare> (256x256 tiles)";
    case GemmPlan::kLdsSuper:
      return parts ? "gemm_lds_kernel<LdsSquareSuper> (256x256 tiles, scale super-stages, K parts) + sum_parts_kernel"
                   : "gemm_lds_kernel<LdsSquareSuper> (256x256 tiles, scale super-stages)";
    case GemmPlan::kLdsMid:
      return parts ? "gemm_lds_kernel<LdsMid> (128x128 tiles, K parts) + sum_parts_kernel"
                   : "gemm_lds_kernel<LdsMid> (128x128 tiles)";
    case GemmPlan::kLdsMidSuper:
      return parts ? "gemm_lds_kernel<LdsMidSuper> (128x128 tiles, scale super-stages, K parts) + sum_parts_kernel"
                   : "gemm_lds_kernel<LdsMidSuper> (128x128 tiles, scale super-stages)";
    case GemmPlan::kLdsLow:
      return parts ? "gemm_lds_kernel<LdsLow> (64x256 tiles, K parts) + sum_parts_kernel"
                   : "gemm_lds_kernel<LdsLow> (64x256 tiles)";
    case GemmPlan::kLdsLowSuper:
      return parts ? "gemm_lds_kernel<LdsLowSuper> (64x256 tiles, scale super-stages, K parts) + sum_parts_kernel"
                   : "gemm_lds_kernel<LdsLowSuper> (64x256 tiles, scale super-stages)";
    case GemmPlan::kLdsSuperTiles:
      return "gemm_lds_kernel<LdsSquareSuper> (256x256 tiles of the last round, K parts) + sum_tiles_kernel";
    case GemmPlan::kLdsTall: return "gemm_lds_kernel<LdsTall> (256x128 tiles)";
    case GemmPlan::kLdsSuperHalves:
      return "gemm_lds_kernel<LdsSquareSuper> (256x256 tiles, two K halves, FP32 partials) + sum_parts_kernel";
    case GemmPlan::kSplitk32x32: return "gemm_splitk_kernel<4,1,1,3> (32x32 tiles, split-K, per-wave rings)";
    case GemmPlan::kSplitk32x64: return "gemm_splitk_kernel<4,1,2,3> (32x64 tiles, split-K, shared activation ring)";
    case GemmPlan::kSplitk64x64: return "gemm_splitk_kernel<4,2,2,3> (64x64 tiles, split-K)";
    case GemmPlan::kSplitk64x96: return "gemm_splitk_kernel<4,2,3,2> (64x96 tiles, split-K)";
    case GemmPlan::kSplitk32x96: return "gemm_splitk_kernel<8,1,3,3> (32x96 tiles, split-K, shared activation ring)";
    case GemmPlan::kSplitk32x160: return "gemm_splitk_kernel<4,1,5,2> (32x160 tiles, split-K, shared activation ring)";
    case GemmPlan::kReg: return "gemm_reg_kernel<2,2,4,4> (256x256 tiles, register path)";
    default: return "none";
  }
}

static const char* decode_kernel_name(DecodeShape d) {
  switch (d) {
    case DecodeShape::kRows16w1: return "gemm_rows16_kernel<16,1,2> (16x32 tiles, split-K)";
    case DecodeShape::kRows8w2: return "gemm_rows16_kernel<8,2,2> (16x64 tiles, split-K)";
    case DecodeShape::kRows8w3: return "gemm_rows16_kernel<8,3,2> (16x96 tiles, split-K)";
    case DecodeShape::kRows4w2: return "gemm_rows16_kernel<4,2,3> (16x64 tiles, split-K)";
    case DecodeShape::k4Private: return "gemm_splitk_kernel<4,1,1,3> (32x32 tiles, split-K, per-wave rings)";
    case DecodeShape::k8SharedPair: return "gemm_splitk_kernel<8,1,2,3> (32x64 tiles, split-K, shared activation ring)";
    case DecodeShape::k8Shared3: return "gemm_splitk_kernel<8,1,3,3> (32x96 tiles, split-K, shared activation ring)";
    case DecodeShape::k4Shared5: return "gemm_splitk_kernel<4,1,5,2> (32x160 tiles, split-K, shared activation ring)";
    case DecodeShape::k8Shared: return "gemm_splitk_kernel<8,1,1,4> (32x32 tiles, split-K, shared activation ring)";
    default: return "gemm_splitk_kernel<4,1,2,3> (32x64 tiles, split-K, shared activation ring)";
  }
}

static const char* narrow_kernel_name(int fragments) {
  switch (fragments) {
    case 1: return "gemm_splitk_kernel<8,1,1,3> (32x32 tiles, split-K, shared activation ring)";
    case 2: return "gemm_splitk_kernel<8,1,2,3> (32x64 tiles, split-K, shared activation ring)";
    case 3: return "gemm_splitk_kernel<8,1,3,3> (32x96 tiles, split-K, shared activation ring)";
    case 4: return "gemm_splitk_kernel<4,1,3,3> (32x96 tiles, split-K, shared activation ring)";
    default: return "gemm_splitk_kernel<4,2,3,3> (64x96 tiles, split-K)";
  }
}

const char* gemm_kernel_for(int64_t M, int64_t N, int64_t K, int part, bool with_ws) {
  const uint32_t n_cu = cu_count();
  if (n_cu == 0) return nullptr;
  // For bf16 rows of N columns.
  const GemmPlan g = plan_gemm(M, N, K, n_cu, with_ws && !keeps_register_path(M, N, K, n_cu, N % 8 == 0));
  if (g.k_pad) K = g.k_pad;                  // after pad_act_kernel
  const int kind = part == 0 ? g.first : g.second;
  if (kind == GemmPlan::kSplitkDecode) return decode_kernel_name(decode_shape(M, N, K, n_cu));
  if (kind == GemmPlan::kSplitkNarrow) return narrow_kernel_name(narrow_fragments(M, N, K, n_cu, NarrowUse::kProduct));
  return kind == GemmPlan::kNone ? nullptr : gemm_kernel_name(kind, part == 0 && g.k_parts > 1);
}

static hipError_t run_one(int kind, const GemmOperands& o, const GemmParams& p, uint32_t n_begin, uint32_t n_end,
                          bool out_f32, bool aligned, hipStream_t stream) {
  switch (kind) {
    case GemmPlan::kLdsSquare: return launch_lds_square(o, p, n_begin, n_end, out_f32, stream);
    case GemmPlan::kLdsSuper:
      return out_f32 ? launch_lds_super_f32(o, p, n_begin, n_end, stream)
                     : launch_lds_super_bf16(o, p, n_begin, n_end, stream);
    case GemmPlan::kLdsMid:
    case GemmPlan::kLdsMidSuper: return launch_lds_mid(o, p, kind == GemmPlan::kLdsMidSuper, 1, nullptr, out_f32, stream);
    case GemmPlan::kLdsLow:
    case GemmPlan::kLdsLowSuper: return launch_lds_low(o, p, kind == GemmPlan::kLdsLowSuper, 1, nullptr, out_f32, stream);
    case GemmPlan::kLdsTall: return launch_lds_tall(o, p, n_begin, n_end, out_f32, stream);
    case GemmPlan::kSplitkNarrow: return launch_splitk_narrow(o, p, out_f32, false, stream);
    case GemmPlan::kSplitk32x32:
    case GemmPlan::kSplitk32x64:
    case GemmPlan::kSplitk64x64:
    case GemmPlan::kSplitk32x96:
    case GemmPlan::kSplitk32x160:
    case GemmPlan::kSplitk64x96: return launch_splitk_tile(o, p, kind, out_f32, stream);
    case GemmPlan::kSplitkDecode: return launch_splitk_decode(o, p, out_f32, stream);
    case GemmPlan::kReg: return launch_reg_square(o, p, out_f32, aligned, stream);
    default: return hipSuccess;
  }
}

size_t gemm_workspace_bytes(int64_t M, int64_t N, int64_t K) {
  const uint32_t n_cu = cu_count();
  if (n_cu == 0 || M == 0) return 0;
  return plan_workspace_bytes(plan_gemm(M, N, K, n_cu, true), M, N);
}

hipError_t launch_gemm(const uint8_t* a_codes, const uint8_t* a_scales, const float* a_g,
                       int64_t M, int64_t K, const void* w_packed, int64_t N,
                       const int64_t* seg_offsets, int n_seg, const float* w_g, void* y,
                       int64_t ldy, bool out_f32, void* workspace, size_t workspace_bytes, hipStream_t stream) {
  if (M == 0) return hipSuccess;
  GemmPlan g = plan_gemm(M, N, K, cu_count(), workspace != nullptr);
  if (workspace_bytes != kNoWorkspace && workspace_bytes < plan_workspace_bytes(plan_gemm(M, N, K, cu_count(), true), M, N)) {
    g = plan_gemm(M, N, K, cu_count(), false);
    if (K % 64 == 0 && N > 96 && M > 32) {
      const GemmPlan h = plan_square(M, N, K, cu_count(), true);
      if (workspace_bytes < plan_workspace_bytes(h, M, N)) return kWorkspaceTooSmall;
      if (h.second == GemmPlan::kLdsSuperHalves) g = h;
    }
  }
  const bool wide_stores = out_f32 || (ldy % 8 == 0 && reinterpret_cast<uintptr_t>(y) % 16 == 0);
  if (g.k_pad && keeps_register_path(M, N, K, cu_count(), wide_stores)) g = plan_gemm(M, N, K, cu_count(), false);
  float* parts = static_cast<float*>(workspace);
  if (g.k_pad) {
    uint8_t* pc = static_cast<uint8_t*>(workspace);
    uint8_t* ps = pc + pad_code_bytes(M, g.k_pad);
    const hipError_t e = launch_pad_act(a_codes, a_scales, M, K, g.k_pad, pc, ps, stream);
    if (e != hipSuccess) return e;
    a_codes = pc;
    a_scales = ps;
    parts = reinterpret_cast<float*>(pc + pad_bytes(M, g.k_pad));
    K = g.k_pad;
  }
  GemmParams p = gemm_params(M, K, N, seg_offsets, n_seg, ldy);
  p.y_pairs = (ldy % 2 == 0) && (reinterpret_cast<uintptr_t>(y) % 4 == 0) ? 1u : 0u;
  p.y_stream = !out_f32 && (uint64_t)M * (uint64_t)N * 2u >= kMallBytes ? 1u : 0u;
  const GemmOperands o{a_codes, a_scales, a_g, static_cast<const uint8_t*>(w_packed), w_g, y};
  const bool aligned = (K % 64) == 0;
  if (g.k_parts > 1) {
    hipError_t e;
    if (g.first == GemmPlan::kLdsSuper)
      e = launch_lds_super_parts(o, p, 0, (uint32_t)N, g.k_parts, parts, stream);
    else if (g.first == GemmPlan::kLdsMid || g.first == GemmPlan::kLdsMidSuper)
      e = launch_lds_mid(o, p, g.first == GemmPlan::kLdsMidSuper, g.k_parts, parts, true, stream);
    else
      e = launch_lds_low(o, p, g.first == GemmPlan::kLdsLowSuper, g.k_parts, parts, true, stream);
    if (e != hipSuccess) return e;
    return launch_sum_parts(parts, o, p, g.k_parts, 0, out_f32, stream);
  }
  if (g.second == GemmPlan::kLdsSuperTiles) {
    const uint32_t tiles = (uint32_t)((M + kSquareTile - 1) / kSquareTile) * (uint32_t)((N + kSquareTile - 1) / kSquareTile);
    hipError_t e = launch_lds_super_tiles(o, p, 0, g.n_full, out_f32, stream);
    if (e == hipSuccess) e = launch_lds_super_tile_parts(o, p, g.n_full, tiles, g.tail_parts, parts, stream);
    if (e == hipSuccess) e = launch_sum_tiles(parts, o, p, g.n_full, tiles, g.tail_parts, out_f32, stream);
    return e;
  }
  hipError_t e = run_one(g.first, o, p, 0, g.n_split, out_f32, aligned, stream);
  if (e != hipSuccess || g.second == GemmPlan::kNone) return e;
  if (g.second == GemmPlan::kLdsSuperHalves) {
    e = launch_lds_super_parts(o, p, g.n_split, (uint32_t)N, 2, parts, stream);
    if (e != hipSuccess) return e;
    return launch_sum_parts(parts, o, p, 2, g.n_split, out_f32, stream);
  }
  return run_one(g.second, o, p, g.n_split, (uint32_t)N, out_f32, aligned, stream);
}

hipError_t launch_gemm_gdn_gates(const uint8_t* a_codes, const uint8_t* a_scales, const float* a_g,
                                 int64_t M, int64_t K, const void* w_packed, int64_t H, const float* w_g,
                                 const float* a_log, const float* dt_bias, void* y, int64_t ldy,
                                 bool out_f32, hipStream_t stream) {
  if (M == 0) return hipSuccess;
  const int64_t offs[3] = {0, H, 2 * H};
  GemmParams p = gemm_params(M, K, 2 * H, offs, 2, ldy);
  p.gate_a_log = a_log;
  p.gate_dt_bias = dt_bias;
  p.gate_h = (uint32_t)H;
  const GemmOperands o{a_codes, a_scales, a_g, static_cast<const uint8_t*>(w_packed), w_g, y};
  return launch_splitk_narrow(o, p, out_f32, true, stream);
}

}  // namespace nvfp4
