// Prefill GEMM instantiation: LdsSquareSuper, bf16 output (see gemm_lds.h).
#include "gemm_lds.h"

namespace nvfp4 {

hipError_t launch_lds_super_bf16(const GemmOperands& o, GemmParams p, uint32_t n_begin, uint32_t n_end,
                                 hipStream_t stream) {
  return launch_lds_as<LdsSquareSuper, false>(o, p, n_begin, n_end, stream);
}

hipError_t launch_lds_super_tiles(const GemmOperands& o, const GemmParams& p, uint32_t tile_begin, uint32_t tile_end,
                                  bool out_f32, hipStream_t stream) {
  GemmParams q = p;
  q.tile_begin = tile_begin;
  q.tile_count = tile_end - tile_begin;
  return out_f32 ? launch_lds_super_f32(o, q, 0, p.N, stream) : launch_lds_super_bf16(o, q, 0, p.N, stream);
}

}  // namespace nvfp4
