// Prefill GEMM instantiation: LdsLow, LdsLowSuper (see gemm_lds.h).
#include "gemm_lds.h"

namespace nvfp4 {

hipError_t launch_lds_low(const GemmOperands& o, const GemmParams& p, bool super, uint32_t k_parts, float* parts,
                          bool out_f32, hipStream_t stream) {
  if (k_parts > 1)
    return super ? launch_lds_parts<LdsLowSuper>(o, p, 0, p.N, k_parts, parts, stream)
                 : launch_lds_parts<LdsLow>(o, p, 0, p.N, k_parts, parts, stream);
  return super ? launch_lds<LdsLowSuper>(o, p, 0, p.N, out_f32, stream)
               : launch_lds<LdsLow>(o, p, 0, p.N, out_f32, stream);
}

}  // namespace nvfp4
