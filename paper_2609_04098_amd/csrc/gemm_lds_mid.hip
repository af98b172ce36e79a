// Prefill GEMM instantiation: LdsMid, LdsMidSuper (see gemm_lds.h).
#include "gemm_lds.h"

namespace nvfp4 {

hipError_t launch_lds_mid(const GemmOperands& o, const GemmParams& p, bool super, uint32_t k_parts, float* parts,
                          bool out_f32, hipStream_t stream) {
  if (k_parts > 1)
    return super ? launch_lds_parts<LdsMidSuper>(o, p, 0, p.N, k_parts, parts, stream)
                 : launch_lds_parts<LdsMid>(o, p, 0, p.N, k_parts, parts, stream);
  return super ? launch_lds<LdsMidSuper>(o, p, 0, p.N, out_f32, stream)
               : launch_lds<LdsMid>(o, p, 0, p.N, out_f32, stream);
}

}  // namespace nvfp4
