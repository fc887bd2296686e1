// The fast kernel's logits products (vp_gemm_bf16_fast.h): pass S with its statistics, pass T with logits formed again.
#include "vp_gemm_bf16_fast.h"

namespace vp {

hipError_t launch_gemm_bf16_fwd_stats(const GemmBf16Group& g, hipStream_t st) { return launch_fast_t<true, true, Epi::FwdStats>(g, st); }
hipError_t launch_gemm_bf16_dlogits(const GemmBf16Group& g, hipStream_t st) { return launch_fast_t<true, true, Epi::DLogits>(g, st); }

}  // namespace vp
