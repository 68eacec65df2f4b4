// Backward dispatch over the input types (their kernels are in bwd_f32.hip,
// bwd_f16.hip and bwd_bf16.hip).
#include "kernels.hpp"

namespace mea {

hipError_t launch_bwd_f32(const BwdParams& p, int d, int dv, bool causal, hipStream_t stream);
hipError_t launch_bwd_f16(const BwdParams& p, int d, int dv, bool causal, bool out_f32, hipStream_t stream);
hipError_t launch_bwd_bf16(const BwdParams& p, int d, int dv, bool causal, bool out_f32, hipStream_t stream);

hipError_t launch_bwd(const BwdParams& p, int dtype, int d, int dv, bool causal, bool out_f32,
                      hipStream_t stream) {
  if ((d != 64 && d != 128) || (dv != 64 && dv != 128)) return hipErrorInvalidValue;
  switch (dtype) {
    case 0: return launch_bwd_f32(p, d, dv, causal, stream);
    case 1: return launch_bwd_f16(p, d, dv, causal, out_f32, stream);
    case 2: return launch_bwd_bf16(p, d, dv, causal, out_f32, stream);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace mea
