// Backward kernels of float16 inputs (one translation unit per input type, built
// in parallel).
#include "bwd_kernels.hpp"

namespace mea {

hipError_t launch_bwd_f16(const BwdParams& p, int d, int dv, bool causal, bool out_f32, hipStream_t stream) {
  return out_f32 ? launch_bwd_dims<_Float16, float>(p, d, dv, causal, stream)
                 : launch_bwd_dims<_Float16, _Float16>(p, d, dv, causal, stream);
}

}  // namespace mea
