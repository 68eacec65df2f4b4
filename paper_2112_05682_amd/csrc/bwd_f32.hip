// Backward kernels of float32 inputs (one translation unit per input type, built
// in parallel).
#include "bwd_kernels.hpp"

namespace mea {

hipError_t launch_bwd_f32(const BwdParams& p, int d, int dv, bool causal, hipStream_t stream) {
  return launch_bwd_dims<float, float>(p, d, dv, causal, stream);
}

}  // namespace mea
