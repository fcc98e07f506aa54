// Forward kernels of the FP32 neural fields at hidden width 128.
#define BODE_NEURAL_F32
#include "neural_fwd.inc"

namespace bode {
hipError_t fwd_f32_h128(const FwdCall& c, hipStream_t s) {
  return fwd_width<1, 8>(c, s);
}
}  // namespace bode
