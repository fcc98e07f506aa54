// Vector-Jacobian products of the FP32 neural fields at hidden width 128.
#define BODE_NEURAL_F32
#include "neural_bwd.inc"

namespace bode {
hipError_t bwd_f32_h128(const BwdCall& c, hipStream_t s) {
  return bwd_width<1, 8>(c, s);
}
}  // namespace bode
