// Vector-Jacobian products of the FP32 neural fields at hidden width 256.
#define BODE_NEURAL_F32
#include "neural_bwd.inc"

namespace bode {
hipError_t bwd_f32_h256(const BwdCall& c, hipStream_t s) {
  return bwd_width<2, 8>(c, s);
}
}  // namespace bode
