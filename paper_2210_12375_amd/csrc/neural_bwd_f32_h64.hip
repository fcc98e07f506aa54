// Vector-Jacobian products of the FP32 neural fields at hidden width 64.
#define BODE_NEURAL_F32
#include "neural_bwd.inc"

namespace bode {
hipError_t bwd_f32_h64(const BwdCall& c, hipStream_t s) {
  return bwd_width<1, 4>(c, s);
}
}  // namespace bode
