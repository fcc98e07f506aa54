// Vector-Jacobian products of the neural fields at hidden width 128.
#include "neural_bwd.inc"

namespace bode {
hipError_t bwd_h128(const BwdCall& c, hipStream_t s) {
  return bwd_width<1, 8>(c, s);
}
}  // namespace bode
