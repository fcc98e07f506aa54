// Vector-Jacobian products of the neural fields at hidden width 512.
#include "neural_bwd.inc"

namespace bode {
hipError_t bwd_h512(const BwdCall& c, hipStream_t s) {
  return bwd_width<4, 8>(c, s);
}
}  // namespace bode
