// Vector-Jacobian products of the neural fields at hidden width 256.
#include "neural_bwd.inc"

namespace bode {
hipError_t bwd_h256(const BwdCall& c, hipStream_t s) {
  return bwd_width<2, 8>(c, s);
}
}  // namespace bode
