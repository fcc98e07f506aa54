// Vector-Jacobian products of the neural fields at hidden width 64.
#include "neural_bwd.inc"

namespace bode {
hipError_t bwd_h64(const BwdCall& c, hipStream_t s) {
  return bwd_width<1, 4>(c, s);
}
}  // namespace bode
