// Forward kernels of the neural fields at hidden width 512.
#include "neural_fwd.inc"

namespace bode {
hipError_t fwd_h512(const FwdCall& c, hipStream_t s) {
  return fwd_width<4, 8>(c, s);
}
}  // namespace bode
