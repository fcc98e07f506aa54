// Forward kernels of the neural fields at hidden width 128.
#include "neural_fwd.inc"

namespace bode {
hipError_t fwd_h128(const FwdCall& c, hipStream_t s) {
  return fwd_width<1, 8>(c, s);
}
}  // namespace bode
