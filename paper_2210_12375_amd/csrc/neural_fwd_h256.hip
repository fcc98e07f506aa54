// Forward kernels of the neural fields at hidden width 256.
#include "neural_fwd.inc"

namespace bode {
hipError_t fwd_h256(const FwdCall& c, hipStream_t s) {
  return fwd_width<2, 8>(c, s);
}
}  // namespace bode
