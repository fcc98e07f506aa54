// Forward kernels of the neural fields at hidden width 64.
#include "neural_fwd.inc"

namespace bode {
hipError_t fwd_h64(const FwdCall& c, hipStream_t s) {
  return fwd_width<1, 4>(c, s);
}
}  // namespace bode
