// Forward kernels of the FP32 neural fields at hidden width 64.
#define BODE_NEURAL_F32
#include "neural_fwd.inc"

namespace bode {
hipError_t fwd_f32_h64(const FwdCall& c, hipStream_t s) {
  return fwd_width<1, 4>(c, s);
}
}  // namespace bode
