// Vector-Jacobian products of the neural fields (neural_tile.hpp): the seven adjoint stages of one step, or one stage of
// the continuous adjoint.
#pragma once

#include <hip/hip_runtime.h>

#include "mlp_mfma.hpp"
#include "neural_fwd.hpp"
#include "vjp_dense.hpp"

namespace bode {

struct BwdArgs {
  int B, D;
  // Stage s = 1 .. 7 (index s - 1): stage inputs [B, D] and the hidden
  // layers its evaluation stored (MfmaArgs::act_out's layout).
  const float* Y[7];
  const float* act[7];
  const float* eps;
  // tape (sample-major); stage s's rows start at kb + (s - 1) Bs
  float *T1in, *T1g, *T2in, *T2g, *T3in, *T3g;
  long kb, Bs;
  // Discrete adjoint: the stages 7 .. 1 of step dense.step; lam [B, D] is
  // the cotangent of y_n+1, replaced by that of y_n.
  float* lam;
  VjpDenseT<float> dense;
  // Continuous adjoint (mu != null): stage s1 only, mu [B, D] = J^T kap of
  // the rows with status kRunning, at times t + c h, with the stage's adjoint
  // kap [B, D] = a0 - h sum_j coef[j] muj[j] formed here and stored.
  float* mu;
  int s1;
  float* kap;
  const float* a0;
  const float* muj[6];
  float coef[6];
  int nc;
  const int32_t* status;
  const float* hs;
  const double* t;
  double c;
};

struct BwdCall {
  const BwdArgs* a;
  const TableauArgs* tab;
  int din, H, cnf, waves;
  MfmaWeights w;
};

hipError_t bwd_run(const BwdCall& c, hipStream_t s);
hipError_t bwd_h64(const BwdCall& c, hipStream_t s);
hipError_t bwd_f32_h64(const BwdCall& c, hipStream_t s);
hipError_t bwd_h128(const BwdCall& c, hipStream_t s);
hipError_t bwd_f32_h128(const BwdCall& c, hipStream_t s);
hipError_t bwd_h256(const BwdCall& c, hipStream_t s);
hipError_t bwd_f32_h256(const BwdCall& c, hipStream_t s);
hipError_t bwd_h512(const BwdCall& c, hipStream_t s);
hipError_t bwd_f32_h512(const BwdCall& c, hipStream_t s);

}  // namespace bode
