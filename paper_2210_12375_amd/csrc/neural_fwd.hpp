// Forward kernels of the neural fields (neural_tile.hpp): a
// whole solve, one step's seven stage evaluations, one stage evaluation.
#pragma once

#include <hip/hip_runtime.h>

#include "mlp_mfma.hpp"
#include "mod.hpp"

namespace bode {

// A pair's coefficients, for kernels not specialised on it.
struct TableauArgs {
  float A[7][6];
  float E[7];
  float P[7][4];
  double C[7];
  int32_t dense;  // bit j: stage j takes part in the interpolant
};

template <class M>
TableauArgs tableau_args() {
  TableauArgs t{};
  for (int s = 0; s < 7; ++s) {
    t.E[s] = float(M::E[s]);
    t.C[s] = M::C[s];
    for (int j = 0; j < 6 && j < s; ++j) t.A[s][j] = float(M::A[s][j]);
    for (int q = 0; q < 4; ++q) {
      t.P[s][q] = float(M::P[s][q]);
      if (M::P[s][q] != 0.0) t.dense |= 1 << s;
    }
  }
  return t;
}

// One step's stages 0 .. 6 of the rows with status kRunning: stage inputs to
// Y[s] and hidden layers to act[s] (MfmaArgs::act_out's layout) where set.
struct FwdSteps {
  int B, D;
  const int32_t* status;
  const float *y, *hs, *eps;
  const double* t;
  float* Y[7];
  float* act[7];
};

// waves: 8 for one 16-row tile per workgroup, 4 for two, 0 for the default
// (where both are built: row_tile_choice).  Both give bitwise the same results.
hipError_t fwd_solve(const Mod<float>& m, const MfmaWeights& w,
                     const TableauArgs& t, int budget, int waves,
                     hipStream_t s);
hipError_t fwd_steps(const FwdSteps& v, int din, int H, bool cnf,
                     const MfmaWeights& w, const TableauArgs& t, int waves,
                     hipStream_t s);
hipError_t fwd_stage(const MfmaArgs& a, hipStream_t s);

// One source file per padded width and mode (_f32: FP32 mode).
struct FwdCall {
  int kind;  // 0 solve, 1 steps, 2 stage
  const Mod<float>* m;
  const FwdSteps* steps;
  const MfmaArgs* stage;
  const TableauArgs* tab;
  int B, D, din, H, cnf, budget, waves;
  MfmaWeights w;
};
hipError_t fwd_h64(const FwdCall& c, hipStream_t s);
hipError_t fwd_f32_h64(const FwdCall& c, hipStream_t s);
hipError_t fwd_h128(const FwdCall& c, hipStream_t s);
hipError_t fwd_f32_h128(const FwdCall& c, hipStream_t s);
hipError_t fwd_h256(const FwdCall& c, hipStream_t s);
hipError_t fwd_f32_h256(const FwdCall& c, hipStream_t s);
hipError_t fwd_h512(const FwdCall& c, hipStream_t s);
hipError_t fwd_f32_h512(const FwdCall& c, hipStream_t s);

}  // namespace bode
