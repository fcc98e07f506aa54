// The dense-output part of one discrete-adjoint step, shared by the
// per-step vector-Jacobian-product kernels.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "common.hpp"

namespace bode {

// The step's dense-output cotangents and step view, formed by the
// workgroup of each tile before its first stage (the discrete adjoint's
// dense-output kernel, folded in): zero lambda_next and the seven kappa
// rows, add h w_j(theta) g to kappa_j and g to lambda_next for every
// evaluation time the step answers, and (setup) the step view act, bh, bt.
template <typename R>
struct VjpDenseT {
  int on, setup, step, cap, E;
  const int32_t* nacc;   // [B] accepted steps in the record
  const double* hacc;    // [B, cap] accepted step sizes
  const double* tn;      // [B, cap + 1] step start times
  const int32_t* owner;  // [B, E] step answering each evaluation time
  const double* t_eval;  // [B, E]
  const R* g_eval;       // [B, E, D] cotangents of the outputs
  R P[7][4];             // interpolant weights: w_j = th (P0 + th (P1 + ...))
  int32_t* act;          // [B] step view (setup)
  R* bh;
  double* bt;
};

// For the tile's PR instances, one wavefront per row.  kap [7, B, D] and
// lamn [B, D] are the cotangents, or (CL) slots 0-6 and 7 of the tile's
// [8][PR][D] block at cl.
template <int PR, int WV, bool CL, typename R>
__device__ __forceinline__ void vjp_dense_rows(const VjpDenseT<R>& d, R* kapg,
                                               R* lamg, int B, int D, R* cl) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  for (int r = wave; r < PR; r += WV) {
    const int row = blockIdx.x * PR + r;
    if (row >= B) continue;
    const int n = d.step;
    const bool on = n < d.nacc[row];
    if (d.setup && lane == 0) {
      d.act[row] = on ? kRunning : kSuccess;
      d.bh[row] = on ? R(d.hacc[(long)row * d.cap + n]) : R(0);
      d.bt[row] = on ? d.tn[(long)row * (d.cap + 1) + n] : 0.0;
    }
    // kappa_j of (row, c): the tile's LDS block or HBM
    auto kap = [&](int j, int c) -> R& {
      return CL ? cl[(j * PR + r) * D + c] : kapg[((long)j * B + row) * D + c];
    };
    auto lamn = [&](int c) -> R& {
      return CL ? cl[(7 * PR + r) * D + c] : lamg[(long)row * D + c];
    };
    for (int c = lane; c < D; c += 64) {
      lamn(c) = R(0);
      for (int j = 0; j < 7; ++j) kap(j, c) = R(0);
    }
    if (!on || d.E == 0) continue;
    const double h = d.hacc[(long)row * d.cap + n];
    const double t = d.tn[(long)row * (d.cap + 1) + n];
    const int32_t* own = d.owner + (long)row * d.E;
    for (int e = 0; e < d.E; ++e) {
      if (own[e] != n) continue;
      const R th = R((d.t_eval[(long)row * d.E + e] - t) / h);
      R w[7];
#pragma unroll
      for (int j = 0; j < 7; ++j)
        w[j] = th * (d.P[j][0] +
                     th * (d.P[j][1] + th * (d.P[j][2] + th * d.P[j][3])));
      for (int c = lane; c < D; c += 64) {
        const R g = d.g_eval[((long)row * d.E + e) * D + c];
        for (int j = 0; j < 7; ++j) kap(j, c) += R(h) * w[j] * g;
        lamn(c) += g;
      }
    }
  }
}

}  // namespace bode
