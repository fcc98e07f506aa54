// Device-side description of a batched neural-field solve, shared by the
// kernels that drive it.
#pragma once

#include <hip/hip_runtime.h>

#include "common.hpp"

namespace bode {

template <typename R>
struct Mod {
  int32_t B, D, E, H, cnf, d_in;  // d_in: state features fed to the field
  const R* y0;
  const double *t0, *t_end, *rtol, *atol, *t_eval, *h0;
  const R *W1, *b1, *W2, *b2, *W3, *b3, *eps;
  R* y_eval;
  R* y_final;
  State<R> st;     // t, h, error history, counters, status, cursor, y, k1
  R* K;            // [7, B, D] stages (K[0] = k1 = st.k1)
  R* Y7;           // [B, D] stage-7 input = candidate solution
  R* hs;           // [B] size of the current attempt
  int32_t* last;   // [B] the current attempt ends on t_end
  R* aux;          // [B] start-step scratch
  double* h_rec;   // [B, rec_cap] attempt record (rejected < 0)
  double* e_rec;   // [B, rec_cap] the attempts' error norms
  int32_t rec_cap;
  int32_t* n_running;
  DenseKeep<R> dk;
  int32_t keep;
  Ctrl ctrl;
  R* ckpt;          // [B, ck_cap, D] y_n for n = 0, k, 2k, ... (or nullptr)
  int32_t ck_every, ck_cap;
  R *wp, *wpT;      // FP64 matrix cores: packed layers, transposed layers
};

}  // namespace bode
