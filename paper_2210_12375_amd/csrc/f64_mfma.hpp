// FP64 evaluation of the neural fields (MLP and CNF) on the FP64 matrix
// cores of gfx950, forward and vector-Jacobian product.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>

#include "vjp_dense.hpp"

namespace bode {

// One stage evaluation (the members have MfmaArgs' meaning).
struct F64Args {
  int B, D, din, H, cnf;
  const int32_t* status;
  const double *y, *K, *hs, *t, *eps;
  double* Y7;
  const double *W, *b1, *b2, *b3;  // packed layers; biases as given
  int n;
  int kidx[6];
  double coef[6];
  double c;
  int write_y7;
  double* out;
  double* act_out;  // [Bs][2][H], or null
  int kslot;
};

// One stage of the adjoint (BwdArgs' meaning, stage by stage); the forward
// layers are always read from act_in.
struct F64VjpArgs {
  int B, D, din, H, cnf;
  const int32_t* act;
  const double *Y, *kap_s, *eps, *bh, *bt;
  double c;
  const double* WT;  // packed transposed layers
  double *T1in, *T1g, *T2in, *T2g, *T3in, *T3g;
  long kb;
  int s, n;
  int kidx[6];
  double coef[6];
  double *lam, *lamn, *kap;
  double* mu_out;
  const double* act_in;
};

struct F64Steps {
  F64Args st[7];
  int n;
  int kl, kl_off;  // as in MfmaSteps
};

struct F64VjpSteps {
  F64VjpArgs st[7];
  int n;
  VjpDenseT<double> dense;
  int cl_off;  // set by the launcher
};
static_assert(sizeof(F64Steps) <= 4096 && sizeof(F64VjpSteps) <= 4096,
              "step arguments exceed the kernel-argument space");

// Whether the kernels' LDS holds a field of this shape.
bool f64_fits(int D, int din, int H, bool cnf);
size_t f64_packed_elems(int din, int H);   // forward layers
size_t f64_packedT_elems(int din, int H);  // transposed layers
hipError_t f64_pack_weights(double* W, double* WT, int din, int H,
                            const double* W1, const double* W2,
                            const double* W3, hipStream_t s);
// Up to seven stages of one step in one launch, in order.
hipError_t launch_field_f64(const F64Steps& v, hipStream_t s);
hipError_t launch_vjp_f64(const F64VjpSteps& v, hipStream_t s);

}  // namespace bode
