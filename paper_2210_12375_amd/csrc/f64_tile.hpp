// Device building blocks of the FP64 neural fields, shared by the step
// kernels and the fused solve.
//
// A workgroup of eight wavefronts owns a tile of RT = 4 MT rows (instances;
// for the CNF the upper half are the tangent rows of the lower half) and
// runs v_mfma_f64_4x4x4_4b_f64: four 4x4 blocks of C share one 4-row operand
// (the same rows broadcast to every block, read from LDS) and take four
// neighbouring column groups, so one instruction is a [4 x 4] x [4 x 16]
// product at the full FP64 matrix rate.  The 4-row granularity is why this
// form and not 16x16x4: a field of 1000 instances is 63 tiles of 16 rows for
// 256 compute units, but 250 tiles of 4.
//
// Lane l of a product holds A[i = l % 4][k = l / 16], B[k = l / 16][j =
// l % 16] and C[i = l / 16][j = l % 16].  Weights are packed once per solve
// into fragments of 8 k x 16 columns, two consecutive k per lane (16-byte
// loads, 1 KiB contiguous per fragment), zero beyond the layer; four k
// blocks are kept in flight.
//
// Bound: at 4 rows a tile, the weight stream (65->256->256->64: 786 KB per
// evaluation and tile from L2, about 12 k cycles at 64 B per cycle), then
// the two layers of double-precision tanh (about 400 cycles per wavefront
// and 64 elements); from 8 rows up, the matrix cores (12.3 k cycles).
// Measured against one plain FMA kernel per stage (a thread per output
// column, weights re-read by every row block) and a host read-back per eight
// attempts: 1000 instances of 65->256->256->64 forward 5.36 -> 0.57 ms; 250
// of 33->128->128->32 forward and backward 25.4 -> 1.31 ms (0.52 and 0.99
// with the tanh below and the tape products on the matrix cores).
#pragma once

#include <hip/hip_runtime.h>

#include "common.hpp"
#include "f64_mfma.hpp"
#include "f64_shape.hpp"
#include "tanh.hpp"

namespace bode {
namespace f64t {

typedef double d2 __attribute__((ext_vector_type(2)));

// C[MT][NT] += A (LDS, 4 MT rows) x column tiles nb0 .. nb0 + NT - 1 of the
// packed layer at W (nk k blocks, nn column tiles; tiles past the last are
// computed on the last one's weights and not used).
template <int MT, int NT>
__device__ __forceinline__ void gemm(double (&acc)[MT][NT], const double* A,
                                     int lda, const double* W, int nk, int nn,
                                     int nb0, int lane) {
  constexpr int P = 4;
  const d2* W2 = reinterpret_cast<const d2*>(W);
  const double* Al = A + (lane & 3) * lda + (lane >> 4) * 2;
  d2 w[P][NT];
  auto fill = [&](d2(&d)[NT], int kb) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      const int nb = nb0 + t < nn ? nb0 + t : nn - 1;
      d[t] = W2[((long)kb * nn + nb) * 64 + lane];
    }
  };
#pragma unroll
  for (int p = 0; p < P; ++p) fill(w[p], p < nk ? p : nk - 1);
  __builtin_amdgcn_sched_barrier(0);
  for (int k0 = 0; k0 < nk; k0 += P) {
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const int kb = k0 + p;
      if (kb >= nk) break;
      d2 a[MT];
#pragma unroll
      for (int g = 0; g < MT; ++g)
        a[g] = *reinterpret_cast<const d2*>(Al + g * 4 * lda + kb * 8);
#pragma unroll
      for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int g = 0; g < MT; ++g)
            acc[g][t] = __builtin_amdgcn_mfma_f64_4x4x4f64(a[g][q], w[p][t][q],
                                                           acc[g][t], 0, 0, 0);
      fill(w[p], kb + P < nk ? kb + P : nk - 1);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  settle(acc);
}

// The field for the tile of instances starting at r0.  KL: the stage values
// are a [7][rows][D] block in LDS at kl instead of a.K / a.out.
template <int MT, int NT, bool CNF, bool KL>
__device__ __forceinline__ void field_tile(const F64Args& a, int r0,
                                           double* smem, double* kl) {
  constexpr int RT = 4 * MT, PR = CNF ? RT / 2 : RT, MP = CNF ? MT / 2 : MT;
  const int B = a.B, D = a.D, din = a.din, H = a.H;
  const Dims d = dims(din, H);
  double* X = smem;
  double* A0 = X + RT * d.SX;
  double* A1 = A0 + RT * d.SA;
  __shared__ int any_running;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i4 = lane >> 4, col = lane & 15;
  if (tid == 0) any_running = 0;
  __syncthreads();
  if (tid < PR && r0 + tid < B && a.status[r0 + tid] == kRunning)
    any_running = 1;
  __syncthreads();
  if (!any_running) return;

  // stage input Y = y + h sum_j a_sj k_j, the time feature, the probe on
  // the tangent rows; zeros up to the last k block
  for (int idx = tid; idx < PR * D; idx += blockDim.x) {
    const int r = idx / D, c = idx % D, row = r0 + r;
    double Yv = 0.0;
    if (row < B) {
      double acc = 0.0;
#pragma unroll
      for (int j = 0; j < 6; ++j)
        if (j < a.n)
          acc += a.coef[j] * (KL ? kl[(a.kidx[j] * PR + r) * D + c]
                                 : a.K[((long)a.kidx[j] * B + row) * D + c]);
      Yv = a.y[(long)row * D + c] + a.hs[row] * acc;
      if (a.write_y7) a.Y7[(long)row * D + c] = Yv;
    }
    if (c < din) {
      X[r * d.SX + c] = Yv;
      if (CNF)
        X[(PR + r) * d.SX + c] = row < B ? a.eps[(long)row * D + c] : 0.0;
    }
  }
  for (int r = tid; r < RT; r += blockDim.x) {
    const int row = r0 + r;
    X[r * d.SX + din] =
        r < PR && row < B ? a.t[row] + a.c * a.hs[row] : 0.0;
    for (int c = din + 1; c < d.nk1 * 8; ++c) X[r * d.SX + c] = 0.0;
  }
  __syncthreads();

#pragma unroll
  for (int layer = 0; layer < 2; ++layer) {
    const double* W = layer == 0 ? a.W : a.W + (size_t)d.nk1 * d.nnh * kFrag;
    const double* bias = layer == 0 ? a.b1 : a.b2;
    double* dst = layer == 0 ? A0 : A1;
    for (int nb0 = wave * NT; nb0 < d.nnh; nb0 += kWV * NT) {
      double acc[MT][NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int n = (nb0 + t) * 16 + col;
        const double b = n < H ? bias[n] : 0.0;
#pragma unroll
        for (int g = 0; g < MT; ++g) acc[g][t] = g < MP ? b : 0.0;
      }
      if (layer == 0)
        gemm<MT, NT>(acc, X, d.SX, W, d.nk1, d.nnh, nb0, lane);
      else
        gemm<MT, NT>(acc, A0, d.SA, W, d.nkh, d.nnh, nb0, lane);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int n = (nb0 + t) * 16 + col;
        if (nb0 + t >= d.nnh) continue;
#pragma unroll
        for (int g = 0; g < MP; ++g) {
          const int r = g * 4 + i4, row = r0 + r;
          // (padding columns stay zero: 0 x inf would spread NaN)
          const double v = n < H ? tanh64<HwMath>(acc[g][t]) : 0.0;
          dst[r * d.SA + n] = v;
          if (CNF)
            dst[(PR + r) * d.SA + n] =
                n < H ? (1.0 - v * v) * acc[MP + g][t] : 0.0;
          if (a.act_out != nullptr && row < B && n < H) {
            a.act_out[((long)row * 2 + layer) * H + n] = v;
            if (CNF)
              a.act_out[((long)(row + B) * 2 + layer) * H + n] =
                  acc[MP + g][t];
          }
        }
      }
    }
    __syncthreads();
  }

  // output layer: one column tile a wavefront at a time
  {
    const double* W =
        a.W + ((size_t)d.nk1 * d.nnh + (size_t)d.nkh * d.nnh) * kFrag;
    for (int nb = wave; nb < d.nnd; nb += kWV) {
      const int n = nb * 16 + col;
      double acc[MT][1];
      const double b = n < din ? a.b3[n] : 0.0;
#pragma unroll
      for (int g = 0; g < MT; ++g) acc[g][0] = g < MP ? b : 0.0;
      gemm<MT, 1>(acc, A1, d.SA, W, d.nkh, d.nnd, nb, lane);
      if (n < din) {
#pragma unroll
        for (int g = 0; g < MP; ++g) {
          const int r = g * 4 + i4, row = r0 + r;
          if (KL)
            kl[(a.kslot * PR + r) * D + n] = acc[g][0];
          else if (row < B)
            a.out[(long)row * D + n] = acc[g][0];
          // probe times tangent output, into the inputs' rows (free: every
          // wave is past layer 1; the layer buffers' rows are as wide as
          // the hidden layer, which may be narrower than the state)
          if (CNF)
            X[r * d.SX + n] =
                row < B ? a.eps[(long)row * D + n] * acc[MP + g][0] : 0.0;
        }
      }
    }
    if (CNF) {
      // l' = -eps^T (dg/dz) eps, summed in output order
      __syncthreads();
      for (int r = tid; r < PR; r += blockDim.x) {
        const int row = r0 + r;
        double q = 0.0;
        for (int j = 0; j < din; ++j) q += X[r * d.SX + j];
        if (KL)
          kl[(a.kslot * PR + r) * D + din] = -q;
        else if (row < B)
          a.out[(long)row * D + din] = -q;
      }
    }
  }
}

// One adjoint stage of the tile: mu = J^T kappa from the stored forward
// layers, the stage's tape rows, and the row updates.  CL: kappa and
// lambda_next are the [8][rows][D] block at cl (as in the FP32 / BF16
// kernel).
template <int MT, int NT, bool CNF, bool CL>
__device__ __forceinline__ void vjp_tile(const F64VjpArgs& a, int r0,
                                         double* smem, double* cl) {
  constexpr int RT = 4 * MT, PR = CNF ? RT / 2 : RT, MP = CNF ? MT / 2 : MT;
  const int B = a.B, D = a.D, din = a.din, H = a.H;
  const Dims d = dims(din, H);
  double* X = smem;
  double* A0 = X + RT * d.SX;
  double* A1 = A0 + RT * d.SA;
  double* MU = X;  // [PR][din] once S2 has read the cotangents
  __shared__ int any_running;
  __shared__ int onr[16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int i4 = lane >> 4, col = lane & 15;
  if (tid == 0) any_running = 0;
  __syncthreads();
  if (tid < PR) {
    const int o = r0 + tid < B && a.act[r0 + tid] == kRunning;
    onr[tid] = o;
    if (o) any_running = 1;
  }
  __syncthreads();
  const long l1 = din + 2, lh = H + 1;
  constexpr int nr = CNF ? 2 : 1;
  if (!any_running) {
    // no row of the tile has this step: its rows of the tape are zero
    for (int idx = tid; idx < PR * lh; idx += blockDim.x) {
      const int r = idx / (int)lh, c = idx % (int)lh, row = r0 + r;
      if (row >= B) continue;
      for (int q = 0; q < nr; ++q) {
        const long k = a.kb + row + (long)q * B;
        if (c < H) a.T1g[k * H + c] = a.T2g[k * H + c] = 0.0;
        a.T2in[k * lh + c] = a.T3in[k * lh + c] = 0.0;
      }
    }
    for (int idx = tid; idx < PR * l1; idx += blockDim.x) {
      const int r = idx / (int)l1, c = idx % (int)l1, row = r0 + r;
      if (row >= B) continue;
      for (int q = 0; q < nr; ++q) {
        const long k = a.kb + row + (long)q * B;
        a.T1in[k * l1 + c] = 0.0;
        if (c < din) a.T3g[k * din + c] = 0.0;
      }
    }
    return;
  }
  // gbar: kappa_z on primal rows, -kappa_l eps on tangent rows; the tape's
  // layer-1 inputs and layer-3 cotangents
  for (int idx = tid; idx < PR * d.nkd * 8; idx += blockDim.x) {
    const int r = idx / (d.nkd * 8), c = idx % (d.nkd * 8), row = r0 + r;
    const bool o = onr[r] != 0;
    const bool in = o && c < din;
    const double* ks =
        CL ? cl + ((a.s - 1) * PR + r) * D : a.kap_s + (long)row * D;
    const double kz = in ? ks[c] : 0.0;
    X[r * d.SX + c] = kz;
    if (c < din && row < B) {
      a.T1in[(a.kb + row) * l1 + c] = o ? a.Y[(long)row * D + c] : 0.0;
      a.T3g[(a.kb + row) * din + c] = kz;
    }
    if (CNF) {
      const double e = in ? a.eps[(long)row * D + c] : 0.0;
      const double g = in ? -ks[din] * e : 0.0;
      X[(PR + r) * d.SX + c] = g;
      if (c < din && row < B) {
        a.T1in[(a.kb + B + row) * l1 + c] = e;
        a.T3g[(a.kb + B + row) * din + c] = g;
      }
    }
  }
  for (int r = tid; r < PR; r += blockDim.x) {
    const int row = r0 + r;
    if (row >= B) continue;
    const long k = a.kb + row;
    a.T1in[k * l1 + din] = onr[r] ? a.bt[row] + a.c * a.bh[row] : 0.0;
    a.T1in[k * l1 + din + 1] = a.T2in[k * lh + H] = a.T3in[k * lh + H] = 1.0;
    if (CNF) {
      const long kt = k + B;
      a.T1in[kt * l1 + din] = a.T1in[kt * l1 + din + 1] = 0.0;
      a.T2in[kt * lh + H] = a.T3in[kt * lh + H] = 0.0;
    }
  }
  __syncthreads();

  // S2 = gbar W3^T, then S1 = G2 W2^T; epilogues form G2, G1
#pragma unroll
  for (int layer = 1; layer >= 0; --layer) {
    const double* W = layer == 1 ? a.WT : a.WT + (size_t)d.nkd * d.nnh * kFrag;
    double* dst = layer == 1 ? A0 : A1;
    double* Tin = layer == 1 ? a.T3in : a.T2in;
    double* Tg = layer == 1 ? a.T2g : a.T1g;
    for (int nb0 = wave * NT; nb0 < d.nnh; nb0 += kWV * NT) {
      double acc[MT][NT], keep[MT][NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int n = (nb0 + t) * 16 + col;
#pragma unroll
        for (int g = 0; g < MT; ++g) {
          const int r = (g < MP ? g : g - MP) * 4 + i4, row = r0 + r;
          acc[g][t] = 0.0;
          keep[g][t] =
              n < H && onr[r]
                  ? a.act_in[((long)(row + (g < MP ? 0 : B)) * 2 + layer) * H +
                             n]
                  : 0.0;
        }
      }
      if (layer == 1)
        gemm<MT, NT>(acc, X, d.SX, W, d.nkd, d.nnh, nb0, lane);
      else
        gemm<MT, NT>(acc, A0, d.SA, W, d.nkh, d.nnh, nb0, lane);
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        const int n = (nb0 + t) * 16 + col;
        if (nb0 + t >= d.nnh) continue;
#pragma unroll
        for (int g = 0; g < MP; ++g) {
          const int r = g * 4 + i4, row = r0 + r;
          const double av = keep[g][t], dv = 1.0 - av * av;
          double s = acc[g][t], gt = 0.0, dp = 0.0;
          if (CNF) {
            dp = keep[MP + g][t];
            gt = dv * acc[MP + g][t];
            s += -2.0 * av * dp * acc[MP + g][t];
            dst[(PR + r) * d.SA + n] = n < H ? gt : 0.0;
          }
          const double gv = dv * s;
          dst[r * d.SA + n] = n < H ? gv : 0.0;
          if (row < B && n < H) {
            const long k = a.kb + row;
            Tin[k * lh + n] = av;
            Tg[k * H + n] = gv;
            if (CNF) {
              Tin[(k + B) * lh + n] = dv * dp;
              Tg[(k + B) * H + n] = gt;
            }
          }
        }
      }
    }
    __syncthreads();
  }

  // mu = G1 W1^T (primal rows)
  {
    const double* W =
        a.WT + ((size_t)d.nkd * d.nnh + (size_t)d.nkh * d.nnh) * kFrag;
    for (int nb = wave; nb < d.nnd; nb += kWV) {
      const int n = nb * 16 + col;
      double acc[MP][1];
#pragma unroll
      for (int g = 0; g < MP; ++g) acc[g][0] = 0.0;
      gemm<MP, 1>(acc, A1, d.SA, W, d.nkh, d.nnd, nb, lane);
      if (n < din)
#pragma unroll
        for (int g = 0; g < MP; ++g) MU[(g * 4 + i4) * din + n] = acc[g][0];
    }
  }
  __syncthreads();
  for (int idx = tid; idx < PR * D; idx += blockDim.x) {
    const int r = idx / D, c = idx % D, row = r0 + r;
    if (!onr[r]) continue;
    const long o = (long)row * D + c;
    double mu = c < din ? MU[r * din + c] : 0.0;
    if (a.mu_out != nullptr) {
      a.mu_out[o] = mu;
      continue;
    }
    const double h = a.bh[row];
    if (a.s == 7) {
      mu = a.lam[o] + mu;  // Lambda
      a.lam[o] = mu;
    }
    double& ln = CL ? cl[(7 * PR + r) * D + c] : a.lamn[o];
    const double l = ln + mu;
    ln = l;
#pragma unroll
    for (int j = 0; j < 6; ++j)
      if (j < a.n) {
        double& kp = CL ? cl[(a.kidx[j] * PR + r) * D + c]
                        : a.kap[((long)a.kidx[j] * B + row) * D + c];
        kp += h * a.coef[j] * mu;
      }
    if (a.s == 1) a.lam[o] = l;
  }
}

// ---- tile shapes -------------------------------------------------------------

// Calls f(integral constants MT, NT, CNF) for the shape.
template <class F>
hipError_t with_shape(int B, int din, int H, bool cnf, F f) {
  const int mt = row_groups(B, din, H, cnf);
  const bool wide = dims(din, H).nnh > kWV;  // two column tiles a wavefront
#define BODE_F64_CASE(m, c)                                             \
  return wide ? f(std::integral_constant<int, m>{},                     \
                  std::integral_constant<int, 2>{},                     \
                  std::integral_constant<bool, c>{})                    \
              : f(std::integral_constant<int, m>{},                     \
                  std::integral_constant<int, 1>{},                     \
                  std::integral_constant<bool, c>{})
  if (cnf) {
    if (mt == 4) BODE_F64_CASE(4, true);
    BODE_F64_CASE(2, true);
  }
  if (mt == 4) BODE_F64_CASE(4, false);
  if (mt == 2) BODE_F64_CASE(2, false);
  BODE_F64_CASE(1, false);
#undef BODE_F64_CASE
}

// More than 64 KiB of LDS for a kernel is asked for once per launch site.
template <class K>
hipError_t allow_lds(K kernel, size_t bytes) {
  if (bytes <= 65536) return hipSuccess;
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel),
                             hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)bytes);
}

}  // namespace f64t
}  // namespace bode
