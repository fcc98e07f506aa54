// FP64 neural fields on the matrix cores: weight packing, the stage
// evaluations of a step and its adjoint stages (building blocks in
// f64_tile.hpp).
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "common.hpp"
#include "f64_mfma.hpp"
#include "f64_tile.hpp"

namespace bode {

namespace {

using namespace f64t;

// M = W (trans = 0) or W^T, K x N, into the fragment layout of f64_tile.hpp
// (W row-major with leading dimension ldw), zero beyond K and N.
struct Pack64 {
  double* dst;
  const double* W;
  int K, N, ldw, nk, nn, trans;
};

struct Pack64Jobs {
  Pack64 j[6];
};

__global__ void pack64_kernel(Pack64Jobs jobs) {
  const Pack64 j = jobs.j[blockIdx.y];
  const long total = (long)j.nk * j.nn * kFrag;
  for (long e = blockIdx.x * (long)blockDim.x + threadIdx.x; e < total;
       e += (long)gridDim.x * blockDim.x) {
    const int q = e & 1, l = (e >> 1) & 63;
    const long f = e / kFrag;
    const int k = int(f / j.nn) * 8 + (l >> 4) * 2 + q;
    const int n = int(f % j.nn) * 16 + (l & 15);
    j.dst[e] = k < j.K && n < j.N
                   ? j.W[j.trans ? (long)n * j.ldw + k : (long)k * j.ldw + n]
                   : 0.0;
  }
}

template <int MT, int NT, bool CNF, bool KL>
__global__ __launch_bounds__(64 * kWV) void field64_kernel(F64Steps v) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* smem = reinterpret_cast<double*>(smem_raw);
  double* kl = KL ? reinterpret_cast<double*>(smem_raw + v.kl_off) : nullptr;
  constexpr int PR = CNF ? 2 * MT : 4 * MT;
  for (int i = 0; i < v.n; ++i) {
    field_tile<MT, NT, CNF, KL>(v.st[i], blockIdx.x * PR, smem, kl);
    __syncthreads();
  }
}

template <int MT, int NT, bool CNF, bool CL>
__global__ __launch_bounds__(64 * kWV) void vjp64_kernel(F64VjpSteps v) {
  extern __shared__ __align__(16) unsigned char smem_raw[];
  double* smem = reinterpret_cast<double*>(smem_raw);
  double* cl = CL ? reinterpret_cast<double*>(smem_raw + v.cl_off) : nullptr;
  constexpr int PR = CNF ? 2 * MT : 4 * MT;
  if (v.dense.on) {
    vjp_dense_rows<PR, kWV, CL>(v.dense, v.st[0].kap, v.st[0].lamn, v.st[0].B,
                                v.st[0].D, cl);
    __syncthreads();
  }
  for (int i = 0; i < v.n; ++i) {
    vjp_tile<MT, NT, CNF, CL>(v.st[i], blockIdx.x * PR, smem, cl);
    __syncthreads();
  }
}

}  // namespace

bool f64_fits(int D, int din, int H, bool cnf) {
  (void)D;
  return tile_fits(din, H, cnf);
}

size_t f64_packed_elems(int din, int H) {
  const Dims d = dims(din, H);
  return ((size_t)d.nk1 * d.nnh + (size_t)d.nkh * d.nnh +
          (size_t)d.nkh * d.nnd) * kFrag;
}

size_t f64_packedT_elems(int din, int H) {
  const Dims d = dims(din, H);
  return ((size_t)d.nkd * d.nnh + (size_t)d.nkh * d.nnh +
          (size_t)d.nkh * d.nnd) * kFrag;
}

hipError_t f64_pack_weights(double* W, double* WT, int din, int H,
                            const double* W1, const double* W2,
                            const double* W3, hipStream_t s) {
  const Dims d = dims(din, H);
  const size_t f2 = (size_t)d.nk1 * d.nnh * kFrag;
  const size_t f3 = f2 + (size_t)d.nkh * d.nnh * kFrag;
  const size_t t2 = (size_t)d.nkd * d.nnh * kFrag;
  const size_t t1 = t2 + (size_t)d.nkh * d.nnh * kFrag;
  const Pack64Jobs j = {{{W, W1, din + 1, H, H, d.nk1, d.nnh, 0},
                         {W + f2, W2, H, H, H, d.nkh, d.nnh, 0},
                         {W + f3, W3, H, din, din, d.nkh, d.nnd, 0},
                         {WT, W3, din, H, din, d.nkd, d.nnh, 1},
                         {WT + t2, W2, H, H, H, d.nkh, d.nnh, 1},
                         {WT + t1, W1, H, din, H, d.nkh, d.nnd, 1}}};
  hipLaunchKernelGGL(pack64_kernel, dim3(128, WT != nullptr ? 6 : 3),
                     dim3(256), 0, s, j);
  return hipGetLastError();
}

hipError_t launch_field_f64(const F64Steps& v0, hipStream_t s) {
  if (v0.n < 1 || v0.n > 7) return hipErrorInvalidValue;
  const F64Args& a = v0.st[0];
  return with_shape(a.B, a.din, a.H, a.cnf, [&](auto mt, auto nt, auto cnf) {
    constexpr int MT = mt(), NT = nt(), PR = cnf() ? 2 * MT : 4 * MT;
    constexpr bool CNF = cnf();
    F64Steps v = v0;
    const LdsPlan p = lds_plan(MT, a.D, a.din, a.H, CNF, v.kl ? 7 : 0);
    v.kl_off = p.off;
    auto k = p.block ? field64_kernel<MT, NT, CNF, true>
                     : field64_kernel<MT, NT, CNF, false>;
    const hipError_t e = allow_lds(k, p.bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3((a.B + PR - 1) / PR), dim3(64 * kWV), p.bytes,
                       s, v);
    return hipGetLastError();
  });
}

hipError_t launch_vjp_f64(const F64VjpSteps& v0, hipStream_t s) {
  if (v0.n < 1 || v0.n > 7) return hipErrorInvalidValue;
  const F64VjpArgs& a = v0.st[0];
  return with_shape(a.B, a.din, a.H, a.cnf, [&](auto mt, auto nt, auto cnf) {
    constexpr int MT = mt(), NT = nt(), PR = cnf() ? 2 * MT : 4 * MT;
    constexpr bool CNF = cnf();
    F64VjpSteps v = v0;
    // the cotangent block in LDS where this launch also seeds it
    const LdsPlan p = lds_plan(MT, a.D, a.din, a.H, CNF, v.dense.on ? 8 : 0);
    v.cl_off = p.off;
    auto k = p.block ? vjp64_kernel<MT, NT, CNF, true>
                     : vjp64_kernel<MT, NT, CNF, false>;
    const hipError_t e = allow_lds(k, p.bytes);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3((a.B + PR - 1) / PR), dim3(64 * kWV), p.bytes,
                       s, v);
    return hipGetLastError();
  });
}

}  // namespace bode
