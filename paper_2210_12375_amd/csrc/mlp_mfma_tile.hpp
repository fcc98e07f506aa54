// Layout of the packed weights and the smallest building blocks of the
// neural-field kernels on the matrix cores of gfx950 (neural_tile.hpp).
//
// Weights are packed once per solve into 16x32 fragments of
// v_mfma_f32_16x16x32_bf16 (64 lanes x 8 elements contiguous per fragment),
// read straight from L2 by each wavefront.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "common.hpp"
#include "mlp_mfma.hpp"

namespace bode {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

namespace mtile {

__device__ __forceinline__ uint16_t f2bf(float x) {
  uint32_t u = __float_as_uint(x);
  if ((u & 0x7f800000u) == 0x7f800000u)  // inf / nan stay inf / nan
    return uint16_t((u >> 16) | ((u & 0xffffu) ? 0x40u : 0u));
  u += 0x7fffu + ((u >> 16) & 1u);  // round to nearest even
  return uint16_t(u >> 16);
}


struct Dims {
  int K1, nk1, nn1, nk2, nn2, nk3, nn3;
  size_t off2, off3;  // packed offsets (elements) of layers 2 and 3
};

__host__ __device__ inline Dims dims(int din, int H) {
  Dims d;
  d.K1 = (din + 31) / 32 * 32;
  d.nk1 = d.K1 / 32;
  d.nn1 = H / 16;
  d.nk2 = H / 32;
  d.nn2 = H / 16;
  d.nk3 = H / 32;
  d.nn3 = din / 16;
  d.off2 = (size_t)d.nk1 * d.nn1 * 512;
  d.off3 = d.off2 + (size_t)d.nk2 * d.nn2 * 512;
  return d;
}

// Packed layout: fragment f = kb * nn + nb, lane l, element i holds
// M[kb*32 + (l/16)*8 + i][nb*16 + l%16] (zero beyond K rows), where M is a
// layer W or its transpose.
//
// Transposed layers: W3^T [din x H], W2^T [H x H], W1^T [H x din].
struct DimsT {
  int nk3, nn3, nk2, nn2, nk1, nn1;
  size_t off2, off1, total;
};

__host__ __device__ inline DimsT dims_t(int din, int H) {
  DimsT d;
  d.nk3 = (din + 31) / 32;
  d.nn3 = H / 16;
  d.nk2 = H / 32;
  d.nn2 = H / 16;
  d.nk1 = H / 32;
  d.nn1 = din / 16;
  d.off2 = (size_t)d.nk3 * d.nn3 * 512;
  d.off1 = d.off2 + (size_t)d.nk2 * d.nn2 * 512;
  d.total = d.off1 + (size_t)d.nk1 * d.nn1 * 512;
  return d;
}

// FP32 mode cuts (rather than rounds) weights and stage inputs from here on
// into BF16 terms (put4 of neural_tile.hpp gives the reason).
constexpr float kBigValue = 512.f;

__device__ __forceinline__ bf16x8 lds8(const uint16_t* p) {
  return *reinterpret_cast<const bf16x8*>(p);
}

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// tanh x = 1 - 2 / (1 + e^{2x}), e^{2x} = 2^(2 x log2 e) by the hardware
// exp2 and reciprocal: absolute error about 1e-7 (FP32's own rounding of an
// activation), and the limits come out exactly (e^{2x} = inf gives 1, 0
// gives -1).
__device__ __forceinline__ float fast_tanh(float x) {
  const float e = __builtin_amdgcn_exp2f(x * 2.8853900817779268f);
  return 1.f - 2.f * __builtin_amdgcn_rcpf(1.f + e);
}

}  // namespace mtile
}  // namespace bode
