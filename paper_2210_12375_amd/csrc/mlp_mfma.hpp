// BF16 MFMA evaluation of the neural fields (MLP and CNF), gfx950.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <string>

#include "vjp_dense.hpp"

namespace bode {

// Packed weights: every layer as 16x32 MFMA fragments (64 lanes x 8 BF16
// elements, contiguous per fragment; FP32 mode, f32 != 0: three planes of
// them), plus FP32 vectors b1, w1t (the time row of W1), b2, b3.
struct MfmaWeights {
  void* packed = nullptr;
  float* fvec = nullptr;
  // Transposed layers for the vector-Jacobian products of the adjoint:
  // W3^T, W2^T and W1^T without its time row (null when not needed).
  void* packedT = nullptr;
  int f32 = 0;
  // BF16 mode: 1 rounds every activation to one BF16 term (plain BF16);
  // 0 splits it into three (hi + mid + lo, FP32's precision).
  int plain = 0;
};

// FP32 mode's weights are three BF16 planes (their exact split) of the
// layers padded to widths the kernels are built for: state features to 16,
// hidden units to 64, 128, 256 or 512 (padding is zero; BF16 mode accepts
// only shapes that need none).
inline int mfma_pad_din(int din) { return (din + 15) / 16 * 16; }
inline int mfma_pad_h(int H) {
  return H <= 64 ? 64 : H <= 128 ? 128 : H <= 256 ? 256 : 512;
}
size_t mfma_packed_bytes(int din, int H, int f32);
size_t mfma_packedT_bytes(int din, int H, int f32);
size_t mfma_plane_elems(int din, int H);   // elements of a forward plane
size_t mfma_planeT_elems(int din, int H);  // of a transposed one
size_t mfma_fvec_elems(int din, int H);
std::string mfma_supported(int din, int H);
// Whether a precision (BODE_*) runs this shape on the matrix-core kernels:
// BF16 always; FP32 as split products (neural_tile.hpp) wherever the packed
// widths hold the shape, at any width in between (padding a 50-wide layer to
// 64 costs nothing beside the FMA kernel it replaces: 11.7 -> 0.78 ms).
bool neural_fused(int precision, int din, int H);
// Whether its kernels are built for one and for two row tiles a workgroup:
// eight wavefronts, none of which has two tiles of the output layer, and in
// BF16 with the weights resident below width 512 (fwd_op in neural_fwd.inc).
inline bool row_tile_choice(bool f32, int din, int H) {
  const int h = mfma_pad_h(H);
  return h > 64 && mfma_pad_din(din) <= (f32 || h == 512 ? 128 : 64);
}

hipError_t mfma_pack_weights(const MfmaWeights& w, int din, int H,
                             const float* W1, const float* b1, const float* W2,
                             const float* b2, const float* W3, const float* b3,
                             hipStream_t s);

struct MfmaArgs {
  int B, D, din, H, cnf;
  const int32_t* status;
  const float* y;
  const float* K;  // [7, B, D]
  float* Y7;
  const float* hs;
  const double* t;
  const float* eps;
  MfmaWeights w;
  int n;
  int kidx[6];
  float coef[6];
  double c;
  int write_y7;
  float* out;
  // If not null, the hidden layers' values of every row are stored here for
  // a later vector-Jacobian product: [Bs][2][H] (Bs = B, or 2B for the CNF
  // whose tangent rows follow), layer 1 then layer 2 of each row; the
  // activation on primal rows, the pre-activation tangent on tangent rows.
  float* act_out;
  // 16-row tiles per workgroup: 8 asks for one, 4 for two (0: the default)
  int waves;
};

MfmaArgs mfma_args(int B, int D, int din, int H, int cnf, const int32_t* status,
                   const float* y, const float* K, float* Y7, const float* hs,
                   const double* t, const float* eps, const MfmaWeights& w);

}  // namespace bode
