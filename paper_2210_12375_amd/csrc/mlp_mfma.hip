// Neural right-hand sides on the matrix cores of gfx950: weight packing (the
// layout in mlp_mfma_tile.hpp).
#include <hip/hip_runtime.h>

#include <cstdint>

#include "../../include/batchode.h"
#include "common.hpp"
#include "mlp_mfma.hpp"
#include "mlp_mfma_tile.hpp"

namespace bode {

namespace {

using namespace mtile;

// One weight matrix to pack: M = W (trans = 0) or W^T, K x N, into the
// fragment layout of mtile (W row-major with leading dimension ldw), zero
// beyond K and N.
struct PackJob {
  uint16_t* dst;
  const float* W;
  int K, N, ldw, nk, nn, trans;
  size_t plane;  // elements between the BF16 terms' planes
};

struct PackJobs {
  PackJob j[6];
  int n, planes;
  float* f;  // b1, W1's time row, b2 (padded to Hp), b3 (padded)
  const float *W1, *b1, *b2, *b3;
  int din, H, Hp, dp;
};

// A thread packs one lane's eight elements of a fragment (one 16-byte store
// per plane); the last grid row does the vector block.  Terms are rounded to
// nearest (from kBigValue on cut, infinities cut from the largest float) and
// each residual is exact; one plane is the BF16 weight itself.
__global__ void pack_weights_kernel(PackJobs p) {
  const int tid = blockIdx.x * blockDim.x + threadIdx.x;
  const int nthr = gridDim.x * blockDim.x;
  if ((int)blockIdx.y < p.n) {
    const PackJob j = p.j[blockIdx.y];
    const int total = j.nk * j.nn * 64;
    for (int e = tid; e < total; e += nthr) {
      const int l = e & 63, f = e >> 6;
      const int k0 = f / j.nn * 32 + (l >> 4) * 8;
      const int n = f % j.nn * 16 + (l & 15);
      float v[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const int k = k0 + i;
        v[i] = k < j.K && n < j.N
                   ? j.W[j.trans ? (long)n * j.ldw + k : (long)k * j.ldw + n]
                   : 0.f;
      }
      uint32_t big = 0;
      if (p.planes > 1)
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          big |= uint32_t(!(fabsf(v[i]) < kBigValue)) << i;
          if (fabsf(v[i]) > FLT_MAX) v[i] = copysignf(FLT_MAX, v[i]);
        }
      for (int q = 0; q < p.planes; ++q) {
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 8; i += 2) {
          uint16_t h[2];
#pragma unroll
          for (int u = 0; u < 2; ++u) {
            float& x = v[i + u];
            h[u] = big >> (i + u) & 1 ? uint16_t(__float_as_uint(x) >> 16)
                                      : f2bf(x);
            x -= __uint_as_float((uint32_t)h[u] << 16);
          }
          w[i / 2] = h[0] | ((uint32_t)h[1] << 16);
        }
        *reinterpret_cast<uint4*>(j.dst + q * j.plane + (size_t)e * 8) =
            make_uint4(w[0], w[1], w[2], w[3]);
      }
    }
    return;
  }
  for (int c = tid; c < 3 * p.Hp + p.dp; c += nthr) {
    const int b = c / p.Hp < 3 ? c / p.Hp : 3, i = c - b * p.Hp;
    float v = 0.f;
    if (i < (b < 3 ? p.H : p.din))
      v = b == 0   ? p.b1[i]
          : b == 1 ? p.W1[(long)p.din * p.H + i]  // time row of W1
          : b == 2 ? p.b2[i]
                   : p.b3[i];
    p.f[c] = v;
  }
}

}  // namespace

size_t mfma_plane_elems(int din, int H) {
  const Dims d = dims(mfma_pad_din(din), mfma_pad_h(H));
  return d.off3 + (size_t)d.nk3 * d.nn3 * 512;
}

size_t mfma_planeT_elems(int din, int H) {
  return dims_t(mfma_pad_din(din), mfma_pad_h(H)).total;
}

size_t mfma_packed_bytes(int din, int H, int f32) {
  return mfma_plane_elems(din, H) * (f32 ? 6 : 2);
}

size_t mfma_packedT_bytes(int din, int H, int f32) {
  return mfma_planeT_elems(din, H) * (f32 ? 6 : 2);
}

size_t mfma_fvec_elems(int din, int H) {
  return 3 * (size_t)mfma_pad_h(H) + mfma_pad_din(din);
}

std::string mfma_supported(int din, int H) {
  if (din < 16 || din % 16 != 0 || din > 256)
    return "matrix-core fields need a state width that is a multiple of 16, "
           "<= 256";
  if (H != 64 && H != 128 && H != 256 && H != 512)
    return "matrix-core fields are built for hidden widths 64, 128, 256, 512";
  return "";
}

bool neural_fused(int precision, int din, int H) {
  return precision == BODE_BF16 ||
         (precision == BODE_FP32 && din <= 256 && H <= 512);
}

hipError_t mfma_pack_weights(const MfmaWeights& w, int din, int H,
                             const float* W1, const float* b1, const float* W2,
                             const float* b2, const float* W3, const float* b3,
                             hipStream_t s) {
  PackJobs p{};
  p.planes = w.f32 ? 3 : 1;
  p.f = w.fvec;
  p.W1 = W1;
  p.b1 = b1;
  p.b2 = b2;
  p.b3 = b3;
  p.din = din;
  p.H = H;
  p.dp = mfma_pad_din(din);
  p.Hp = mfma_pad_h(H);
  const Dims d = dims(p.dp, p.Hp);
  const DimsT t = dims_t(p.dp, p.Hp);
  uint16_t *a = static_cast<uint16_t*>(w.packed),
           *b = static_cast<uint16_t*>(w.packedT);
  const size_t pl = mfma_plane_elems(din, H), plt = mfma_planeT_elems(din, H);
  const PackJob j[6] = {{a, W1, din, H, H, d.nk1, d.nn1, 0, pl},
                        {a + d.off2, W2, H, H, H, d.nk2, d.nn2, 0, pl},
                        {a + d.off3, W3, H, din, din, d.nk3, d.nn3, 0, pl},
                        {b, W3, din, H, din, t.nk3, t.nn3, 1, plt},
                        {b + t.off2, W2, H, H, H, t.nk2, t.nn2, 1, plt},
                        {b + t.off1, W1, H, din, H, t.nk1, t.nn1, 1, plt}};
  p.n = b != nullptr ? 6 : 3;
  for (int q = 0; q < p.n; ++q) p.j[q] = j[q];
  const int blocks = (d.nk2 * d.nn2 * 64 + 255) / 256;
  hipLaunchKernelGGL(pack_weights_kernel, dim3(blocks, p.n + 1), dim3(256), 0,
                     s, p);
  return hipGetLastError();
}

MfmaArgs mfma_args(int B, int D, int din, int H, int cnf, const int32_t* status,
                   const float* y, const float* K, float* Y7, const float* hs,
                   const double* t, const float* eps, const MfmaWeights& w) {
  MfmaArgs a{};
  a.B = B;
  a.D = D;
  a.din = din;
  a.H = H;
  a.cnf = cnf;
  a.status = status;
  a.y = y;
  a.K = K;
  a.Y7 = Y7;
  a.hs = hs;
  a.t = t;
  a.eps = eps;
  a.w = w;
  return a;
}

}  // namespace bode
