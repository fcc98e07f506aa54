// The neural field of one row tile on the matrix cores of gfx950, with the
// stage arithmetic around it held in registers: the building block of the
// forward kernels (neural_fwd.inc).
//
// A workgroup owns RT = 16 MT rows (MLP: instances; CNF: instances and their
// tangent rows, 8 + 8 in one 16-row tile or, MT = 2, a tile of each).  The
// products run transposed, C^T = W^T A^T: the weights are the 16-row operand
// and the instances the 16 columns of v_mfma_f32_16x16x32_bf16, so a lane
// ends up with four consecutive features of one instance (instance l % 16,
// features 4 (l / 16) .. + 3 of a 16-feature tile).  Activations are split
// into BF16 terms and stored to LDS four at a time (one 8-byte store per
// term), and the state-sized vectors (y, the seven stages, the probe) stay
// in the registers of the lanes that own those elements for a whole solve:
// forming a stage input, the error estimate and the dense output touches no
// memory.
//
// Weights are the same packed 16x32 fragments as the adjoint kernels'.
// RES: all three layers stay in registers for the whole launch (width 256
// and up to 64 state features in BF16: 24 fragments, 96 registers in each of
// 8 wavefronts), so no evaluation reads a weight; otherwise they stream from
// L2 through a ring of k blocks requested one phase ahead.
// Measured against a field kernel that read its weights from L2 and its
// stages from LDS for every evaluation: solve of 4096 instances of
// 65->256->256->64 309 -> 177 us, of the 8192-instance CNF 17->512->512->16
// 2.55 -> 1.33 ms.
// The output layer's k blocks are split over the wavefronts its few feature
// tiles would leave idle (partials meet in LDS, summed in a fixed order).
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>

#include "common.hpp"
#include "mlp_mfma.hpp"
#include "mlp_mfma_tile.hpp"
#include "tanh.hpp"

namespace bode {
namespace ntile {

using mtile::fast_tanh;
using mtile::kBigValue;

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// Operand policies: BF16 terms per activation and per weight, and the
// products issued (weight term, activation term), smallest first.
struct Bf3 {
  static constexpr bool kTwo = false;
  static constexpr int kA = 3, kW = 1, kN = 3;
  static constexpr int kTerm[kN][2] = {{0, 2}, {0, 1}, {0, 0}};
  __device__ static __forceinline__ float tanh(float x) { return fast_tanh(x); }
};
struct Bf1 {
  static constexpr bool kTwo = false;
  static constexpr int kA = 1, kW = 1, kN = 1;
  static constexpr int kTerm[kN][2] = {{0, 0}};
  __device__ static __forceinline__ float tanh(float x) { return fast_tanh(x); }
};

// FP32 mode: weights and activations both as three terms.  Of the nine
// products the six largest are issued; terms are rounded to nearest, so the
// three dropped are at most about 2^-26 of a product together, below the
// FP32 accumulation's own rounding.  v_mfma_f32_16x16x4_f32 takes 16 cycles
// per 1024 products of a tile, six BF16 products of 8 k each 3; measured
// against it (40,000 instances of 65->256->256->64) 4.57 -> 2.94 ms, and
// against plain FMA where the widths are no multiples of 16 (300 instances
// of 7->50->50->6 with their adjoint) 11.7 -> 0.78 ms.  Relative l2 errors
// beside those of the kernels replaced, at three regular and five padded
// widths (50 to 256 units, 200 to 1200 instances, 8 draws), against 64 bits on
// the same steps, in 2^-24: state gradients 2.5-3.0 -> 2.5-2.6 (padded 2.5-2.9
// -> 2.5-2.6), parameter gradients, worst layer, 4.5-4.7 -> 3.0-3.3 (3.6-4.9 ->
// 2.7-3.8); of 16 shapes' final states against 64-bit solves, 0.37 to 0.98 of
// the former error.
struct Bf6 {
  // the five small products accumulate apart from hi x hi, so a sum over k is
  // rounded at its own size once per 32 k, not six times (in one accumulator
  // the bias gradients, sums of one sign, came out 1.5 times further off)
  static constexpr bool kTwo = true;
  static constexpr int kA = 3, kW = 3, kN = 6;
  static constexpr int kTerm[kN][2] = {{0, 2}, {2, 0}, {1, 1},
                                       {0, 1}, {1, 0}, {0, 0}};
  __device__ static __forceinline__ float tanh(float x) {
    return tanh32<HwMath>(x);
  }
};

__device__ __forceinline__ uint32_t pack2(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(
                                          f32x2{a, b}, bf16x2));
}
__device__ __forceinline__ float lo_f(uint32_t u) {
  return __uint_as_float(u << 16);
}
__device__ __forceinline__ float hi_f(uint32_t u) {
  return __uint_as_float(u & 0xffff0000u);
}

// Four values as BF16 terms that sum to them, one 8-byte store per term,
// rounded to nearest; each residual is exact.
//
// kInput (stage inputs, any float): a product that overflows has to come out as
// the infinity of its sign, as a plain FP32 product would, so that the unit
// saturates; terms of both signs would give NaN.  In the BF16 mode all values
// are cut instead of rounded (exact as well, and every term has the value's
// sign).  FP32 mode, whose cut terms would drop more of a product, cuts values
// from 512 on, as the packed weights are (a product whose small part overflows
// has both factors beyond it), and bounds them by 2^119 (every unit with a
// weight above 2^-115 is saturated there, and what 256 of them drop stays
// below 2^128); an infinity is then no special case.
// kCotangent (any float, not to be bounded): cut where rounding could overflow.
enum PutKind { kPlain, kInput, kCotangent };
template <class Op, PutKind KIND>
__device__ __forceinline__ void put4(uint16_t* p, int plane, f32x4 v) {
  // (the residuals are of the rounded value: no fusing with its product)
#pragma clang fp contract(off)
  constexpr int kA = Op::kA;
  constexpr bool kCut = KIND != kPlain && !Op::kTwo && kA > 1;
  constexpr float kBig = KIND == kInput && Op::kTwo ? kBigValue : 0x1p127f;
  if constexpr (kCut) {
#pragma unroll
    for (int k = 0; k < kA; ++k) {
      uint32_t w[2];
#pragma unroll
      for (int i = 0; i < 4; i += 2) {
        w[i / 2] = __builtin_amdgcn_perm(
            __float_as_uint(v[i + 1]), __float_as_uint(v[i]), 0x07060302u);
        v[i] -= lo_f(w[i / 2]);
        v[i + 1] -= hi_f(w[i / 2]);
      }
      *reinterpret_cast<u32x2*>(p + k * plane) = u32x2{w[0], w[1]};
    }
    return;
  }
  const f32x4 u = v;
  uint32_t a = pack2(v[0], v[1]), b = pack2(v[2], v[3]);
  *reinterpret_cast<u32x2*>(p) = u32x2{a, b};
#pragma unroll
  for (int k = 1; k < kA; ++k) {
    v[0] -= lo_f(a);
    v[1] -= hi_f(a);
    v[2] -= lo_f(b);
    v[3] -= hi_f(b);
    a = pack2(v[0], v[1]);
    b = pack2(v[2], v[3]);
    *reinterpret_cast<u32x2*>(p + k * plane) = u32x2{a, b};
  }
  if constexpr (KIND != kPlain) {
    // (written over afterwards: 2916 us against 2995 to 3050 with the selects
    // or the two paths ahead of the stores, 40,000 FP32 instances)
    const bool big = !(fmaxf(fmaxf(fabsf(u[0]), fabsf(u[1])),
                             fmaxf(fabsf(u[2]), fabsf(u[3]))) < kBig);
    if (__builtin_expect(__any(big), 0)) {
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float x = u[i];
        if (!(fabsf(x) < kBig)) {
          if (KIND == kInput && Op::kTwo && fabsf(x) > 0x1p119f)
            x = copysignf(0x1p119f, x);
#pragma unroll
          for (int k = 0; k < kA; ++k) {
            p[k * plane + i] = uint16_t(__float_as_uint(x) >> 16);
            x -= __uint_as_float(__float_as_uint(x) & 0xffff0000u);
          }
        }
      }
    }
  }
}

// The value of the lane 8 places away within its row of 16 lanes.
__device__ __forceinline__ float xor8(float v) {
  return __uint_as_float(__builtin_amdgcn_update_dpp(
      0, __float_as_uint(v), 0x128, 0xf, 0xf, true));  // row_ror:8
}

// Shape constants.  NTW feature tiles of the hidden layers per wavefront,
// NO output tiles per wavefront.
template <class Op_, int NTW_, int WV_, int MT_, bool CNF_, int NO_, bool RES_>
struct Shape {
  typedef Op_ Op;
  static constexpr int NTW = NTW_, WV = WV_, MT = MT_, NO = NO_;
  static constexpr bool CNF = CNF_, RES = RES_;
  static constexpr int H = NTW * 16 * WV, NKH = H / 32, RT = 16 * MT;
  static constexpr int OM = CNF ? 1 : MT;  // row tiles that own state
  static constexpr int PR = CNF ? 8 * MT : RT;  // instances
  static constexpr int SA = H + 8, PA = RT * SA;
  // both hidden layers' outputs in LDS while two buffers are small
  static constexpr bool DB = 2 * Op::kA * PA * 2 <= 56 * 1024;
  // weight k blocks in flight: about 32 registers of ring, 2 to 4 blocks
  static constexpr int P =
      NTW * Op::kW >= 12 ? 1 : NTW * Op::kW >= 4 ? 2 : 4;
  // LDS offsets known at compile time: biases, layer buffers
  static constexpr int oFv = 0, oA = 4 * (3 * H + 256);
  static constexpr int oT = oA + 2 * Op::kA * PA * (DB ? 2 : 1);
  static constexpr int oX = oT + 4 * 32;
};

// Two wavefronts per SIMD: 256 registers, all ordinary ones (with more, the
// compiler keeps sums in accumulation registers and copies them out).
#define BODE_TILE_BOUNDS(S)             \
  __launch_bounds__(64 * S::WV)         \
      __attribute__((amdgpu_waves_per_eu(2)))

// The network, from the host.
struct Net {
  int B, D, din, dr, H;  // din, dr: state features, padded and not; H: the
                         // hidden width, not padded (act_out's rows)
  int nk1, nn3, ks;  // k blocks of layer 1, output tiles, k split
  int off2, off3, plane;  // in fragments
  const uint16_t* w;
  unsigned wbytes;
  const float* fvec;
};

__host__ __device__ inline int k_split(int nn3, int wv, int nkh) {
  int k = 1;
  while (nn3 * 2 * k <= wv && 2 * k <= nkh) k *= 2;
  return k;
}

// Byte offsets of a tile's LDS.
struct Lds {
  int red, ldot, end;
  int sx, px;
};

template <class S>
__host__ __device__ inline Lds lds_map(int din) {
  const int nk1 = (din + 31) / 32, nn3 = din / 16;
  const int ks = k_split(nn3, S::WV, S::NKH);
  Lds l;
  l.sx = nk1 * 32 + 8;
  l.px = S::RT * l.sx;
  l.red = S::oX + 2 * S::Op::kA * l.px;
  l.ldot = l.red + (ks - 1) * nn3 * S::MT * 1024;
  l.end = l.ldot + (S::CNF ? 4 * nn3 * S::PR : 0);
  l.end = (l.end + 15) / 16 * 16;
  return l;
}


// One k block's weight fragments of NT feature tiles.
template <class S, int NT>
struct Frag {
  bf16x8 f[NT][S::Op::kW];
};

// A kernel's by-value argument, through a pointer the compiler cannot see
// through: its fields are loaded (scalar, cached) where they are used instead
// of being held in scalar registers across the whole kernel, where they
// spilled.
template <class T>
using Karg = const __attribute__((address_space(4))) T*;
template <class T>
__device__ __forceinline__ Karg<T> kernarg() {
  auto p = (Karg<T>)__builtin_amdgcn_kernarg_segment_ptr();
  asm volatile("" : "+s"(p));
  return p;
}

// A uniform value the compiler recomputes from (offsets derived from it are
// not hoisted out of the stage loop into spilled scalars).
__device__ __forceinline__ int opaque(int x) {
  asm volatile("" : "+s"(x));
  return x;
}

// Packed layers as a buffer: a fragment's address is the uniform offset of
// its 1 KiB (a scalar) plus the lane's 16 bytes, so no lane holds 64-bit
// addresses (as pointers the compiler kept one per fragment of an unrolled
// layer and spilled them).
struct WBuf {
  __amdgpu_buffer_rsrc_t r;
  __device__ __forceinline__ WBuf(const uint16_t* w, unsigned bytes)
      : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(w), 0,
                                            (int)bytes, 0x00027000)) {}
  __device__ __forceinline__ bf16x8 frag(int f, int lane) const {
    return __builtin_bit_cast(
        bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, lane * 16, f * 1024,
                                                      0));
  }
};

// Fragments nb0 .. nb0 + NT - 1 of k block kb of the layer at fragment f0
// (nn column tiles a k block, `plane` fragments between the terms).
template <class S, int NT>
__device__ __forceinline__ void load_frag(Frag<S, NT>& d, const WBuf& W,
                                          int f0, int plane, int kb, int nn,
                                          int nb0, int lane) {
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int p = 0; p < S::Op::kW; ++p)
      d.f[t][p] = W.frag(f0 + p * plane + kb * nn + nb0 + t, lane);
}

// Accumulators of NT feature tiles (Op::kTwo: the small products apart).
template <class S, int NT>
struct Acc {
  f32x4 v[S::MT][NT], lo[S::Op::kTwo ? S::MT : 1][S::Op::kTwo ? NT : 1];
  __device__ __forceinline__ Acc() {
#pragma unroll
    for (int m = 0; m < S::MT; ++m)
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        v[m][t] = f32x4{0.f, 0.f, 0.f, 0.f};
        if constexpr (S::Op::kTwo) lo[m][t] = v[m][t];
      }
  }
  // The sums for ordinary instructions.  A matrix product's result may be
  // read by them only some wait states after its issue; the compiler counts
  // those inside a block, but was seen to miss them where a branch leads
  // straight from the last product to the first read (stale sums in the
  // wavefronts that skip the output layer's loads), so they are spent here:
  // the empty statements tie every accumulator to its place.
  __device__ __forceinline__ void finish() {
    tie();
    asm volatile("s_nop 11");
    tie();
    if constexpr (S::Op::kTwo)
#pragma unroll
      for (int m = 0; m < S::MT; ++m)
#pragma unroll
        for (int t = 0; t < NT; ++t) v[m][t] += lo[m][t];
  }
  __device__ __forceinline__ void tie() {
#pragma unroll
    for (int m = 0; m < S::MT; ++m)
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        asm volatile("" : "+v"(v[m][t]));
        if constexpr (S::Op::kTwo) asm volatile("" : "+v"(lo[m][t]));
      }
  }
};

// C^T[MT][NT] += W^T block x A^T block (k block kb of the rows in LDS at A).
template <class S, int NT>
__device__ __forceinline__ void products(Acc<S, NT>& acc,
                                         const Frag<S, NT>& w,
                                         const uint16_t* A, int plane,
                                         int stride, int kb, int lane) {
  typedef typename S::Op Op;
  bf16x8 b[S::MT][Op::kA];
#pragma unroll
  for (int m = 0; m < S::MT; ++m)
#pragma unroll
    for (int p = 0; p < Op::kA; ++p)
      b[m][p] = mtile::lds8(A + p * plane + (m * 16 + (lane & 15)) * stride +
                            kb * 32 + (lane >> 4) * 8);
#pragma unroll
  for (int q = 0; q < Op::kN; ++q)
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int m = 0; m < S::MT; ++m) {
        f32x4* c = &acc.v[m][t];
        if constexpr (Op::kTwo)
          if (q + 1 < Op::kN) c = &acc.lo[m][t];
        *c = mtile::mfma(w.f[t][Op::kTerm[q][0]], b[m][Op::kTerm[q][1]], *c);
      }
}

// Weight stream of one layer: k blocks k0 .. k0 + nk - 1, P in flight.
template <class S, int NT>
struct Stream {
  Frag<S, NT> r[S::P];
  __device__ __forceinline__ void start(const WBuf& W, int f0, int plane,
                                        int k0, int nk, int nn, int nb0,
                                        int lane) {
    f0 = opaque(f0);
    plane = opaque(plane);
#pragma unroll
    for (int p = 0; p < S::P; ++p)
      if (p < nk) load_frag<S, NT>(r[p], W, f0, plane, k0 + p, nn, nb0, lane);
    __builtin_amdgcn_sched_barrier(0);
  }
  __device__ __forceinline__ void run(Acc<S, NT>& acc, const WBuf& W,
                                      int f0, int plane, int k0, int nk,
                                      int nn, int nb0, const uint16_t* A,
                                      int aplane, int stride, int lane) {
    f0 = opaque(f0);
    plane = opaque(plane);
    for (int i = 0; i < nk; i += S::P) {
#pragma unroll
      for (int p = 0; p < S::P; ++p) {
        if (i + p >= nk) break;
        products<S, NT>(acc, r[p], A, aplane, stride, k0 + i + p, lane);
        const int nx = i + p + S::P;
        if (nx < nk)
          load_frag<S, NT>(r[p], W, f0, plane, k0 + nx, nn, nb0, lane);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
  }
};

// The weights of a launch: resident, or the streams' rings.
template <class S, bool RES = S::RES>
struct Weights {
  Stream<S, S::NTW> s1, s2;
  Stream<S, 1> s3[S::NO];
};
template <class S>
struct Weights<S, true> {
  Frag<S, S::NTW> w1[2], w2[S::NKH];
  Frag<S, 1> w3[S::NKH / 2];
};

template <class S>
struct Tile {
  typedef typename S::Op Op;
  typedef f32x4 Vec[S::OM][S::NO];  // this lane's elements of a state vector
  const Net& n;
  Lds l;
  unsigned char* sm;
  int tid, lane, wave, c, q;  // c: column (row of the tile), q: feature group
  int nb3, kh, k0, nk3;       // output layer: tile, k split, k blocks
  bool owner;                 // this wavefront owns state elements
  WBuf wb;
  Weights<S> w;

  __device__ __forceinline__ uint16_t* X() const {
    return reinterpret_cast<uint16_t*>(sm + S::oX);
  }
  __device__ __forceinline__ uint16_t* A(int i) const {
    return reinterpret_cast<uint16_t*>(sm + S::oA) +
           (S::DB ? i * Op::kA * S::PA : 0);
  }
  __device__ __forceinline__ f32x4* red() const {
    return reinterpret_cast<f32x4*>(sm + l.red);
  }
  __device__ __forceinline__ float* ldot() const {
    return reinterpret_cast<float*>(sm + l.ldot);
  }
  __device__ __forceinline__ float* tcol() const {
    return reinterpret_cast<float*>(sm + S::oT);
  }
  __device__ __forceinline__ float* fv() const {
    return reinterpret_cast<float*>(sm + S::oFv);
  }
  // output tile and its first feature for owned tile o; whether it exists
  __device__ __forceinline__ int nb_of(int o) const {
    return S::NO == 1 ? nb3 : wave + o * S::WV;
  }
  __device__ __forceinline__ int f0(int o) const {
    return nb_of(o) * 16 + q * 4;
  }
  __device__ __forceinline__ bool has(int o) const {
    return owner && nb_of(o) < n.nn3;
  }

  __device__ __forceinline__ Tile(const Net& net, unsigned char* smem)
      : n(net), l(lds_map<S>(net.din)), sm(smem), wb(net.w, net.wbytes) {
    tid = threadIdx.x;
    lane = tid & 63;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    c = lane & 15;
    q = lane >> 4;
    if (S::NO == 1) {
      nb3 = wave % n.nn3;
      kh = wave / n.nn3;
      owner = kh == 0;
      nk3 = S::NKH / n.ks;
      k0 = kh * nk3;
    } else {
      nb3 = wave;
      kh = 0;
      owner = wave < n.nn3;
      nk3 = S::NKH;
      k0 = 0;
    }
    if (n.fvec != nullptr)
      for (int i = tid; i < 3 * S::H + n.din; i += 64 * S::WV)
        fv()[i] = n.fvec[i];
    if constexpr (S::RES) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb)
        load_frag<S, S::NTW>(w.w1[kb], wb, 0, n.plane, kb < n.nk1 ? kb : 0,
                             S::H / 16, wave * S::NTW, lane);
#pragma unroll
      for (int kb = 0; kb < S::NKH; ++kb)
        load_frag<S, S::NTW>(w.w2[kb], wb, n.off2, n.plane, kb, S::H / 16,
                             wave * S::NTW, lane);
#pragma unroll
      for (int kb = 0; kb < S::NKH / 2; ++kb)
        load_frag<S, 1>(w.w3[kb], wb, n.off3, n.plane,
                        kh < n.ks && kb < nk3 ? k0 + kb : 0, n.nn3, nb3, lane);
    } else {
      start1();
    }
  }

  __device__ __forceinline__ void start1() {
    if constexpr (!S::RES)
      w.s1.start(wb, 0, n.plane, 0, n.nk1, S::H / 16, wave * S::NTW, lane);
  }

  // Constant parts of the layer-1 input: zero columns beyond the state, and
  // for the CNF the probe on the tangent rows (ep: this lane's elements).
  __device__ __forceinline__ void begin(const Vec& ep) {
    const int w1 = n.nk1 * 32 - n.din;
    for (int i = tid; i < S::RT * w1; i += 64 * S::WV)
#pragma unroll
      for (int p = 0; p < Op::kA; ++p)
        X()[p * l.px + (i / w1) * l.sx + n.din + i % w1] = 0;
    if (S::CNF) {
#pragma unroll
      for (int o = 0; o < S::NO; ++o)
        if (has(o) && (S::MT == 2 || c < 8))
          put4<Op, kPlain>(X() + (c + S::PR) * l.sx + f0(o), l.px,
                              ep[0][o]);
    }
  }

  // The stage input (or a stage's cotangent) into LDS.
  template <PutKind KIND = kInput>
  __device__ __forceinline__ void put_input(const Vec& Y) {
#pragma unroll
    for (int o = 0; o < S::NO; ++o)
#pragma unroll
      for (int m = 0; m < S::OM; ++m)
        if (has(o) && (!S::CNF || S::MT == 2 || c < 8))
          put4<Op, KIND>(X() + (m * 16 + c) * l.sx + f0(o), l.px,
                             Y[m][o]);
  }

  // The products of hidden layer LAYER (0 or 1) from buffer `in`, then
  // epi(acc) once the output buffer may be written.
  template <int LAYER, class Epi>
  __device__ __forceinline__ void layer(const uint16_t* in, int plane,
                                        int stride, Epi epi) {
    Acc<S, S::NTW> acc;
    if constexpr (S::RES) {
      if constexpr (LAYER == 0) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb)
          if (kb < n.nk1)
            products<S, S::NTW>(acc, w.w1[kb], in, plane, stride, kb, lane);
      } else {
#pragma unroll
        for (int kb = 0; kb < S::NKH; ++kb)
          products<S, S::NTW>(acc, w.w2[kb], in, plane, stride, kb, lane);
      }
    } else if constexpr (LAYER == 0) {
      w.s1.run(acc, wb, 0, n.plane, 0, n.nk1, S::H / 16, wave * S::NTW, in,
               plane, stride, lane);
      w.s2.start(wb, n.off2, n.plane, 0, S::NKH, S::H / 16, wave * S::NTW,
                 lane);
    } else {
      w.s2.run(acc, wb, n.off2, n.plane, 0, S::NKH, S::H / 16,
               wave * S::NTW, in, plane, stride, lane);
#pragma unroll
      for (int o = 0; o < S::NO; ++o)
        if (S::NO == 1 ? kh < n.ks : nb_of(o) < n.nn3)
          w.s3[o].start(wb, n.off3, n.plane, k0, nk3, n.nn3, nb_of(o), lane);
    }
    // in place: every wave has read its input first
    if (!S::DB && LAYER == 1) __syncthreads();
    acc.finish();
    epi(acc.v);
  }

  // tanh layer LAYER from buffer `in`; act: the layer values of row r0 + r
  // are stored there (MfmaArgs::act_out), or null.
  template <int LAYER>
  __device__ __forceinline__ void hidden(const uint16_t* in, int plane,
                                         int stride, float* act, int r0) {
    layer<LAYER>(in, plane, stride, [&](f32x4(&acc)[S::MT][S::NTW]) {
      tanh_out<LAYER>(acc, act, r0);
    });
  }
  template <int LAYER>
  __device__ __forceinline__ void tanh_out(f32x4 (&acc)[S::MT][S::NTW],
                                           float* act, int r0) {
    const float* bias = fv() + (LAYER == 0 ? 0 : 2 * S::H);
    const float* w1t = fv() + S::H;
    uint16_t* out = A(LAYER);
    float tc[S::OM];
#pragma unroll
    for (int m = 0; m < S::OM; ++m)
      tc[m] = LAYER == 0 ? tcol()[S::CNF && S::MT == 1 ? (c & 7) : m * 16 + c]
                         : 0.f;
#pragma unroll
    for (int t = 0; t < S::NTW; ++t) {
      const int f = (wave * S::NTW + t) * 16 + q * 4;
      const f32x4 b = *reinterpret_cast<const f32x4*>(bias + f);
      f32x4 wt{0.f, 0.f, 0.f, 0.f};
      if (LAYER == 0) wt = *reinterpret_cast<const f32x4*>(w1t + f);
#pragma unroll
      for (int m = 0; m < S::OM; ++m) {
        const bool prim = !S::CNF || S::MT == 2 || c < 8;
        f32x4 a, keep = acc[m][t], ta{}, tk{};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          float v = acc[m][t][i] + b[i];
          if (LAYER == 0) v += tc[m] * wt[i];
          a[i] = Op::tanh(v);
        }
        if (S::CNF && S::MT == 2) {  // tangents: the other tile, same lane
          tk = acc[S::MT - 1][t];
#pragma unroll
          for (int i = 0; i < 4; ++i)
            ta[i] = fmaf(-a[i], a[i], 1.f) * tk[i];
        } else if (S::CNF) {  // tangents: the lanes 8 places away
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float ap = xor8(a[i]);
            if (!prim) a[i] = fmaf(-ap, ap, 1.f) * keep[i];
          }
        }
        put4<Op, kPlain>(out + (m * 16 + c) * S::SA + f, S::PA, a);
        if (S::CNF && S::MT == 2)
          put4<Op, kPlain>(out + (16 + c) * S::SA + f, S::PA, ta);
        if (act != nullptr) {
          // activations of primal rows, pre-activation tangents of tangents
          const int g = r0 + (prim ? m * 16 + c : c - 8);
          if (g < n.B) {
            float* p =
                act + ((size_t)(g + (prim ? 0 : n.B)) * 2 + LAYER) * n.H + f;
            put_act(p, prim ? a : keep, f);
            if (S::CNF && S::MT == 2)
              put_act(p + (size_t)n.B * 2 * n.H, tk, f);
          }
        }
      }
    }
  }
  __device__ __forceinline__ void put_act(float* p, f32x4 v, int f) const {
    if ((n.H & 3) == 0) {
      if (f < n.H) *reinterpret_cast<f32x4*>(p) = v;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (f + i < n.H) p[i] = v[i];
    }
  }

  // The output layer from A(1), whole in the owning lanes (one barrier when
  // its k blocks are split).
  __device__ __forceinline__ void output(f32x4 (&acc)[S::NO][S::MT][1]) {
    const uint16_t* in = A(1);
#pragma unroll
    for (int o = 0; o < S::NO; ++o) {
      Acc<S, 1> c;
      const bool on = S::NO == 1 ? kh < n.ks : nb_of(o) < n.nn3;
      if (on) {
        if constexpr (S::RES) {
#pragma unroll
          for (int kb = 0; kb < S::NKH / 2; ++kb)
            if (kb < nk3)
              products<S, 1>(c, w.w3[kb], in, S::PA, S::SA, k0 + kb,
                             lane);
        } else {
          w.s3[o].run(c, wb, n.off3, n.plane, k0, nk3, n.nn3, nb_of(o),
                      in, S::PA, S::SA, lane);
        }
        c.finish();
        if (S::NO == 1 && kh > 0)
#pragma unroll
          for (int m = 0; m < S::MT; ++m)
            red()[(((kh - 1) * n.nn3 + nb3) * S::MT + m) * 64 + lane] =
                c.v[m][0];
      }
#pragma unroll
      for (int m = 0; m < S::MT; ++m) acc[o][m][0] = c.v[m][0];
    }
    start1();
    if (S::NO == 1 && n.ks > 1) __syncthreads();
    if (S::NO == 1 && owner)
      for (int j = 0; j + 1 < n.ks; ++j)
#pragma unroll
        for (int m = 0; m < S::MT; ++m)
          acc[0][m][0] += red()[((j * n.nn3 + nb3) * S::MT + m) * 64 + lane];
  }

  // k = f(t, Y) for the rows of the tile: Y's elements are in LDS
  // (put_input), the stage time in tcol; kl: the CNF's log-density
  // derivative of row c (in every owning lane).  Barriers: one at entry,
  // one after each layer; the caller may write the next input as soon as
  // this returns.
  __device__ __forceinline__ void eval(Vec& k, float& kl, const Vec& ep,
                                       float* act, int r0) {
    __syncthreads();
    hidden<0>(X(), l.px, l.sx, act, r0);
    __syncthreads();
    hidden<1>(A(0), S::PA, S::SA, act, r0);
    __syncthreads();
    f32x4 acc[S::NO][S::MT][1];
    output(acc);
#pragma unroll
    for (int o = 0; o < S::NO; ++o) {
      if (!has(o)) continue;
      const f32x4 b = *reinterpret_cast<const f32x4*>(fv() + 3 * S::H + f0(o));
#pragma unroll
      for (int m = 0; m < S::OM; ++m) k[m][o] = acc[o][m][0] + b;
      if (S::CNF) {
        // eps . (dg/dz eps): over this lane's features, then the four
        // feature groups; the output tiles meet in LDS
        const f32x4 v = acc[o][S::MT - 1][0];
        float d = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) d = fmaf(ep[0][o][i], v[i], d);
        d += __shfl_xor(d, 16, 64);
        d += __shfl_xor(d, 32, 64);
        if (q == 0 && (S::MT == 2 || c >= 8))
          ldot()[nb_of(o) * S::PR + (S::MT == 2 ? c : c - 8)] = d;
      }
    }
    if (S::CNF) {
      __syncthreads();
      float s = 0.f;
      if (owner)
        for (int nb = 0; nb < n.nn3; ++nb)
          s += ldot()[nb * S::PR + (S::MT == 2 ? c : (c & 7))];
      kl = -s;
    }
  }
};

// Four floats of a caller's array, which may lie at any float.
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));

// Elements f .. f + 3 of a row of `lim` (zero beyond).
__device__ __forceinline__ f32x4 row4(const float* p, int f, int lim,
                                      bool vec) {
  if (vec && f + 3 < lim) return *reinterpret_cast<const f32x4u*>(p + f);
  f32x4 v{};
#pragma unroll
  for (int i = 0; i < 4; ++i) v[i] = f + i < lim ? p[f + i] : 0.f;
  return v;
}
__device__ __forceinline__ void put_row4(float* p, int f, int lim, bool vec,
                                         f32x4 v) {
  if (vec && f + 3 < lim) {
    *reinterpret_cast<f32x4u*>(p + f) = v;
    return;
  }
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (f + i < lim) p[f + i] = v[i];
}

// acc += a * v, skipped for a zero coefficient (uniform).
__device__ __forceinline__ void axpy(f32x4& acc, float a, f32x4 v) {
  if (a != 0.f) acc += a * v;
}

constexpr size_t kLdsMax = 160 * 1024;

template <class K, class A>
hipError_t launch(K kernel, int grid, int block, size_t sm, const A& args,
                  hipStream_t s) {
  if (sm > kLdsMax) return hipErrorInvalidValue;
  if (sm > 65536) {
    const hipError_t e = hipFuncSetAttribute(
        reinterpret_cast<const void*>(kernel),
        hipFuncAttributeMaxDynamicSharedMemorySize, (int)sm);
    if (e != hipSuccess) return e;
  }
  hipLaunchKernelGGL(kernel, dim3(grid), dim3(block), sm, s, args);
  return hipGetLastError();
}

}  // namespace ntile
}  // namespace bode
