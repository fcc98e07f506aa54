// Tile shapes and LDS of the FP64 neural fields: host arithmetic alone, so
// that it can be checked without a GPU.
#pragma once

#include <cstddef>

#if defined(__HIPCC__)
#define BODE_HD __host__ __device__
#else
#define BODE_HD
#endif

namespace bode {
namespace f64t {

constexpr int kWV = 8;     // wavefronts per tile
constexpr int kPad = 8;    // LDS row padding (doubles): rows 64 bytes apart
constexpr int kFrag = 128; // elements per fragment

struct Dims {
  int nk1, nkd, nkh, nnh, nnd;  // k blocks of 8, column tiles of 16
  int SX, SA;                   // LDS row strides
};

BODE_HD inline Dims dims(int din, int H) {
  Dims d;
  d.nk1 = (din + 1 + 7) / 8;  // inputs and the time feature
  d.nkd = (din + 7) / 8;
  d.nkh = (H + 7) / 8;
  d.nnh = (H + 15) / 16;
  d.nnd = (din + 15) / 16;
  d.SX = d.nk1 * 8 + kPad;
  d.SA = d.nnh * 16 + kPad;
  return d;
}

// A compute unit's LDS, and what the kernels declare statically of it beside
// the dynamic part laid out here (flags of the tile and its rows: 16 bytes
// the field and solve kernels, 80 the vector-Jacobian products).
constexpr size_t kLdsUnit = 160 * 1024, kLdsStatic = 128;
constexpr size_t kLdsMax = kLdsUnit - kLdsStatic;

// Bytes of a tile of 4 mt rows: inputs and two layer buffers.
inline size_t tile_lds(int mt, int din, int H) {
  const Dims d = dims(din, H);
  return sizeof(double) * 4 * mt * ((size_t)d.SX + 2 * (size_t)d.SA);
}

// Whether a field's smallest tile fits.
inline bool tile_fits(int din, int H, bool cnf) {
  return tile_lds(cnf ? 2 : 1, din, H) <= kLdsMax;
}

// 4-row groups of a tile (tangent rows included): as many as still give
// every compute unit a tile, 4 instances up to 1024 of them, 8 to 2048, then
// 16 (CNF: 4, then 8 with their tangents), while the layers fit in LDS.
inline int row_groups(int B, int din, int H, bool cnf) {
  int mt = cnf ? (B > 1024 ? 4 : 2) : (B > 2048 ? 4 : B > 1024 ? 2 : 1);
  while (mt > (cnf ? 2 : 1) && tile_lds(mt, din, H) > kLdsMax) mt /= 2;
  return mt;
}

// A launch's dynamic LDS: the tile, and behind it a block of `slots` vectors
// [D] of each of its instances while that fits too.
struct LdsPlan {
  size_t bytes;
  int off;     // of the block
  bool block;  // it is there
};

inline LdsPlan lds_plan(int mt, int D, int din, int H, bool cnf, int slots) {
  LdsPlan p{tile_lds(mt, din, H), 0, false};
  p.off = (int)p.bytes;
  const int rows = cnf ? 2 * mt : 4 * mt;
  const size_t all = p.bytes + sizeof(double) * slots * rows * (size_t)D;
  p.block = slots > 0 && all <= kLdsMax;
  if (p.block) p.bytes = all;
  return p;
}

}  // namespace f64t
}  // namespace bode
