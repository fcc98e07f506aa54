// Host dispatch of the neural-field kernels by hidden width.
#include "neural_bwd.hpp"
#include "neural_fwd.hpp"

namespace bode {

namespace {

hipError_t by_width(const FwdCall& c, hipStream_t s) {
  switch (mfma_pad_h(c.H)) {
    case 512: return c.w.f32 ? fwd_f32_h512(c, s) : fwd_h512(c, s);
    case 256: return c.w.f32 ? fwd_f32_h256(c, s) : fwd_h256(c, s);
    case 128: return c.w.f32 ? fwd_f32_h128(c, s) : fwd_h128(c, s);
    case 64: return c.w.f32 ? fwd_f32_h64(c, s) : fwd_h64(c, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t fwd_solve(const Mod<float>& m, const MfmaWeights& w,
                     const TableauArgs& t, int budget, int waves,
                     hipStream_t s) {
  FwdCall c{};
  c.kind = 0;
  c.m = &m;
  c.tab = &t;
  c.B = m.B;
  c.D = m.D;
  c.din = m.d_in;
  c.H = m.H;
  c.cnf = m.cnf;
  c.budget = budget;
  c.waves = waves;
  c.w = w;
  return by_width(c, s);
}

hipError_t fwd_steps(const FwdSteps& v, int din, int H, bool cnf,
                     const MfmaWeights& w, const TableauArgs& t, int waves,
                     hipStream_t s) {
  FwdCall c{};
  c.kind = 1;
  c.steps = &v;
  c.tab = &t;
  c.B = v.B;
  c.D = v.D;
  c.din = din;
  c.H = H;
  c.cnf = cnf;
  c.waves = waves;
  c.w = w;
  return by_width(c, s);
}

hipError_t fwd_stage(const MfmaArgs& a, hipStream_t s) {
  FwdCall c{};
  c.kind = 2;
  c.stage = &a;
  c.B = a.B;
  c.D = a.D;
  c.din = a.din;
  c.H = a.H;
  c.cnf = a.cnf;
  c.waves = a.waves;
  c.w = a.w;
  return by_width(c, s);
}

hipError_t bwd_run(const BwdCall& c, hipStream_t s) {
  switch (mfma_pad_h(c.H)) {
    case 512: return c.w.f32 ? bwd_f32_h512(c, s) : bwd_h512(c, s);
    case 256: return c.w.f32 ? bwd_f32_h256(c, s) : bwd_h256(c, s);
    case 128: return c.w.f32 ? bwd_f32_h128(c, s) : bwd_h128(c, s);
    case 64: return c.w.f32 ? bwd_f32_h64(c, s) : bwd_h64(c, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace bode
