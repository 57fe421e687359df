// Online-softmax state of a slice of one row of logits, and how two slices combine (Sec. 4.2: Eq. 3 and the entropy signal;
// Sec. 4.3: confidence and prediction).  Shared by the streamed vocabulary reduction and by the LM-head epilogue that produces
// the same states per column group.
#pragma once
#include "common.h"

constexpr float NEG_BIG = -3.0e38f;   // "minus infinity" that keeps every product finite
constexpr float MASKED = -1.0e30f;    // logit given to the mask token: e^(MASKED - m) == 0

struct Part {  // online-softmax state of a slice of one row
  float m, s, t, w;
  float bv;    // best logit
  int bi;      // its token id
  float pm, ps;  // max and sum e^(z'-pm) of the previous-step row (only when its lse is not stored)
};

static_assert(sizeof(Part) == STATS_STATE_BYTES, "the workspace is sized in states of 32 bytes");

__device__ inline Part part_init() { return Part{NEG_BIG, 0.f, 0.f, 0.f, NEG_BIG, 0x7fffffff, NEG_BIG, 0.f}; }

__device__ inline Part part_merge(const Part& a, const Part& b) {
  Part r;
  r.m = fmaxf(a.m, b.m);
  float da = a.m - r.m, db = b.m - r.m;
  float fa = __expf(da), fb = __expf(db);
  r.s = fa * a.s + fb * b.s;
  r.t = fa * (a.t + da * a.s) + fb * (b.t + db * b.s);
  r.w = fa * a.w + fb * b.w;
  bool tb = (b.bv > a.bv) || (b.bv == a.bv && b.bi < a.bi);
  r.bv = tb ? b.bv : a.bv;
  r.bi = tb ? b.bi : a.bi;
  r.pm = fmaxf(a.pm, b.pm);
  r.ps = __expf(a.pm - r.pm) * a.ps + __expf(b.pm - r.pm) * b.ps;
  return r;
}

__device__ inline Part part_from(const Part& p, int ofs) {  // (from_up)
  return Part{from_up(p.m, ofs), from_up(p.s, ofs), from_up(p.t, ofs), from_up(p.w, ofs), from_up(p.bv, ofs), from_up(p.bi, ofs), from_up(p.pm, ofs), from_up(p.ps, ofs)};
}

// The part of a row's online-softmax state that a pass without a previous-step distribution needs (stats_part.h has the whole):
// maximum (= the best logit), sum e^(z-m), sum e^(z-m)(z-m), lowest token id of the maximum.
struct LiteState {
  float m, s, t;
  int bi;
};
__device__ __attribute__((always_inline)) inline LiteState lite_init() { return LiteState{NEG_BIG, 0.f, 0.f, 0x7fffffff}; }
__device__ __attribute__((always_inline)) inline LiteState lite_merge(const LiteState a, const LiteState b) {
  LiteState r;
  r.m = fmaxf(a.m, b.m);
  const float da = a.m - r.m, db = b.m - r.m;
  const float fa = __expf(da), fb = __expf(db);
  r.s = fa * a.s + fb * b.s;
  r.t = fa * (a.t + da * a.s) + fb * (b.t + db * b.s);
  r.bi = (b.m > a.m || (b.m == a.m && b.bi < a.bi)) ? b.bi : a.bi;
  return r;
}
__device__ __attribute__((always_inline)) inline LiteState lite_from(const LiteState p, int ofs) {  // (from_up)
  return LiteState{from_up(p.m, ofs), from_up(p.s, ofs), from_up(p.t, ofs), from_up(p.bi, ofs)};
}
// state of four consecutive logits, token ids n .. n+3, token `skip` left out
__device__ __attribute__((always_inline)) inline LiteState lite_of(f32x4 v, int n, int skip) {
  float z[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) z[i] = (float)(bf16_t)v[i];  // the logit as stored
  LiteState r = lite_init();
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (n + i != skip && z[i] > r.m) { r.m = z[i]; r.bi = n + i; }  // ascending ids and strict '>' keep the lowest id
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (n + i == skip) continue;
    const float d = z[i] - r.m, ex = __expf(d);
    r.s += ex;
    r.t = fmaf(ex, d, r.t);
  }
  return r;
}
