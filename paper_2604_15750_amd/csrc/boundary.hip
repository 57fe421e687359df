// DepGA-Block boundary search (paper Sec. 4.2, Eq. 4; cumulative form of Sec. 4.4).
// One workgroup per sequence, one lane per candidate position (window <= 256).  Smoothing uses
// differences of a prefix sum, the cumulative rule a second prefix sum; both are wavefront-shuffle
// scans with a cross-wave carry, in fp64 so the decision does not depend on summation order.
// What bounds it is that chain of dependent exchanges: the two signals go through it side by side, and windows of up to 64
// positions get one wavefront, which waits for no other (64 positions, one signal after the other on 256 threads / now:
// 4.1 / 2.4 us for one sequence, 4.4 / 3.5 for 16).
#include "common.h"

namespace {

struct Two { double a, b; };

template <int NW>
struct Block {
  static constexpr int TPB = NW * 64;
  Two carry[NW];
  Two pre[TPB + 1];

  __device__ Two scan_inclusive(Two v) {
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const double ua = __shfl_up(v.a, o, 64), ub = __shfl_up(v.b, o, 64);
      if (lane >= o) { v.a += ua; v.b += ub; }
    }
    if (NW == 1) return v;
    __syncthreads();  // carry may still be read from a previous scan
    if (lane == 63) carry[wv] = v;
    __syncthreads();
    Two add = {0.0, 0.0};
    for (int i = 0; i < wv; ++i) { add.a += carry[i].a; add.b += carry[i].b; }
    return Two{v.a + add.a, v.b + add.b};
  }
  template <typename Op>
  __device__ Two reduce(Two v, Op op) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const double ua = __shfl_xor(v.a, o, 64), ub = __shfl_xor(v.b, o, 64);
      v = Two{op(v.a, ua), op(v.b, ub)};
    }
    if (NW == 1) return v;
    __syncthreads();
    if ((threadIdx.x & 63) == 0) carry[threadIdx.x >> 6] = v;
    __syncthreads();
    Two r = carry[0];
    for (int i = 1; i < NW; ++i) r = Two{op(r.a, carry[i].a), op(r.b, carry[i].b)};
    return r;
  }
};

struct OpSum { __device__ double operator()(double a, double b) const { return a + b; } };
struct OpMin { __device__ double operator()(double a, double b) const { return a < b ? a : b; } };
struct OpMax { __device__ double operator()(double a, double b) const { return a > b ? a : b; } };

// smoothed and normalised signals for position k (inactive lanes pass 0 and get 0)
template <int NW>
__device__ inline Two smooth_normalise(Two x, int k, int W, int r, int mode, Block<NW>& s) {
  const bool act = k < W;
  const Two inc = s.scan_inclusive(act ? x : Two{0.0, 0.0});
  if (threadIdx.x == 0) s.pre[0] = Two{0.0, 0.0};
  s.pre[threadIdx.x + 1] = inc;
  __syncthreads();
  Two sm = {0.0, 0.0};
  if (act) {
    const int lo = max(0, k - r), hi = min(W - 1, k + r);
    const double n = (double)(hi - lo + 1);
    sm = Two{(s.pre[hi + 1].a - s.pre[lo].a) / n, (s.pre[hi + 1].b - s.pre[lo].b) / n};
  }
  __syncthreads();
  const double eps = 1e-12;
  if (mode == 0) {
    const Two sum = s.reduce(sm, OpSum());
    return Two{sm.a / (sum.a / (double)W + eps), sm.b / (sum.b / (double)W + eps)};
  }
  if (mode == 3) return sm;
  const Two mx = s.reduce(act ? sm : Two{-1.0e300, -1.0e300}, OpMax());
  if (mode == 1) return Two{sm.a / (mx.a + eps), sm.b / (mx.b + eps)};
  const Two mn = s.reduce(act ? sm : Two{1.0e300, 1.0e300}, OpMin());
  return Two{(sm.a - mn.a) / (mx.a - mn.a + eps), (sm.b - mn.b) / (mx.b - mn.b + eps)};
}

template <int NW>
__global__ __launch_bounds__(NW * 64) void block_boundary_kernel(const float* __restrict__ I, const float* __restrict__ H, BoundaryMeta meta,
                                                                 dlm_boundary_params p, int32_t* __restrict__ L_out,
                                                                 float* __restrict__ S_out, float* __restrict__ margin_out) {
  __shared__ Block<NW> sh;
  __shared__ int first_neg[NW];
  const int b = blockIdx.x, k = threadIdx.x;
  const int off = meta.win_start[b], W = meta.win_len[b];
  if (meta.cold[b]) {  // first block: conservative cold start
    if (k < W && S_out) S_out[off + k] = 0.f;
    if (k == 0) {
      L_out[b] = min(p.l_min, W);
      if (margin_out) margin_out[b] = __builtin_inff();
    }
    return;
  }
  const bool act = k < W;
  const Two t = smooth_normalise<NW>(act ? Two{(double)I[off + k], (double)H[off + k]} : Two{0.0, 0.0}, k, W, p.smooth_radius, p.norm_mode, sh);
  double S = act ? t.a - (double)p.lambda * t.b : 0.0;
  if (act && S_out) S_out[off + k] = (float)S;
  double q = S;
  if (p.rule == 1) q = sh.scan_inclusive(Two{S, 0.0}).a;
  // first position whose decision quantity is negative
  unsigned long long neg = __ballot(act && q < 0.0);
  if ((k & 63) == 0) first_neg[k >> 6] = neg ? (k + __ffsll((long long)neg) - 1) : NW * 64;
  __syncthreads();
  int kstar = NW * 64;
  for (int i = 0; i < NW; ++i) kstar = min(kstar, first_neg[i]);
  const bool crossed = kstar < W;
  const double mrg = sh.reduce(Two{(act && (!crossed || k <= kstar)) ? fabs(q) : 1.0e300, 0.0}, OpMin()).a;
  if (k == 0) {
    int L_raw = crossed ? kstar : W;
    L_out[b] = min(max(L_raw, p.l_min), W);
    if (margin_out) margin_out[b] = (float)mrg;
  }
}

}  // namespace

void launch_block_boundary(const float* I, const float* H, const BoundaryMeta& meta, int n_seqs, dlm_boundary_params p,
                                int32_t* L_out, float* S_out, float* margin_out, hipStream_t st) {
  int longest = 0;
  for (int b = 0; b < n_seqs; ++b) longest = meta.win_len[b] > longest ? meta.win_len[b] : longest;
  if (longest <= 64) block_boundary_kernel<1><<<n_seqs, 64, 0, st>>>(I, H, meta, p, L_out, S_out, margin_out);
  else block_boundary_kernel<4><<<n_seqs, 256, 0, st>>>(I, H, meta, p, L_out, S_out, margin_out);
}
