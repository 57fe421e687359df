// GEMM of the fp32 model  Y[M,N] = X[M,K] * W[N,K]^T, row-major operands, with the layer's row-wise glue in its epilogue
// (GemmF32Epi): QKV (1/rms, rotary embedding, Q and the KV cache), gated activation, residual + next norm's input, or the product.
//
// The fp32 model is small (its matrices are tens to hundreds of KiB), so a launch is bound by latency: one trip to memory, a
// reduction, one trip back.  A workgroup of four wavefronts owns MT row tiles x two 16-column tiles - the two halves of a rotary
// pair, a gate tile and its up tile, or two neighbours - so that the epilogue has both in one lane; its wavefronts split K, fetch
// their operands straight into registers, D steps of 16 k at a time, and multiply them on the fp32 matrix cores
// (v_mfma_f32_16x16x4_f32: lane 16 kq + r holds four consecutive k of row r, one per instruction; W and X use the same order of
// k, so it is only a permutation of the sum); the four accumulators meet in LDS and are added in wavefront order (deterministic).
// The first loads need only arguments that arrive in registers and go out without a path around any of them, and what the epilogue
// reads goes out right behind them.  8 rows x 768 columns x 128: 18 us with 64 x 64 tiles staged through LDS 16 k at a time, 3.7 with operands
// in registers but guarded loads and an epilogue that reads on its own, 3.4 now; 8 rows x 128 columns x 384: 48 / 5.2 / 4.2, x 128: 3.6 -> 2.7
// (kernel trace).
#include "gemm_epilogue.h"

namespace {

constexpr int NWV = 4, TPB = NWV * 64;

// four consecutive k of a row whose elements need not be aligned, or K no multiple of 4
__device__ inline f32x4 load4(const float* row, int k, int K) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (k + i < K) v[i] = row[k + i];
  return v;
}

// VEC: rows are 16-byte aligned and K is a multiple of 4.  unit: EPI_QKV the head's size, EPI_SWIGLU the activation's columns (with the
// arguments before it, what the first loads need: they arrive in registers, and e is read behind those loads)
template <int MT, int D, int EPI, bool VEC>
__global__ __launch_bounds__(TPB) void gemm_f32_kernel(const float* __restrict__ x, const float* __restrict__ w, int M, int N, int K, int unit, GemmF32Epi e) {
  __shared__ f32x4 red[NWV][2 * MT][64];
  __shared__ float s_rinv[MT * 16];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), g = lane >> 4, r = lane & 15;
  const int p = blockIdx.x, m0 = blockIdx.y * MT * 16;
  // the workgroup's two column tiles
  int c0 = 32 * p, c1 = 32 * p + 16, end0 = N, end1 = N;
  if (EPI == EPI_QKV) {
    const int per = unit >> 5, head = p / per;
    c0 = head * unit + 16 * (p - head * per);
    c1 = c0 + (unit >> 1);
  } else if (EPI == EPI_SWIGLU) {
    c0 = 16 * p;
    c1 = unit + 16 * p;
    end0 = unit;
  }
  const int steps = (K + 15) >> 4, per = (steps + NWV - 1) / NWV, s1 = min(steps, (wave + 1) * per);
  // rows and columns that do not exist read the last one that does: the loads are unconditional, and what they get is never stored
  const float* wr[2] = {w + (size_t)min(c0 + r, end0 - 1) * K, w + (size_t)min(c1 + r, end1 - 1) * K};
  const float* xr[MT];
#pragma unroll
  for (int j = 0; j < MT; ++j) xr[j] = x + (size_t)min(m0 + j * 16 + r, M - 1) * K;

  f32x4 acc[2][MT];
#pragma unroll
  for (int j = 0; j < MT; ++j) acc[0][j] = acc[1][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  f32x4 wv[D][2], xv[D][MT];
  auto load = [&](int s) __attribute__((always_inline)) {  // steps past the wavefront's last one, and k past the end, are left out by multiply
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int k = min(s + d, steps - 1) * 16 + 4 * g, kc = VEC ? min(k, K - 4) : k;
#pragma unroll
      for (int t = 0; t < 2; ++t) wv[d][t] = VEC ? *(const f32x4*)(wr[t] + kc) : load4(wr[t], kc, K);
#pragma unroll
      for (int j = 0; j < MT; ++j) xv[d][j] = VEC ? *(const f32x4*)(xr[j] + kc) : load4(xr[j], kc, K);
    }
  };
  auto multiply = [&](int s) __attribute__((always_inline)) {
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const bool in = s + d < s1 && (s + d) * 16 + 4 * g < K;
#pragma unroll
      for (int t = 0; t < 2; ++t) wv[d][t] = in ? wv[d][t] : zero;
#pragma unroll
      for (int j = 0; j < MT; ++j) xv[d][j] = in ? xv[d][j] : zero;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j)
#pragma unroll
          for (int t = 0; t < 2; ++t) acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[d][t][i], xv[d][j][i], acc[t][j], 0, 0, 0);
    }
  };
  load(wave * per);
  __builtin_amdgcn_sched_barrier(0);
  // what the epilogue reads besides the products, fetched while the first operands are in flight: 1/rms of the input rows (published by the
  // reduction's barrier), and for the row tile that this wavefront finishes (wavefront j row tile j) residuals and gains, or rotary cosines
  // and sines and the rows' places in the cache
  constexpr bool SCALED = EPI == EPI_QKV || EPI == EPI_SWIGLU || EPI == EPI_DIRECT;
  typedef RinvBatch<TPB, MT * 16, 4> Rinv;
  const int rows = min(M - m0, MT * 16);
  Rinv rinv;
  const bool rinv_batched = Rinv::fits(e.rs);
  if (SCALED && rinv_batched) rinv.fetch(e.rs, m0, rows);
  const int j = wave < MT ? wave : 0, m = m0 + j * 16 + r, mc = min(m, M - 1), n0 = c0 + 4 * g, n1 = c1 + 4 * g;
  const int head = EPI == EPI_QKV ? c0 / unit : 0, half = unit >> 1, i0 = n0 - head * unit;
  f32x4 ahead[2][2] = {};
  int slot = 0, pos = 0;
  if (wave < MT) {
    if (EPI == EPI_RESID) {  // (N is a multiple of 4)
#pragma unroll
      for (int t = 0; t < 2; ++t) {
        const int n = min(t ? n1 : n0, N - 4);
        ahead[t][0] = *(const f32x4*)(e.h + (size_t)mc * N + n);
        ahead[t][1] = *(const f32x4*)(e.gain + n);
      }
    } else if (EPI == EPI_QKV) {
      if (head < e.n_q + e.n_kv) {
        ahead[0][0] = *(const f32x4*)(e.rope_cos + (size_t)mc * half + i0);
        ahead[0][1] = *(const f32x4*)(e.rope_sin + (size_t)mc * half + i0);
      }
      if (head >= e.n_q) {
        slot = e.row_slot[mc];
        pos = e.row_pos[mc];
      }
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  int s = wave * per;
  while (true) {
    multiply(s);
    s += D;
    if (s >= s1) break;
    load(s);
  }
  if (SCALED) {
    if (rinv_batched) rinv.publish(e.rs, rows, s_rinv);
    else block_rinv<TPB>(e.rs, m0, rows, s_rinv);
  }
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int j = 0; j < MT; ++j) red[wave][t * MT + j][lane] = acc[t][j];
  __syncthreads();

  // wavefront j finishes row tile j: lane 16 g + r has columns 4g .. 4g + 3 of both column tiles of row r
  if (wave >= MT) return;
  f32x4 a = ((red[0][j][lane] + red[1][j][lane]) + red[2][j][lane]) + red[3][j][lane];
  f32x4 b = ((red[0][MT + j][lane] + red[1][MT + j][lane]) + red[2][MT + j][lane]) + red[3][MT + j][lane];
  const bool row = m < M;
  if (EPI == EPI_RESID) {  // (N is a multiple of 4)
    float ss[2] = {0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int n = t ? n1 : n0;
      if (row && n < N) {
        const f32x4 v = ahead[t][0] + (t ? b : a);
        *(f32x4*)(e.h + (size_t)m * N + n) = v;
        *(f32x4*)(e.x + (size_t)m * N + n) = v * ahead[t][1];
        ss[t] = v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
      }
    }
    const float sum = sum_row4(ss[0] + ss[1]);
    if (row && g == 0) e.ssq_out[(size_t)m * ((N + 31) >> 5) + p] = sum;
    return;
  }
  if (!row) return;
  if (EPI == EPI_DIRECT) {
    const float sc = s_rinv[j * 16 + r];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      if (n0 + i < N) e.out[(size_t)m * N + n0 + i] = a[i] * sc;
      if (n1 + i < N) e.out[(size_t)m * N + n1 + i] = b[i] * sc;
    }
    return;
  }
  const float scale = s_rinv[j * 16 + r];
  a *= scale;
  b *= scale;
  if (EPI == EPI_SWIGLU) {  // (ffn is a multiple of 4)
    if (n0 >= unit) return;
    f32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = a[i] / (1.f + __expf(-a[i])) * b[i];
    *(f32x4*)(e.act + (size_t)m * unit + n0) = v;
    return;
  }
  if (head < e.n_q + e.n_kv) {  // Q and K heads are rotated
    const f32x4 c = ahead[0][0], sn = ahead[0][1];
    const f32x4 ra = a * c - b * sn, rb = b * c + a * sn;
    a = ra;
    b = rb;
  }
  float* dst;
  if (head < e.n_q) {
    dst = e.q + ((size_t)m * e.n_q + head) * unit;
  } else {
    const bool is_k = head < e.n_q + e.n_kv;
    dst = (is_k ? e.kcache : e.vcache) + (size_t)slot * e.slot_stride + ((size_t)pos * e.n_kv + (head - e.n_q - (is_k ? 0 : e.n_kv))) * unit;
  }
  *(f32x4*)(dst + i0) = a;
  *(f32x4*)(dst + i0 + half) = b;
}

template <int MT, int D, int EPI>
void launch_mt(const float* x, const float* w, int M, int N, int K, const GemmF32Epi& e, bool vec, hipStream_t st) {
  const dim3 grid(gemm_f32_pairs(N, EPI), (M + MT * 16 - 1) / (MT * 16));
  const int unit = EPI == EPI_QKV ? e.hd : EPI == EPI_SWIGLU ? e.ffn : 0;
  if (vec) DLM_LAUNCH((gemm_f32_kernel<MT, D, EPI, true>), grid, TPB, 0, st, x, w, M, N, K, unit, e);
  else if constexpr (EPI == EPI_DIRECT) DLM_LAUNCH((gemm_f32_kernel<MT, D, EPI, false>), grid, TPB, 0, st, x, w, M, N, K, unit, e);
}

template <int EPI>
void launch_epi(const float* x, const float* w, int M, int N, int K, const GemmF32Epi& e, bool vec, hipStream_t st) {
  // as many steps per trip as a quarter of K usually is (K = 384: 6, K = 128: 2) where the registers hold them; a step too many is four
  // products of zeros per column tile
  if (M <= 32 && K <= 128) { if (M <= 16) launch_mt<1, 2, EPI>(x, w, M, N, K, e, vec, st); else launch_mt<2, 2, EPI>(x, w, M, N, K, e, vec, st); }
  else if (M <= 16) launch_mt<1, 6, EPI>(x, w, M, N, K, e, vec, st);
  else if (M <= 32) launch_mt<2, 4, EPI>(x, w, M, N, K, e, vec, st);
  else launch_mt<4, 2, EPI>(x, w, M, N, K, e, vec, st);
}

}  // namespace

// pairs of 16-column tiles (workgroups along the columns) of a launch; EPI_RESID writes one chunk of the sums of squares for each
int gemm_f32_pairs(int N, int kind) { return kind == EPI_SWIGLU ? (N / 2 + 15) / 16 : (N + 31) / 32; }

void launch_gemm_f32(const float* x, const float* w, int M, int N, int K, int kind, const GemmF32Epi& e, hipStream_t st) {
  // vector loads: every row of both operands on a 16-byte boundary.  A model's buffers and dimensions always are; the operands
  // of a plain product need not be.
  const bool vec = K % 4 == 0 && (((uintptr_t)x | (uintptr_t)w) & 15) == 0;
  switch (kind) {
    case EPI_QKV: launch_epi<EPI_QKV>(x, w, M, N, K, e, vec, st); break;
    case EPI_SWIGLU: launch_epi<EPI_SWIGLU>(x, w, M, N, K, e, vec, st); break;
    case EPI_RESID: launch_epi<EPI_RESID>(x, w, M, N, K, e, vec, st); break;
    default: launch_epi<EPI_DIRECT>(x, w, M, N, K, e, vec, st); break;
  }
}
