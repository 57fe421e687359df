// GEMM of the fp32 model  Y[M,N] = X[M,K] * W[N,K]^T, row-major operands, with the layer's row-wise glue in its epilogue
// (GemmF32Epi): QKV (1/rms, rotary embedding, Q and the KV cache), gated activation, residual + next norm's input, or the product.
//
// The fp32 model is small (its matrices are tens to hundreds of KiB), so a launch is bound by latency: one trip to memory, a
// reduction, one trip back.  A workgroup of four wavefronts owns MT row tiles x two 16-column tiles - the two halves of a rotary
// pair, a gate tile and its up tile, or two neighbours - so that the epilogue has both in one lane; its wavefronts split K, fetch
// their operands straight into registers, D steps of 16 k at a time, and multiply them on the fp32 matrix cores
// (v_mfma_f32_16x16x4_f32: lane 16 kq + r holds four consecutive k of row r, one per instruction; W and X use the same order of
// k, so it is only a permutation of the sum); the four accumulators meet in LDS and are added in wavefront order (deterministic).
// 8 rows x 768 columns x 128: 18 us with 64 x 64 tiles staged through LDS 16 k at a time, 4.4 with as many steps per trip as at K = 384, 3.7
// with two; 8 rows x 128 columns x 384: 48 / 5.2 (kernel trace).
#include "gemm_epilogue.h"

namespace {

constexpr int NWV = 4, TPB = NWV * 64;

// four consecutive k of a row; VEC: rows are 16-byte aligned and K is a multiple of 4
template <bool VEC>
__device__ inline f32x4 load4(const float* row, int k, int K, bool ok) {
  f32x4 v = {0.f, 0.f, 0.f, 0.f};
  if (!ok) return v;
  if (VEC) {
    if (k < K) v = *(const f32x4*)(row + k);
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (k + i < K) v[i] = row[k + i];
  }
  return v;
}

template <int MT, int D, int EPI, bool VEC>
__global__ __launch_bounds__(TPB) void gemm_f32_kernel(const float* __restrict__ x, const float* __restrict__ w, int M, int N, int K, GemmF32Epi e) {
  __shared__ f32x4 red[NWV][2 * MT][64];
  __shared__ float s_rinv[MT * 16];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, r = lane & 15;
  const int p = blockIdx.x, m0 = blockIdx.y * MT * 16;
  // the workgroup's two column tiles
  int c0 = 32 * p, c1 = 32 * p + 16, end0 = N, end1 = N;
  if (EPI == EPI_QKV) {
    const int per = e.hd >> 5, head = p / per;
    c0 = head * e.hd + 16 * (p - head * per);
    c1 = c0 + (e.hd >> 1);
  } else if (EPI == EPI_SWIGLU) {
    c0 = 16 * p;
    c1 = e.ffn + 16 * p;
    end0 = e.ffn;
  }
  const int steps = (K + 15) >> 4, per = (steps + NWV - 1) / NWV, s1 = min(steps, (wave + 1) * per);
  const float* wr[2] = {w + (size_t)(c0 + r) * K, w + (size_t)(c1 + r) * K};
  const bool wok[2] = {c0 + r < end0, c1 + r < end1};

  f32x4 acc[2][MT];
#pragma unroll
  for (int j = 0; j < MT; ++j) acc[0][j] = acc[1][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  bool first = true;
  for (int s = wave * per; s < s1; s += D) {
    f32x4 wv[D][2], xv[D][MT];
#pragma unroll
    for (int d = 0; d < D; ++d) {
      const int k = (s + d) * 16 + 4 * g;
      const bool in = s + d < s1;
#pragma unroll
      for (int t = 0; t < 2; ++t) wv[d][t] = load4<VEC>(wr[t], k, K, in && wok[t]);
#pragma unroll
      for (int j = 0; j < MT; ++j) xv[d][j] = load4<VEC>(x + (size_t)(m0 + j * 16 + r) * K, k, K, in && m0 + j * 16 + r < M);
    }
    // 1/rms of the input rows, needed only by the epilogue: fetched while the first operands are in flight (published by the
    // reduction's barrier)
    if (first && (EPI == EPI_QKV || EPI == EPI_SWIGLU || EPI == EPI_DIRECT)) block_rinv<TPB>(e.rs, m0, min(M - m0, MT * 16), s_rinv);
    first = false;
#pragma unroll
    for (int d = 0; d < D; ++d)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < MT; ++j)
#pragma unroll
          for (int t = 0; t < 2; ++t) acc[t][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[d][t][i], xv[d][j][i], acc[t][j], 0, 0, 0);
  }
  if (first && (EPI == EPI_QKV || EPI == EPI_SWIGLU || EPI == EPI_DIRECT)) block_rinv<TPB>(e.rs, m0, min(M - m0, MT * 16), s_rinv);
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int j = 0; j < MT; ++j) red[wave][t * MT + j][lane] = acc[t][j];
  __syncthreads();

  // wavefront j finishes row tile j: lane 16 g + r has columns 4g .. 4g + 3 of both column tiles of row r
  if (wave >= MT) return;
  const int j = wave, m = m0 + j * 16 + r, n0 = c0 + 4 * g, n1 = c1 + 4 * g;
  f32x4 a = ((red[0][j][lane] + red[1][j][lane]) + red[2][j][lane]) + red[3][j][lane];
  f32x4 b = ((red[0][MT + j][lane] + red[1][MT + j][lane]) + red[2][MT + j][lane]) + red[3][MT + j][lane];
  const bool row = m < M;
  if (EPI == EPI_RESID) {  // (N is a multiple of 4)
    float ss[2] = {0.f, 0.f};
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int n = t ? n1 : n0;
      if (row && n < N) {
        const f32x4 v = *(const f32x4*)(e.h + (size_t)m * N + n) + (t ? b : a);
        *(f32x4*)(e.h + (size_t)m * N + n) = v;
        *(f32x4*)(e.x + (size_t)m * N + n) = v * *(const f32x4*)(e.gain + n);
        ss[t] = v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
      }
    }
    float s = ss[0] + ss[1];
    s += __shfl_xor(s, 16, 64);
    s += __shfl_xor(s, 32, 64);
    if (row && g == 0) e.ssq_out[(size_t)m * gridDim.x + p] = s;
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
  const float rinv = s_rinv[j * 16 + r];
  a *= rinv;
  b *= rinv;
  if (EPI == EPI_SWIGLU) {  // (ffn is a multiple of 4)
    if (n0 >= e.ffn) return;
    f32x4 v;
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = a[i] / (1.f + __expf(-a[i])) * b[i];
    *(f32x4*)(e.act + (size_t)m * e.ffn + n0) = v;
    return;
  }
  const int hd = e.hd, half = hd >> 1, head = c0 / hd, i0 = n0 - head * hd;
  if (head < e.n_q + e.n_kv) {  // Q and K heads are rotated
    const f32x4 c = *(const f32x4*)(e.rope_cos + (size_t)m * half + i0), sn = *(const f32x4*)(e.rope_sin + (size_t)m * half + i0);
    const f32x4 ra = a * c - b * sn, rb = b * c + a * sn;
    a = ra;
    b = rb;
  }
  float* dst;
  if (head < e.n_q) {
    dst = e.q + ((size_t)m * e.n_q + head) * hd;
  } else {
    const bool is_k = head < e.n_q + e.n_kv;
    dst = (is_k ? e.kcache : e.vcache) + (size_t)e.row_slot[m] * e.slot_stride + ((size_t)e.row_pos[m] * e.n_kv + (head - e.n_q - (is_k ? 0 : e.n_kv))) * hd;
  }
  *(f32x4*)(dst + i0) = a;
  *(f32x4*)(dst + i0 + half) = b;
}

template <int MT, int D, int EPI>
void launch_mt(const float* x, const float* w, int M, int N, int K, const GemmF32Epi& e, bool vec, hipStream_t st) {
  const dim3 grid(gemm_f32_pairs(N, EPI), (M + MT * 16 - 1) / (MT * 16));
  if (vec) DLM_LAUNCH((gemm_f32_kernel<MT, D, EPI, true>), grid, TPB, 0, st, x, w, M, N, K, e);
  else if constexpr (EPI == EPI_DIRECT) DLM_LAUNCH((gemm_f32_kernel<MT, D, EPI, false>), grid, TPB, 0, st, x, w, M, N, K, e);
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
