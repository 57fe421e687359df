// The first launch of a pass: row tables, rotary tables, embedding and the first norm's input.  (All other row-wise steps of a
// layer run in its GEMMs' epilogues.)
#include "common.h"

namespace {

__device__ inline float block_sum_256(float v, float* buf) {
  v = wave_sum(v);
  __syncthreads();
  if ((threadIdx.x & 63) == 0) buf[threadIdx.x >> 6] = v;
  __syncthreads();
  return buf[0] + buf[1] + buf[2] + buf[3];
}

// RMSNorm is split in two so that no kernel has to see a whole row: the producer writes
// x = h * gain (unnormalised) plus the sum of squares of its chunk of columns; since
// 1/rms is one scalar per row it commutes with the following GEMM, whose consumer multiplies
// it back in.
constexpr int NORM_CHUNK = 1024;

__device__ inline f32x4 load_embed(const float* e) { return *(const f32x4*)e; }
__device__ inline f32x4 load_embed(const bf16_t* e) {
  const bf16x4 v = *(const bf16x4*)e;
  return f32x4{(float)v[0], (float)v[1], (float)v[2], (float)v[3]};
}
__device__ inline void store_x(float* x, f32x4 v) { *(f32x4*)x = v; }
__device__ inline void store_x(op_t* x, f32x4 v) { *(op4*)x = op4{to_f16_sat(v[0]), to_f16_sat(v[1]), to_f16_sat(v[2]), to_f16_sat(v[3])}; }

// grid (chunks, rows): h = embedding row, x = h * gain, ssq[row][chunk] (four consecutive columns lie together in both layouts
// of x); the row's first workgroup also writes its tables: row -> (position, slot, retained-logit offsets), rotary cosines and
// sines, which it copies from a table by position that the state keeps (computed here in 64 bits: 2822 rows 37 us, 8 rows of the fp32
// model 5.9; now 28 and 4.9).  Bound by its launch at the row counts of a decode: one kernel for both halves instead of two.
template <typename T>
__global__ __launch_bounds__(256) void embed_kernel(SeqMeta meta, StatsMeta sm, const T* __restrict__ embed, const int32_t* __restrict__ tokens,
                                                    RowTables t, const float* __restrict__ gain, float* __restrict__ h,
                                                    typename Act<T>::x_t* __restrict__ x, float* __restrict__ ssq, int d, int vocab, int head_dim,
                                                    const float* __restrict__ rope_table) {
  __shared__ float buf[4];
  const int r = blockIdx.y, k = blockIdx.x * NORM_CHUNK + threadIdx.x * 4;
  const int lane = threadIdx.x & 63;  // the row's sequence: a lane per boundary (a loop over them is a chain of scalar loads)
  const int b = __popcll(__ballot(lane < DLM_MAX_SEQS && lane + 1 < meta.n_seqs && r >= meta.row_off[min(lane, DLM_MAX_SEQS - 1) + 1]));
  const int rel = r - meta.row_off[b], pos = meta.span_start[b] + rel;
  // the token buffer is the caller's device memory, which the host cannot validate: an id outside the vocabulary is clamped
  // into it instead of reading outside the embedding table
  const int tok = min(max(tokens[meta.tok_start[b] + rel], 0), vocab - 1);
  if (blockIdx.x == 0) {
    if (threadIdx.x == 0) {
      t.row_pos[r] = pos;
      t.row_slot[r] = meta.slot[b];
      const int kr = rel - sm.kl_first[b];
      t.prev_row[r] = (kr >= 0 && kr < sm.kl_count[b]) ? sm.prev_off[b] + (int64_t)kr * vocab : -1;
      const int sr = rel - sm.save_first[b];
      t.save_row[r] = (sr >= 0 && sr < sm.save_count[b]) ? sm.save_off[b] + (int64_t)sr * vocab : -1;
    }
    const int half = head_dim / 2;
    for (int i = threadIdx.x; i < head_dim; i += blockDim.x)
      (i < half ? t.rope_cos + i : t.rope_sin + (i - half))[(size_t)r * half] = rope_table[(size_t)pos * head_dim + i];
  }
  float ss = 0.f;
  if (k < d) {
    const f32x4 v = load_embed(embed + (size_t)tok * d + k), g = *(const f32x4*)(gain + k);
    *(f32x4*)(h + (size_t)r * d + k) = v;
    store_x(x + Act<T>::idx(r, k, d), v * g);
    ss = v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
  }
  ss = block_sum_256(ss, buf);
  if (threadIdx.x == 0) ssq[(size_t)r * gridDim.x + blockIdx.x] = ss;
}

// table [positions][head_dim]: a position's cosines, then its sines
__global__ void rope_table_kernel(float* __restrict__ table, int positions, int head_dim, float theta) {
  const int half = head_dim / 2;
  for (size_t k = (size_t)blockIdx.x * blockDim.x + threadIdx.x; k < (size_t)positions * half; k += (size_t)gridDim.x * blockDim.x) {
    const int pos = (int)(k / half), i = (int)(k - (size_t)pos * half);
    const double inv_freq = pow((double)theta, -2.0 * (double)i / (double)head_dim);
    double s, c;
    sincos((double)pos * inv_freq, &s, &c);
    table[(size_t)pos * head_dim + i] = (float)c;
    table[(size_t)pos * head_dim + half + i] = (float)s;
  }
}

}  // namespace

void launch_rope_table(float* table, int positions, int head_dim, float theta, hipStream_t st) {
  const size_t blocks = ((size_t)positions * (head_dim / 2) + 63) / 64;
  rope_table_kernel<<<(int)(blocks < 4096 ? blocks : 4096), 64, 0, st>>>(table, positions, head_dim, theta);
}

int norm_chunks(int d) { return (d + NORM_CHUNK - 1) / NORM_CHUNK; }

template <typename T>
void launch_embed(const SeqMeta& meta, const StatsMeta& sm, const T* embed, const int32_t* tokens, const RowTables& t, const float* gain, float* h,
                  typename Act<T>::x_t* x, float* ssq, int rows, int d, int vocab, int head_dim, const float* rope_table, hipStream_t st) {
  embed_kernel<T><<<dim3(norm_chunks(d), rows), 256, 0, st>>>(meta, sm, embed, tokens, t, gain, h, x, ssq, d, vocab, head_dim, rope_table);
}
template void launch_embed<float>(const SeqMeta&, const StatsMeta&, const float*, const int32_t*, const RowTables&, const float*, float*, float*, float*, int,
                                  int, int, int, const float*, hipStream_t);
template void launch_embed<bf16_t>(const SeqMeta&, const StatsMeta&, const bf16_t*, const int32_t*, const RowTables&, const float*, float*, op_t*, float*, int,
                                   int, int, int, const float*, hipStream_t);
