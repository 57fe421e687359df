// Internal declarations shared by the HIP sources of libdlm (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>

#include "../../include/dlm.h"

typedef __bf16 bf16_t;
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// IEEE half: what a bf16 model's matrix-core operands are stored as.  Same bytes and matrix-core rate as bf16 with three more
// mantissa bits; values beyond +-65504 saturate (to_f16_sat).
//   * attention: Q, the KV cache, the unnormalised probabilities;
//   * GEMMs (op_t): every activation a GEMM reads (the norm outputs h * gain, the attention output, the gated FFN activation)
//     and the packed weights.  A bf16 weight converts exactly unless it is below 2^-14 in magnitude (then it keeps an absolute
//     error of at most 2^-25).  Rounding the activations to bf16's 8 mantissa bits instead is what carries most of a deep
//     model's logit error: at 32 layers of the 8B shape the worst logit error is 1.4e-2 of the row's scale with bf16 norm
//     outputs (whatever the precision of the others) and 0.5e-2 with all of them in half.
// The residual stream stays fp32, the logits bf16.
typedef _Float16 f16_t;
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef f16_t op_t;
typedef f16x8 op8;
typedef f16x4 op4;

#define DLM_WAVE 64

int dlm_fail(int code, const char* fmt, ...);
#define DLM_HIP(expr)                                                                        \
  do {                                                                                       \
    hipError_t e_ = (expr);                                                                  \
    if (e_ != hipSuccess) return dlm_fail(DLM_EHIP, "%s: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

// ---- activation layouts -------------------------------------------------------------------
// fp32 models keep activations row-major.  bf16 models keep every GEMM input (op_t) in "fragment tiles":
// element (m, k) of an [M, K] matrix lives in the 1 KiB tile (m/16, k/32), at lane
// (m%16) + 16*((k%32)/8), slot k%8 -- exactly one operand of the 16x16x32 half-precision matrix-core
// instruction per tile, so a wavefront fetches an operand as 64 consecutive 16-byte pieces.
__host__ __device__ inline size_t tile_index(int m, int k, int K) {
  return ((size_t)(m >> 4) * (size_t)(K >> 5) + (size_t)(k >> 5)) * 512 + (size_t)(((m & 15) + 16 * ((k & 31) >> 3)) * 8 + (k & 7));
}
// bf16 KV cache of one (slot, kv head): K in tiles of 16 positions x 32 dims (A operand of S^T = K Q^T), V in tiles of 16 dims x 32
// positions (A operand of O^T = V^T P^T) whose 8-element lane slots hold positions {4g..4g+3, 16+4g..16+4g+3} of the 32-block: the order in
// which the first product leaves the keys in a lane's registers.
__host__ __device__ inline size_t kv_k_index(int pos, int d, int hd) {
  return ((size_t)(pos >> 4) * (size_t)(hd >> 5) + (size_t)(d >> 5)) * 512 + (size_t)(((pos & 15) + 16 * ((d & 31) >> 3)) * 8 + (d & 7));
}
__host__ __device__ inline size_t kv_v_index(int pos, int d, int hd) {
  const int p32 = pos & 31, r = p32 & 15, g = r >> 2, j = (r & 3) + 4 * (p32 >> 4);
  return ((size_t)(pos >> 5) * (size_t)(hd >> 4) + (size_t)(d >> 4)) * 512 + (size_t)(((d & 15) + 16 * g) * 8 + j);
}

template <typename T> struct Act;
template <> struct Act<float> {  // x_t: what the model's GEMM inputs are stored as
  typedef float x_t;
  static __device__ inline size_t idx(int m, int k, int K) { return (size_t)m * K + k; }
};
template <> struct Act<bf16_t> {
  typedef op_t x_t;
  static __device__ inline size_t idx(int m, int k, int K) { return tile_index(m, k, K); }
};

__device__ inline float to_f32(float x) { return x; }
__device__ inline float to_f32(bf16_t x) { return (float)x; }
__device__ inline float to_f32(f16_t x) { return (float)x; }
__device__ inline f16_t to_f16_sat(float x) { return (f16_t)__builtin_amdgcn_fmed3f(x, -65504.f, 65504.f); }
__device__ inline f32x4 mfma_op(op8 a, op8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }

// ---- values over the lanes of a wavefront without trips through LDS (all 64 lanes together).  A butterfly (lanes 32, 16, 8, 4, 2, 1 apart):
// permlane swaps across the rows of 16 lanes, then rotations within a row, which behind the step before them meet the butterfly's
// values (they repeat every 8, 4 and 2 lanes), so sums are those of a chain of __shfl_xor.
template <int CTRL>
__device__ inline unsigned rotate(unsigned v) { return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false); }
template <typename Op>
__device__ inline unsigned row_butterfly(unsigned v, Op op) {  // over the 16 lanes of a row
  v = op(v, rotate<0x128>(v));  // row_ror:8, 4, 2, 1
  v = op(v, rotate<0x124>(v));
  v = op(v, rotate<0x122>(v));
  return op(v, rotate<0x121>(v));
}
template <typename Op>
__device__ inline unsigned butterfly(unsigned v, Op op) {
  auto x = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  v = op(x[0], x[1]);
  x = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  return row_butterfly(op(x[0], x[1]), op);
}
struct BitsAdd { __device__ unsigned operator()(unsigned a, unsigned b) const { return __float_as_uint(__uint_as_float(a) + __uint_as_float(b)); } };
struct BitsMax { __device__ unsigned operator()(unsigned a, unsigned b) const { return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b))); } };
__device__ inline float wave_sum(float v) { return __uint_as_float(butterfly(__float_as_uint(v), BitsAdd())); }
__device__ inline float wave_max(float v) { return __uint_as_float(butterfly(__float_as_uint(v), BitsMax())); }
__device__ inline float row_sum(float v) { return __uint_as_float(row_butterfly(__float_as_uint(v), BitsAdd())); }
__device__ inline float row_max(float v) { return __uint_as_float(row_butterfly(__float_as_uint(v), BitsMax())); }
// the value `ofs` lanes up (1, 2, 4, 8, 16 or 32; the same for all), in the lanes below ofs: what a reduction into lane 0 needs
__device__ inline unsigned from_up(unsigned v, int ofs) {
  switch (ofs) {
    case 32: return __builtin_amdgcn_permlane32_swap(v, v, false, false)[1];
    case 16: return __builtin_amdgcn_permlane16_swap(v, v, false, false)[1];  // (also in lanes 32 .. 47)
    case 8: return rotate<0x108>(v);  // row_shl:8, 4, 2, 1
    case 4: return rotate<0x104>(v);
    case 2: return rotate<0x102>(v);
    default: return rotate<0x101>(v);
  }
}
__device__ inline float from_up(float v, int ofs) { return __uint_as_float(from_up(__float_as_uint(v), ofs)); }
__device__ inline int from_up(int v, int ofs) { return (int)from_up((unsigned)v, ofs); }

// ---- per-pass metadata, passed to kernels by value -------------------------------------------
#define DLM_MAX_SEQS 32

struct SeqMeta {
  int32_t n_seqs;
  int32_t row_off[DLM_MAX_SEQS + 1];
  int32_t span_start[DLM_MAX_SEQS];
  int32_t slot[DLM_MAX_SEQS];
  int32_t tok_start[DLM_MAX_SEQS];
};
struct StatsMeta {  // which rows are compared with / retained as p^prev; offsets in elements of the retained-logit buffer
  int32_t kl_first[DLM_MAX_SEQS], kl_count[DLM_MAX_SEQS], save_first[DLM_MAX_SEQS], save_count[DLM_MAX_SEQS];
  int64_t prev_off[DLM_MAX_SEQS], save_off[DLM_MAX_SEQS];
};
inline int compared_rows(const StatsMeta& sm) {  // (entries beyond the pass's sequences are zero)
  int n = 0;
  for (int c : sm.kl_count) n += c;
  return n;
}
struct AttnMeta {
  int32_t n_seqs;
  int32_t row_off[DLM_MAX_SEQS + 1];
  int32_t n_keys[DLM_MAX_SEQS];   // keys [0, n_keys) of the slot's cache are visible to every row of the sequence
  int32_t slot[DLM_MAX_SEQS];
};
struct BoundaryMeta {
  int32_t win_start[DLM_MAX_SEQS];
  int32_t win_len[DLM_MAX_SEQS];
  int32_t cold[DLM_MAX_SEQS];
};
struct SelectMeta {
  int32_t row_start[DLM_MAX_SEQS];
  int32_t tok_start[DLM_MAX_SEQS];
  int32_t block_len[DLM_MAX_SEQS];
};
struct RowTables {  // device arrays of one pass, [rows]
  int32_t* row_pos;   // absolute position
  int32_t* row_slot;  // KV-cache slot of the row's sequence
  float* rope_cos;    // [rows, hd/2]
  float* rope_sin;
  int64_t* prev_row;  // element offset of the row's retained p^prev logits, or -1
  int64_t* save_row;  // element offset where the row's logits are retained, or -1
};

// ---- launchers (callers have validated shapes) -------------------------------------------------
// weight tiling: W [N, K] row-major bf16 -> 1 KiB fragments of 16 rows x 32 k in half precision (op_t), `pr` (1 or 2) row-tiles interleaved along k:
// fragment (nt, kt) sits at ((nt/pr * K/32 + kt) * pr + nt%pr) KiB.  The rows may be permuted first so that the columns an
// epilogue has to combine share one 16-column output tile (packed row n holds source row weight_source_row(n, ...)):
//   PERM_ROTARY (param = head_dim): tile b of a head holds dims 8b..8b+7 and their rotary partners 8b+hd/2..8b+hd/2+7
//   PERM_GATED  (param = d_ffn):    tile g holds gate rows 8g..8g+7 and the up rows 8g..8g+7
enum { PERM_NONE = 0, PERM_ROTARY = 1, PERM_GATED = 2 };
__host__ __device__ inline int weight_source_row(int n, int perm, int param) {
  if (perm == PERM_ROTARY) {
    const int head = n / param, w = n % param, c = w & 15;
    return head * param + 8 * (w >> 4) + (c & 7) + (c >= 8 ? param / 2 : 0);
  }
  if (perm == PERM_GATED) {
    const int c = n & 15, o = 8 * (n >> 4) + (c & 7);
    return c < 8 ? o : param + o;
  }
  return n;
}
__host__ __device__ inline int weight_pack_rows(int N) { return N <= 8192 ? 1 : 2; }  // narrow matrices: one run per 16-column tile
void launch_pack_weight(const bf16_t* w, op_t* out, int N, int K, int perm, int perm_param, hipStream_t st);
// W [N, K] row-major -> step-major fragments for the kernel that serves (N, K) at up to 16 rows: column groups of ct tiles
// and W = 4 wavefronts per workgroup (the mid kernel's no-split launches), or ct = 1 and W = 8 (the skinny kernel's 16-column
// workgroups).  The fragment (column tile g ct + r, k-tile w KT/W + s) that wavefront w of workgroup g reads at its step s sits
// at (((s G + g) W + w) ct + r) KiB, G = N / (16 ct): what all workgroups read at the same step is one run of memory, and the
// chip's reads at any moment are one moving window instead of thousands of separate streams.
void launch_pack_weight_steps(const bf16_t* w, op_t* out, int N, int K, int ct, int perm, int perm_param, hipStream_t st);
int gemm_bf16_steps_ct(int N, int K, int kind);  // ct of that layout for (N, K) under epilogue `kind`, 0 if the kernel that serves 16 rows has none
int gemm_mid_steps_ct(int N, int K);   // ... if the mid kernel serves (N, K) at up to 16 rows without a K split, else 0
void launch_pack_act(const bf16_t* x, op_t* out, int M, int K, hipStream_t st);  // row-major bf16 -> fragment tiles in half (rows padded to 16 with zeros)
size_t gemm_bf16_part_elems(int M, int N, int K, int kind);  // floats of GemmEpi::part a launch of this shape and epilogue needs (0: it does not split K)
int gemm_bf16_ssq_chunks(int M, int N, int K);     // chunks per row of the sums of squares an EPI_RESID launch of this shape writes
int gemm_bf16_counters(int max_n);                 // counters a state needs in GemmEpi::counters (zero-initialised, self-resetting)
// rs (optional): every output row m is multiplied by rsqrt(sum_c rs.ssq[m][c] * rs.inv_d + rs.eps).
struct RowScale {
  const float* ssq;
  int nch;
  float inv_d, eps;
};
enum { EPI_DIRECT = 0, EPI_QKV = 1, EPI_SWIGLU = 2, EPI_RESID = 3, EPI_SUM = 4, EPI_STATS = 5 };
// What the bf16 GEMM does with a finished output tile (see gemm_bf16.hip).
struct GemmEpi {
  int kind;
  float* part;        // gemm_bf16_part_elems floats: the partial tiles of a launch that splits K
  int* counters;      // gemm_bf16_counters tickets of such a launch
  RowScale rs;        // 1/rms of the GEMM's input rows (QKV, SWIGLU, DIRECT, SUM; ssq may be null)
  // EPI_QKV (weights packed with PERM_ROTARY)
  const int32_t *row_pos, *row_slot;
  const float *rope_cos, *rope_sin;
  f16_t *q, *kcache, *vcache;  // IEEE half (see f16_t); q in fragment tiles [rows, n_q * hd]
  size_t slot_stride, head_stride;
  int n_q, n_kv, hd;
  // EPI_SWIGLU (weights packed with PERM_GATED): act in fragment tiles
  op_t* act;
  int ffn;
  // EPI_RESID: h += y; x = h * gain (fragment tiles); ssq_out[m][gemm_bf16_ssq_chunks(M, N, K)] = each column tile's share of sum h^2
  float* h;
  const float* gain;
  op_t* x;
  float* ssq_out;
  // EPI_DIRECT / EPI_SUM
  bf16_t* out_bf16;
  // EPI_STATS (the LM head of a pass that compares and retains no row; at most GEMM_STATS_MAX_ROWS rows): logits to out_bf16 as
  // EPI_DIRECT does, and per row and column group the online-softmax state of the group's logits as written (rounded to bf16,
  // token skip_col left out) to stat_parts[m][gemm_bf16_stat_parts(M, N, K)]
  void* stat_parts;
  int skip_col;
  // optional second copy of W in the step-major layout (launch_pack_weight_steps) of column groups of w_steps_ct tiles
  const op_t* w_steps;
  int w_steps_ct;
  bool w_cached;  // W may still be in the memory-side cache from the pass before (WEIGHTS_CACHED_BYTES): it is read there, not past it
};
// A model whose matrices are together no larger than this finds them, or enough of them, in the memory-side cache (256 MB) at its next
// pass; the weights of a larger one never stay that long and are read non-temporally.  Layers of 1024 x 2816 behind a head of 16384, 8
// and 37 rows, non-temporal / plain: 265 MB 212 / 202 and 292 / 271 us a pass, 316 MB 254 / 251 and 351 / 345, 342 MB 275 / 274 and 381 /
// 380, 393 MB 317 / 322 and 439 / 443; 4 layers of 1024 x 3584 (135 MB) 115 / 103 and 160 / 138.
constexpr size_t WEIGHTS_CACHED_BYTES = (size_t)320 << 20;
constexpr int GEMM_STATS_MAX_ROWS = 64;
int gemm_bf16_stat_parts(int M, int N, int K);       // column groups per row an EPI_STATS launch of this shape writes states for
// The GEMM kernels are launched through hipExtLaunchKernelGGL, which can stamp two events with the kernel's own start and end
// (the dispatch's timestamps: what a profiler reports, with no marker packets between dependent kernels).  A caller that
// wants the next GEMM launch of this thread timed sets g_launch_stamp; the launch takes the events and clears it.
struct LaunchStamp { hipEvent_t start, stop; };
extern thread_local LaunchStamp g_launch_stamp;
#define DLM_LAUNCH(kernel, grid, block, lds, st, ...)                                                                           \
  do {                                                                                                                          \
    const LaunchStamp ls_ = g_launch_stamp;                                                                                     \
    g_launch_stamp = LaunchStamp{nullptr, nullptr};                                                                             \
    hipExtLaunchKernelGGL((kernel), dim3(grid), dim3(block), (unsigned)(lds), (st), ls_.start, ls_.stop, 0, __VA_ARGS__);       \
  } while (0)
// Y = X * W^T.  xt: fragment-tiled [Mpad, K]; wt: weights [N, K] as packed by launch_pack_weight.
void launch_gemm_bf16(const op_t* xt, const op_t* wt, int M, int N, int K, const GemmEpi& e, hipStream_t st);
#define GEMM_SKINNY_MAX_ROWS 64
void launch_gemm_skinny(const op_t* xt, const op_t* wt, int pr, int M, int N, int K, const GemmEpi& e, hipStream_t st);  // M <= GEMM_SKINNY_MAX_ROWS
size_t gemm_mid_part_elems(int M, int N, int K);
int gemm_mid_ssq_chunks(int M, int N, int K);
bool gemm_mid_fills_chip(int M, int N, int K);  // its column groups are a whole number of rounds over the compute units, without a K split
bool gemm_mid_one_round(int M, int N, int K);   // its workgroups are at most one round
int gemm_mid_counters(int max_n);
void launch_gemm_mid(const op_t* xt, const op_t* wt, int M, int N, int K, const GemmEpi& e, hipStream_t st);  // the row counts choose_kernel sends (gemm_bf16.hip)
int gemm_macro_ssq_chunks(int M, int N, int K);
struct GemmPlan {
  int kernel;                // 0 skinny, 1 mid, 2 macro (choose_kernel)
  int tile_rows, tile_cols;  // of a workgroup
  int splits, k_parts;       // workgroups that share a tile; parts K is summed in (one workgroup can keep two)
  int workgroups, ssq_parts; // ...; EPI_RESID: chunks of the sums of squares per column block
};
GemmPlan gemm_macro_plan(int M, int N, int K, int kind);  // (kernel left to the caller)
GemmPlan gemm_mid_plan(int M, int N, int K);
GemmPlan gemm_bf16_plan(int M, int N, int K, int kind);
size_t gemm_macro_part_elems(int M, int N, int K, int kind);
int gemm_macro_stat_parts(int M, int N, int K);
int gemm_macro_counters();
void launch_gemm_macro(const op_t* xt, const op_t* wt, int M, int N, int K, const GemmEpi& e, hipStream_t st);
// What the fp32 model's GEMM does with a finished output tile (gemm_f32.hip); the same kinds as GemmEpi, on row-major operands.
struct GemmF32Epi {
  RowScale rs;  // 1/rms of the GEMM's input rows (QKV, SWIGLU, DIRECT; ssq may be null)
  // EPI_QKV: Q row-major, K (after the rotary embedding) and V to cache[slot][pos][n_kv * hd]
  const int32_t *row_pos, *row_slot;
  const float *rope_cos, *rope_sin;
  float *q, *kcache, *vcache;
  size_t slot_stride;
  int n_q, n_kv, hd;
  // EPI_SWIGLU
  float* act;
  int ffn;
  // EPI_RESID: h += y; x = h * gain; ssq_out[m][gemm_f32_pairs(N, EPI_RESID)]
  float* h;
  const float* gain;
  float *x, *ssq_out;
  // EPI_DIRECT
  float* out;
};
int gemm_f32_pairs(int N, int kind);
void launch_gemm_f32(const float* x, const float* w, int M, int N, int K, int kind, const GemmF32Epi& e, hipStream_t st);

// RMSNorm in two halves: producers write x = h * gain and per-row sums of squares (ssq; the embedding writes norm_chunks(d) chunks
// per row); the consumer of the following GEMM multiplies rsqrt(sum(ssq)/d + eps) back in (a per-row scalar commutes with the GEMM).
int norm_chunks(int d);
// The first launch of a pass: row tables and rotary tables, h = embedding row, x = h * gain, ssq
template <typename T>
void launch_embed(const SeqMeta& meta, const StatsMeta& sm, const T* embed, const int32_t* tokens, const RowTables& t, const float* gain, float* h,
                  typename Act<T>::x_t* x, float* ssq, int rows, int d, int vocab, int head_dim, const float* rope_table, hipStream_t st);
// cosines and sines of every position, [positions][hd]: hd/2 cosines, then hd/2 sines (computed in 64 bits)
void launch_rope_table(float* table, int positions, int head_dim, float theta, hipStream_t st);
// softmax(q k^T / sqrt(hd)) v over keys [0, n_keys) of the row's slot.  fp32 model: q, out [rows, n_q*hd] and the cache (row-major
// [pos][n_kv*hd] per slot) are row-major; bf16 models' cache: per (slot, kv head) a region of head_stride elements in the fragment tiling above.
void launch_attention_f32(const float* q, const float* kcache, const float* vcache, size_t slot_stride, const AttnMeta& meta, float* out,
                          int max_seq_rows, int n_q, int n_kv, int hd, hipStream_t st);
// bf16 models: q (fragment tiles [rows, n_q*hd]) and the KV cache hold IEEE half; the output goes to out_tiles (fragment tiles [rows, n_q*hd] in half: the O
// projection's input) if that is given, else to out_rows (row-major bf16)
struct AttnPlan {
  int waves, shares, tiles;  // of a workgroup: wavefronts, workgroups that share a head's output dims, 16-query tiles
};
AttnPlan attention_plan(int max_seq_rows, int n_seqs, int n_tiles, int n_q, int hd);  // n_tiles: of all sequences together
void launch_attention_f16(const f16_t* q, const f16_t* kcache, const f16_t* vcache, size_t slot_stride, size_t head_stride, const AttnMeta& meta,
                          op_t* out_tiles, bf16_t* out_rows, int rows, int max_seq_rows, int n_q, int n_kv, int hd, hipStream_t st);
// test helper of dlm_attention: K, V [T, n_kv, hd] row-major bf16 -> the tiled half-precision cache layout of one slot
void launch_pack_kv(const bf16_t* k, const bf16_t* v, f16_t* kt, f16_t* vt, int T, int n_kv, int hd, size_t head_stride, hipStream_t st);

struct StatsOut {
  float *max_logit, *lse, *entropy, *kl, *conf;
  int32_t* argmax;
};
struct StatsRows {
  const int64_t* prev_row;  // DEVICE [rows] or null: offset (elements) of the row's p^prev logits in prev_base, -1 = none
  const int64_t* save_row;  // DEVICE [rows] or null: offset where the row's logits are copied, -1 = none
  const void* prev_base;
  void* save_base;
  const float* prev_lse;    // indexed by prev_row / vocab; null = recompute from the logits
  float* save_lse;          // indexed by save_row / vocab
};
struct StatsPlan {
  int threads;        // of a workgroup
  int chunk, chunks;  // tokens of a chunk, chunks of a row (more than one: a second launch merges them)
  bool vector;        // rows are read in 16-byte vectors
  int per_unit;       // workgroups of 256 threads of that path on a compute unit
};
StatsPlan stats_plan(int rows, int vocab, int elem_size);
size_t stats_workspace_bytes(int rows);
constexpr size_t STATS_STATE_BYTES = 32;  // one online-softmax state (stats_part.h)
// Finishes rows whose online-softmax states were written per column group by an EPI_STATS GEMM: parts [rows][nparts] states
// (stats_part.h), merged in a fixed order.
void launch_stats_merge(const void* parts, int rows, int nparts, int vocab, const StatsRows& sr, const StatsOut& o, hipStream_t st);
template <typename T>
void launch_vocab_stats(const T* logits, int rows, int compared, int vocab, int mask_id, const StatsRows& sr, const StatsOut& o, void* workspace, hipStream_t st);

void launch_block_boundary(const float* I, const float* H, const BoundaryMeta& meta, int n_seqs, dlm_boundary_params p, int32_t* L_out,
                           float* S_out, float* margin_out, hipStream_t st);
template <typename T>
void launch_select(const T* logits, int vocab, const float* lse, const float* conf, const int32_t* argmax, int32_t* tokens,
                   const SelectMeta& meta, int n_seqs, int mask_id, dlm_select_params p, int apply, uint8_t* sel, int32_t* nsel,
                   float* margin, hipStream_t st);
