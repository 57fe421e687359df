// Block-vs-prefix attention: every row of a sequence's span attends, without causal mask, to keys
// [0, n_keys) of the sequence's KV-cache slot (cached prefix + the span's own rows, which the
// QKV GEMM's epilogue has already written there).  Grouped-query heads share K/V.
//
// fp32 model (head_dim 32/64/128, row-major cache [pos][n_kv*hd]): one workgroup per (16-query
// tile, head, sequence); keys are streamed in tiles through LDS with an online softmax in fp32.
#include "attention_core.h"

namespace {

constexpr int QT = 16;        // query rows per workgroup
constexpr int KTILE = 32;     // keys per LDS tile
constexpr float NEG_BIG = -3.0e38f;

// What bounds it is latency (the fp32 model's passes are small): K and V of the next tile are in flight while a tile is computed, and
// LDS is read four values at a time; maxima and sums over a query's lanes go by rotation (8 rows x 72 keys, 4 heads: 8.2 us with a trip to
// memory per tile and one value per read, 5.6 with exchanges through LDS and a barrier behind the probabilities, 4.9 now).
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));  // (a caller's rows need not lie on 16 bytes)

template <int HD>
__global__ __launch_bounds__(256) void attention_kernel(const float* __restrict__ q, const float* __restrict__ kcache, const float* __restrict__ vcache,
                                                        size_t slot_stride, AttnMeta meta, float* __restrict__ out, int n_q, int n_kv) {
  constexpr int EPT = HD / 16;                   // output elements per thread: consecutive ones
  constexpr int VPT = KTILE * HD / (256 * 4);    // vectors of a tile per thread
  constexpr int PAD = 4;                         // (rows of 16 lanes start four banks apart)
  __shared__ __align__(16) float qs[QT][HD];
  __shared__ __align__(16) float ks[KTILE][HD + PAD];
  __shared__ __align__(16) float vs[KTILE][HD];
  __shared__ __align__(16) float ps[QT][KTILE];
  typedef float vec_t __attribute__((ext_vector_type(EPT)));

  const int b = blockIdx.z, head = blockIdx.y;
  const int row0 = meta.row_off[b] + blockIdx.x * QT;
  const int row_end = meta.row_off[b + 1];
  if (row0 >= row_end) return;
  const int n_keys = meta.n_keys[b];
  const int kvh = head / (n_q / n_kv);
  const size_t kv_row = (size_t)n_kv * HD;
  const float* kbase = kcache + (size_t)meta.slot[b] * slot_stride + (size_t)kvh * HD;
  const float* vbase = vcache + (size_t)meta.slot[b] * slot_stride + (size_t)kvh * HD;
  const int tid = threadIdx.x, qi = tid >> 4, lx = tid & 15;
  const float scale = rsqrtf((float)HD);

  f32x4 kn[VPT], vn[VPT];  // the next tile's vectors; keys past the end re-read the last one (they are masked below)
  auto fetch = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      const int at = (tid + 256 * i) * 4;
      const size_t o = (size_t)min(k0 + at / HD, n_keys - 1) * kv_row + at % HD;
      kn[i] = *(const f32x4_any*)(kbase + o);
      vn[i] = *(const f32x4_any*)(vbase + o);
    }
  };
  fetch(0);
  for (int i = tid * 4; i < QT * HD; i += 256 * 4) {
    const int r = i / HD, e = i % HD;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
    if (row0 + r < row_end) v = *(const f32x4_any*)(q + (size_t)(row0 + r) * n_q * HD + (size_t)head * HD + e) * scale;
    *(f32x4*)&qs[r][e] = v;
  }
  float m = NEG_BIG, l = 0.f;
  vec_t o = {};

  for (int k0 = 0; k0 < n_keys; k0 += KTILE) {
    if (k0) __syncthreads();  // the previous tile has been read
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
      const int at = (tid + 256 * i) * 4;
      const bool ok = k0 + at / HD < n_keys;
      const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
      *(f32x4*)&ks[at / HD][at % HD] = ok ? kn[i] : zero;
      *(f32x4*)&vs[at / HD][at % HD] = ok ? vn[i] : zero;
    }
    __syncthreads();
    if (k0 + KTILE < n_keys) fetch(k0 + KTILE);
    // scores: thread (qi, lx) handles keys lx and lx + 16
    float s0 = 0.f, s1 = 0.f;
#pragma unroll 8
    for (int e = 0; e < HD; e += 4) {
      const f32x4 qv = *(const f32x4*)&qs[qi][e], a = *(const f32x4*)&ks[lx][e], c = *(const f32x4*)&ks[lx + 16][e];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        s0 = fmaf(qv[t], a[t], s0);
        s1 = fmaf(qv[t], c[t], s1);
      }
    }
    if (k0 + lx >= n_keys) s0 = NEG_BIG;
    if (k0 + lx + 16 >= n_keys) s1 = NEG_BIG;
    const float tm = row_max(fmaxf(s0, s1));
    const float mn = fmaxf(m, tm);
    const float corr = __expf(m - mn);
    const float p0 = (k0 + lx < n_keys) ? __expf(s0 - mn) : 0.f;
    const float p1 = (k0 + lx + 16 < n_keys) ? __expf(s1 - mn) : 0.f;
    const float ts = row_sum(p0 + p1);
    l = l * corr + ts;
    m = mn;
    ps[qi][lx] = p0;
    ps[qi][lx + 16] = p1;
    asm volatile("" ::: "memory");  // (a query's 16 lanes, which read these, are of one wavefront, whose accesses to LDS stay in order)
    o *= corr;
#pragma unroll 4
    for (int kk = 0; kk < KTILE; kk += 4) {
      const f32x4 p = *(const f32x4*)&ps[qi][kk];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const vec_t v = *(const vec_t*)&vs[kk + t][lx * EPT];
#pragma unroll
        for (int n = 0; n < EPT; ++n) o[n] = fmaf(p[t], v[n], o[n]);
      }
    }
  }
  const int r = row0 + qi;
  if (r < row_end) {
    float* dst = out + (size_t)r * n_q * HD + head * HD + lx * EPT;
#pragma unroll
    for (int n = 0; n < EPT; ++n) dst[n] = o[n] / l;
  }
}

// ---- bf16 models: on the matrix cores, half-precision operands (attention_core.h) -----------------------------
// One workgroup per (T 16-query tiles, head, sequence), or DS of them with a share of the head's output dims each; `groups` of T
// tiles cover the longest span.
// per_unit = 0: grid (groups * DS, heads, sequences).  per_unit > 0: a 1-D grid in which the per_unit workgroups that read the
// same K and V (the query tiles, output-dim shares and query heads of one kv head of one sequence) have ids congruent mod 8:
// they run on the same XCD, and all but the first reader find K and V in its L2 (the XCDs' L2s are separate: spread over
// them, every tile of a block fetches its own copy from memory).
// The arguments in front of slot_stride arrive in registers.  ONE: a single sequence of `rows` rows and `keys` keys, whose slot kcache
// and vcache point at: nothing is read from memory before Q and K (8 rows x 400 keys 5.7 -> 5.3
// us, 37 rows x 1537 13.4 -> 12.7, 152 rows x 792 13.5 -> 12.7).
template <int HD, int NWV, int DS, int T, bool ONE>
__global__ __launch_bounds__(NWV * 64, T > 1 ? 2 : 1) void attention_mfma_kernel(const f16_t* __restrict__ q, const f16_t* __restrict__ kcache,
                                                                  const f16_t* __restrict__ vcache, size_t head_stride, int n_q, int n_kv, int per_unit,
                                                                  int groups, int rows, int keys, size_t slot_stride, AttnMeta meta,
                                                                  op_t* __restrict__ out_tiles, bf16_t* __restrict__ out_rows) {
  __shared__ AttnLds<HD, NWV, DS, T> L;
  int b = blockIdx.z, head = blockIdx.y, x = blockIdx.x;
  if (per_unit > 0) {
    const int j = blockIdx.x >> 3, w = j % per_unit, unit = (j / per_unit) * 8 + (blockIdx.x & 7);
    if (unit >= n_kv * (ONE ? 1 : meta.n_seqs)) return;
    b = ONE ? 0 : unit / n_kv;
    head = (unit - b * n_kv) * (n_q / n_kv) + w / (groups * DS);
    x = w % (groups * DS);
  }
  const int group = x / DS, dpart = x - group * DS;
  const int row0 = (ONE ? 0 : meta.row_off[b]) + group * 16 * T;
  const int row_end = ONE ? rows : meta.row_off[b + 1];
  if (row0 >= row_end) return;
  const int kvh = head / (n_q / n_kv);
  const size_t region = (ONE ? 0 : (size_t)meta.slot[b] * slot_stride) + (size_t)kvh * head_stride;
  attention_tiles<HD, NWV, DS, T>(q, kcache + region, vcache + region, row0, min(row_end, row0 + 16 * T), ONE ? keys : meta.n_keys[b], head, n_q, out_tiles, out_rows, L, dpart);
}

// K [T, n_kv, hd] and V row-major bf16 -> the tiled half-precision cache layout of one slot (test helper for dlm_attention)
__global__ void pack_kv_kernel(const bf16_t* __restrict__ k, const bf16_t* __restrict__ v, f16_t* __restrict__ kt, f16_t* __restrict__ vt,
                               int T, int n_kv, int hd, size_t head_stride) {
  const size_t total = (size_t)T * n_kv * hd;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (size_t)gridDim.x * blockDim.x) {
    const int d = i % hd, h = (i / hd) % n_kv, pos = i / ((size_t)hd * n_kv);
    kt[(size_t)h * head_stride + kv_k_index(pos, d, hd)] = to_f16_sat((float)k[i]);
    vt[(size_t)h * head_stride + kv_v_index(pos, d, hd)] = to_f16_sat((float)v[i]);
  }
}

}  // namespace

void launch_pack_kv(const bf16_t* k, const bf16_t* v, f16_t* kt, f16_t* vt, int T, int n_kv, int hd, size_t head_stride, hipStream_t st) {
  pack_kv_kernel<<<256, 256, 0, st>>>(k, v, kt, vt, T, n_kv, hd, head_stride);
}

void launch_attention_f32(const float* q, const float* kcache, const float* vcache, size_t slot_stride, const AttnMeta& meta, float* out,
                          int max_seq_rows, int n_q, int n_kv, int hd, hipStream_t st) {
  dim3 grid((max_seq_rows + QT - 1) / QT, n_q, meta.n_seqs);
  if (hd == 32) attention_kernel<32><<<grid, 256, 0, st>>>(q, kcache, vcache, slot_stride, meta, out, n_q, n_kv);
  else if (hd == 64) attention_kernel<64><<<grid, 256, 0, st>>>(q, kcache, vcache, slot_stride, meta, out, n_q, n_kv);
  else attention_kernel<128><<<grid, 256, 0, st>>>(q, kcache, vcache, slot_stride, meta, out, n_q, n_kv);
}

// How a pass is laid out.  A narrow one (few query tiles x heads): eight wavefronts per workgroup to shorten each wavefront's chain
// of dependent loads, and the output dims of a head split over four workgroups (two for 64 dims) to spread its K / V traffic.  A
// wide one has enough workgroups to fill the chip with four wavefronts each.
// Query tiles per workgroup, where a span has more than one: a wide pass takes two (the K and V traffic is what bounds it); a narrow
// one the fewest that leave at most one workgroup per compute unit (8B shape, 24 rows x 856 keys, one tile / two: 7.7 / 9.7 us;
// 37 rows x 1537: 22.3 / 16.1; two shares of a 64-dim head never are more than that).  Spans of one tile gain nothing from a second
// that no row fills (28 heads, 3 sequences of 16 rows x 1516 keys, two tiles / one: 25.7 / 22.2).
// A middling pass has eight wavefronts, of which a unit holds one workgroup (128 dims): two tiles where that makes one round of two (by events, 28 heads,
// 152 rows x 792 keys, 280 workgroups / 140: 17.9 / 13.9).  Not where two tiles are more than a round themselves (32 heads, 5 spans of 40
// rows x 640, 480 / 320: 24.8 / 28.5), nor where spans of other lengths leave so many workgroups without rows that one tile each is a
// round as well (40 + 8 + 8 rows x 640, 160 of 288 / 128 of 192: 14.2 / 16.4; 40 + 4 x 8, 224 of 480 / 192 of 320: 16.8 / 25.0).  But workgroups
// go round the 8 XCDs and each XCD's 4 shader engines by their number: where the longest span has 2, or 4, 8, .. tiles, those of the spans
// of one tile, every 2nd, 4th .. of the numbers, meet in a few of these places and take a second round of them after all (17 + 4 x 8
// rows x 640, 192 of 320 / 160 of 160: 23.1 / 18.5; 64 + 8 + 8, 192 of 384 / 128 of 192: 21.8 / 16.3).
AttnPlan attention_plan(int max_seq_rows, int n_seqs, int n_tiles, int n_q, int hd) {
  const int tiles = (max_seq_rows + 15) / 16;
  const size_t units = (size_t)tiles * n_q * n_seqs;
  if (units < 128 && hd >= 64) return AttnPlan{8, hd == 128 ? 4 : 2, hd == 128 && tiles > 1 && units * 4 > 256 ? 2 : 1};
  if (units >= 512) return AttnPlan{4, 1, tiles > 1 ? 2 : 1};
  const bool one_round_of_pairs = (size_t)(tiles + 1) / 2 * n_q * n_seqs <= 256;
  const bool two_rounds_of_tiles = n_tiles * n_q >= 256 || tiles == 2 || tiles % 4 == 0;
  return AttnPlan{8, 1, units > 256 && tiles > 1 && one_round_of_pairs && two_rounds_of_tiles ? 2 : 1};
}

void launch_attention_f16(const f16_t* q, const f16_t* kcache, const f16_t* vcache, size_t slot_stride, size_t head_stride, const AttnMeta& meta,
                          op_t* out_tiles, bf16_t* out_rows, int rows, int max_seq_rows, int n_q, int n_kv, int hd, hipStream_t st) {
  const int tiles = (max_seq_rows + 15) / 16;
  int n_tiles = 0;
  for (int b = 0; b < meta.n_seqs; ++b) n_tiles += (meta.row_off[b + 1] - meta.row_off[b] + 15) / 16;
  const AttnPlan p = attention_plan(max_seq_rows, meta.n_seqs, n_tiles, n_q, hd);
  // enough (kv head, sequence) units to keep every XCD busy (four each): the workgroups of a unit share an XCD (see the kernel)
  const int units = n_kv * meta.n_seqs;
  const bool by_unit = units >= 32;
  const int groups = (tiles + p.tiles - 1) / p.tiles, per_unit = by_unit ? groups * p.shares * (n_q / n_kv) : 0;
  const dim3 grid = by_unit ? dim3((units + 7) / 8 * 8 * per_unit) : dim3(groups * p.shares, n_q, meta.n_seqs);
  const bool one = meta.n_seqs == 1 && meta.row_off[0] == 0;
  if (one) {
    kcache += (size_t)meta.slot[0] * slot_stride;
    vcache += (size_t)meta.slot[0] * slot_stride;
  }
  const int one_rows = meta.row_off[1], one_keys = meta.n_keys[0];
#define LAUNCH(HD, NWV, DS, T, ONE)                                                                                                                  \
  attention_mfma_kernel<HD, NWV, DS, T, ONE><<<grid, NWV * 64, 0, st>>>(q, kcache, vcache, head_stride, n_q, n_kv, per_unit, groups, one_rows, one_keys, \
                                                                        slot_stride, meta, out_tiles, out_rows)
#define GO(HD, NWV, DS, T)                    \
  do {                                        \
    if (one) LAUNCH(HD, NWV, DS, T, true);    \
    else LAUNCH(HD, NWV, DS, T, false);       \
  } while (0)
#define BY_TILES(HD, NWV, DS)              \
  do {                                     \
    if (p.tiles == 2) GO(HD, NWV, DS, 2);  \
    else GO(HD, NWV, DS, 1);               \
  } while (0)
  if (hd == 32) { if (p.waves == 4) BY_TILES(32, 4, 1); else BY_TILES(32, 8, 1); }
  else if (hd == 64) { if (p.shares > 1) GO(64, 8, 2, 1); else if (p.waves == 4) BY_TILES(64, 4, 1); else BY_TILES(64, 8, 1); }
  else { if (p.shares > 1) BY_TILES(128, 8, 4); else if (p.waves == 4) BY_TILES(128, 4, 1); else BY_TILES(128, 8, 1); }
#undef BY_TILES
#undef GO
#undef LAUNCH
}
