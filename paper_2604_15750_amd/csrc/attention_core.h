// Block-vs-prefix attention on the matrix cores for a bf16 model's KV cache: the work of one workgroup on T consecutive
// 16-query tiles of one head of one sequence.
// (Running it in the tail of the QKV GEMM of a narrow pass, in the workgroup that finishes a head last, was measured: the
// fused launch took 37 us against 23 + 9 us for the two launches, because the tail is a serial chain of memory round trips.)
//
// The KV cache of a bf16 model holds IEEE half (f16_t in common.h: Q, K, V and the unnormalised probabilities are the
// matrix-core operands here, and with bf16's 8 mantissa bits their rounding is the largest single part of a deep model's
// logit error; half has the same size and matrix-core rate).  It is kept per (slot, kv head) in matrix-core fragment tiles
// (kv_k_index / kv_v_index), so a wavefront fetches a K operand (16 keys x 32 dims) or a V^T operand
// (16 dims x 32 keys) as 64 consecutive 16-byte pieces.  The NWV wavefronts of the workgroup take
// every NWV-th block of 32 keys with their own online-softmax state and are merged through LDS.
// S^T = K Q^T puts 8 keys of one query in each lane (the lane's query is lane%16 in
// both S^T and O^T), so the probabilities feed the second product straight from registers: the V
// tiling stores keys in the order the first product emits them.
//
// What bounds it: with one query tile per workgroup a wavefront fetches 16 KiB of K and V for 32 products, so wide passes ran
// at the L2 -> compute unit rate (1280 rows x 1280 keys x 32 heads: 1.7 GB in 100 us, 17 TB/s).  The T tiles of a workgroup share
// every K and V fragment (two tiles: 64 us).  A tile's arithmetic does not depend on T: the same wavefronts take the same blocks
// and are merged in the same order, so results are bit for bit those of one tile per workgroup.  Then the vector
// instructions of the softmax weigh most: keys are masked in the last block only, the running sums are rescaled only
// where a maximum moved, and lanes exchange by permlane instead of through LDS.  The loads of a step are pinned in front of it:
// 1280 rows 64 -> 57 us, 37 rows x 1537 keys 15.5 -> 14.1 (kernel trace; these and the merge below).
#pragma once
#include "common.h"

typedef float f32x4_lds __attribute__((ext_vector_type(4), aligned(8)));

template <int HD, int NWV, int DS, int T>
struct AttnLds {  // merge buffers of one workgroup (T query tiles, HD / DS of the head's dims)
  float sm[T][NWV][16], sl[T][NWV][16];
  // a query's dims in a row, padded by two banks and accessed in 8-byte halves (by events, rows padded to 16 bytes and accessed whole: 152 rows x
  // 792 keys, 32 heads, 15.6 us against 14.9).  The struct is its kernel's only LDS object, at address 0; told so by alignas, the
  // compiler orders the loads of the shortest passes worse (24 rows x 124 keys 6.6 -> 6.9 us).
  float so[T][NWV][16][HD / DS + 2];
  static_assert(HD / DS % 2 == 0, "rows start on 8 bytes");
};

// v of the lane and of its partner 16 (32) lanes away, in one order or the other (for commutative uses)
struct Two { float a, b; };
__device__ inline Two with16(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return Two{__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ inline Two with32(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return Two{__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ inline float max4(float v) {  // over the four lanes of a query
  Two t = with16(v);
  t = with32(fmaxf(t.a, t.b));
  return fmaxf(t.a, t.b);
}
__device__ inline float sum4(float v) {
  Two t = with16(v);
  t = with32(t.a + t.b);
  return t.a + t.b;
}

// q: fragment tiles [rows, n_q * HD] (as every GEMM input: the QKV epilogue writes whole 16-byte slots, 256 bytes of 16 rows together); kt / vt: the (slot, kv head) region of the tiled cache; rows [row0, row_end) (at most 16 T of
// them) x head `head` against keys [0, n_keys); output to out_tiles (fragment tiles [rows, n_q * HD] in half: the O projection's
// input) if given, else to out_rows (row-major bf16).  Called by every thread of a workgroup of NWV wavefronts.
// DS > 1: the workgroup produces only dims [dpart * HD / DS, (dpart + 1) * HD / DS) of the output: it reads all of K (the
// scores and the softmax are computed by each of the DS workgroups of a head, identically) but only its share of V.  What
// bounds a narrow pass is what one compute unit can pull through its L2 (about 50 GB/s), and K and V of a head are its whole
// traffic: four workgroups per head move 5/8 of it each, with nothing to merge.
template <int HD, int NWV, int DS, int T>
__device__ __attribute__((always_inline)) inline void attention_tiles(const f16_t* __restrict__ q, const f16_t* __restrict__ kregion, const f16_t* __restrict__ vregion,
                                       int row0, int row_end, int n_keys, int head, int n_q, op_t* __restrict__ out_tiles, bf16_t* __restrict__ out_rows,
                                       AttnLds<HD, NWV, DS, T>& L, int dpart) {
  constexpr int KS = HD / 32, DT = HD / 16 / DS, HDP = HD / DS;
  constexpr float NEG_BIG = -3.0e38f;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, g = lane >> 4, c = lane & 15;
  const float scale = rsqrtf((float)HD);
  const f16x8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};

  f16x8 qf[T][KS];
#pragma unroll
  for (int u = 0; u < T; ++u) {
    const int r = row0 + 16 * u + c;
#pragma unroll
    for (int t = 0; t < KS; ++t)
      qf[u][t] = r < row_end ? *(const f16x8*)(q + tile_index(r, head * HD + 32 * t + 8 * g, n_q * HD)) : zero8;
  }
  const f16x8* kt = (const f16x8*)kregion + lane;
  const f16x8* vt = (const f16x8*)vregion + lane;
  float m[T], l[T];
  f32x4 o[T][DT];
#pragma unroll
  for (int u = 0; u < T; ++u) {
    m[u] = NEG_BIG;
    l[u] = 0.f;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) o[u][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // K of the next block and V of the current one are in flight while the current one's scores are computed
  const int nblk = (n_keys + 31) >> 5;
  f16x8 kf[2][2 * KS], vf[DT];
  // A step's loads are pinned in front of it, K of the next block too: past the last block a line per fragment of this one, which
  // nothing uses, as a path around the loads would be one that the compiler's count of them cannot follow (it would wait for all of
  // them).  Not for one query tile with eight wavefronts, which are few blocks each: there the copies it makes of what is in
  // flight cost more (8 rows x 392 keys, four shares, 6.9 us against 6.5; 128 rows x 228 keys, one share, by events 9.4 against 8.3).
  constexpr bool PINNED = T > 1 || (DS == 1 && NWV == 4);
  // (inlined by force: where two kernels of one shape call them the compiler leaves them as functions, and what they share lies in scratch)
  auto load_k = [&](int buf, int blk) __attribute__((always_inline)) {
    const bool there = blk < nblk;
    const f16x8* from = there || !PINNED ? kt : (const f16x8*)kregion;
    const int b = there || !PINNED ? blk : blk - NWV;
#pragma unroll
    for (int t = 0; t < 2 * KS; ++t) kf[buf][t] = there || PINNED ? from[((size_t)b * 2 * KS + t) * 64] : zero8;
  };
  auto load_v = [&](int blk) __attribute__((always_inline)) {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) vf[dt] = vt[((size_t)blk * (DT * DS) + dpart * DT + dt) * 64];
  };
  auto step = [&](int buf, int blk) __attribute__((always_inline)) {
    load_v(blk);
    load_k(buf ^ 1, blk + NWV);
    if (PINNED) __builtin_amdgcn_sched_barrier(0);  // (left alone the scheduler sinks the loads behind the products, and each step waits for its own)
    const bool ragged = blk * 32 + 32 > n_keys;  // (uniform: only the last block has keys to leave out)
#pragma unroll
    for (int u = 0; u < T; ++u) {
      f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int t = 0; t < KS; ++t) {
        s0 = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf[buf][t], qf[u][t], s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf[buf][KS + t], qf[u][t], s1, 0, 0, 0);
      }
      // lane holds, for query c, keys blk*32 + 4g + i (s0) and + 16 (s1)
      float sv[8];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        sv[i] = s0[i] * scale;
        sv[4 + i] = s1[i] * scale;
      }
      if (ragged) {
        const int key0 = blk * 32 + 4 * g;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (key0 + i >= n_keys) sv[i] = NEG_BIG;
          if (key0 + 16 + i >= n_keys) sv[4 + i] = NEG_BIG;
        }
      }
      float mx = sv[0];
#pragma unroll
      for (int i = 1; i < 8; ++i) mx = fmaxf(mx, sv[i]);
      const float mn = fmaxf(m[u], max4(mx));
      const bool moved = __builtin_amdgcn_ballot_w64(mn != m[u]) != 0;  // (a factor of one changes nothing)
      const float corr = __expf(m[u] - mn);
      float pv[8], ps = 0.f;
#pragma unroll
      for (int i = 0; i < 8; ++i) pv[i] = __expf(sv[i] - mn);
      if (ragged) {
        const int key0 = blk * 32 + 4 * g;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          if (key0 + i >= n_keys) pv[i] = 0.f;
          if (key0 + 16 + i >= n_keys) pv[4 + i] = 0.f;
        }
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) ps += pv[i];
      l[u] = l[u] * corr + sum4(ps);
      m[u] = mn;
      if (moved)
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) o[u][dt] *= corr;
      const f16x8 pb = {(f16_t)pv[0], (f16_t)pv[1], (f16_t)pv[2], (f16_t)pv[3], (f16_t)pv[4], (f16_t)pv[5], (f16_t)pv[6], (f16_t)pv[7]};  // in [0, 1]
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) o[u][dt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vf[dt], pb, o[u][dt], 0, 0, 0);
    }
  };
  if (wave < nblk) load_k(0, wave);
  for (int blk = wave; blk < nblk; blk += 2 * NWV) {
    step(0, blk);
    if (blk + NWV < nblk) step(1, blk + NWV);
  }
  // Merge the wavefronts: all query tiles together, four dims per access, and a thread finishes 8 (4) consecutive dims of a query,
  // which are one slot (half of one) of the output tile.  One tile and one value at a time, written two bytes at a time, this
  // took 3.8 us of a workgroup's 21 at 1280 rows x 1280 keys (3.1 now) and 4.2 of 19 at 16 spans of 30 rows x 400 (2.8).  In the kernels
  // of the shortest passes, which share a head's dims, there is a thread for every dim (4 rows x 492 keys 9.0 us with four dims
  // each, 8.6 with one).
#pragma unroll
  for (int u = 0; u < T; ++u) {
    if (row0 + 16 * u >= row_end) break;  // (uniform)
    if (g == 0) { L.sm[u][wave][c] = m[u]; L.sl[u][wave][c] = l[u]; }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) *(f32x4_lds*)&L.so[u][wave][c][16 * dt + 4 * g] = o[u][dt];
  }
  __syncthreads();
  constexpr int CH = 2 * HDP >= NWV * 64 ? 8 : T == 1 && DS > 1 ? 1 : 4, V = CH < 4 ? CH : 4, PER_TILE = 16 * HDP / CH;
  typedef float vec_t __attribute__((ext_vector_type(V), aligned(V == 4 ? 8 : 4)));
  for (int item = tid; item < T * PER_TILE; item += NWV * 64) {
    const int u = item / PER_TILE, qi = item & 15, d0 = (item % PER_TILE >> 4) * CH, r = row0 + 16 * u + qi;
    if (r >= row_end) continue;
    float M = L.sm[u][0][qi];
#pragma unroll
    for (int wv = 1; wv < NWV; ++wv) M = fmaxf(M, L.sm[u][wv][qi]);
    float w[NWV], Lsum = 0.f, acc[CH] = {};
#pragma unroll
    for (int wv = 0; wv < NWV; ++wv) { w[wv] = __expf(L.sm[u][wv][qi] - M); Lsum += w[wv] * L.sl[u][wv][qi]; }
#pragma unroll
    for (int wv = 0; wv < NWV; ++wv)
#pragma unroll
      for (int j = 0; j < CH; j += V) {
        const vec_t t = *(const vec_t*)&L.so[u][wv][qi][d0 + j];
#pragma unroll
        for (int k = 0; k < V; ++k) acc[j + k] += w[wv] * t[k];
      }
    const int width = n_q * HD, col = head * HD + dpart * HDP + d0;
    if (out_tiles) {
      typedef f16_t slot_t __attribute__((ext_vector_type(CH)));
      slot_t v;
#pragma unroll
      for (int j = 0; j < CH; ++j) v[j] = to_f16_sat(acc[j] / Lsum);
      *(slot_t*)(out_tiles + tile_index(r, col, width)) = v;
    } else {
#pragma unroll
      for (int j = 0; j < CH; ++j) out_rows[(size_t)r * width + col + j] = (bf16_t)(acc[j] / Lsum);
    }
  }
}
