// CAP-Decoding (paper Sec. 4.3, Eq. 5-6, Alg. 1) and the token write of Eq. 2.
// One workgroup per sequence, one lane of its first four wavefronts per block row (block <= 256 rows).  What bounds it is
// latency: a chain of dependent steps, each a trip to memory or to LDS.  So
//   * the pairwise conflict scores (two scalars per pair of pooled rows, gathered straight from the logits) go over all threads
//     of the workgroup, four pairs of loads in flight per thread, over a compacted list of the pooled rows: 1024 threads for
//     blocks of more than 32 rows, whose pairs would otherwise take several trips one after another; the conflicts are a bit
//     matrix in LDS;
//   * the order of the rows is a bit matrix too, a ballot per row and 64 others; ranks are counts of its bits;
//   * the greedy walk of phase 2 (in the order of confidence: take a row, drop its conflicts) runs in rounds: a row whose
//     undecided conflicts all come later in that order is taken, and what conflicts with a row just taken is dropped.  That is
//     the same set as the walk's, in as many rounds as the longest chain of conflicts instead of as many steps as rows.
//   * blocks of up to 64 rows have kernels of their own with sets of two words: straight-line code that runs once is bound by the
//     fetching of its instructions.
// Kernel time on logits in the caches, 16 sequences x 64 rows: 32 us with one thread walking and one pair per thread and trip, 14.6
// with a loop over the rows in each lane for the order and the margin, 7.0 without, 5.7 with sets of two words; one sequence x 8 rows
// 4.3 -> 3.6.
#include "common.h"

namespace {

constexpr float INF = __builtin_inff();

template <int MAXL>
union RowSet {  // one bit per row
  unsigned long long q[MAXL / 64];
  uint32_t w[MAXL / 32];
};

// MAXL: rows a block can have
template <typename T, int TPB, int MAXL>
__global__ __launch_bounds__(TPB) void select_kernel(const T* __restrict__ logits, int vocab, const float* __restrict__ lse_g,
                                                     const float* __restrict__ conf_g, const int32_t* __restrict__ argmax_g,
                                                     int32_t* __restrict__ tokens, SelectMeta meta, int mask_id, dlm_select_params p,
                                                     int apply, uint8_t* __restrict__ sel_out, int32_t* __restrict__ nsel_out,
                                                     float* __restrict__ margin_out) {
  constexpr int RW = MAXL / 64, WORDS = MAXL / 32;  // wavefronts that own rows
  typedef RowSet<MAXL> Rows;
  __shared__ float c[MAXL], lse[MAXL], fbuf[TPB / 64];
  __shared__ int yh[MAXL], list[MAXL];
  __shared__ uint32_t bits[MAXL][WORDS + 1];  // conflicts of a row (padded: lanes read the same word of neighbouring rows)
  __shared__ uint32_t ahead[MAXL][WORDS + 1];  // rows that come before a row in the order of confidence
  __shared__ float sorted[MAXL + 1];
  __shared__ Rows s_elig, s_pool, s_high, s_und, s_new, s_sel;
  __shared__ int top_row, second_row;

  const int b = blockIdx.x, i = threadIdx.x, wave = i >> 6;
  const int row0 = meta.row_start[b], tok0 = meta.tok_start[b], L = meta.block_len[b];
  const bool own = i < MAXL, act = i < L;  // (L <= MAXL)
  float margin = INF;
  // publishes one bit per row: called by every thread, read after the next barrier
  auto publish = [&](Rows& s, bool v) {
    const unsigned long long m = __ballot(v);
    if (own && (i & 63) == 0) s.q[wave] = m;
  };

  float ci = -1.f;
  bool e = false;
  if (act) {
    ci = conf_g[row0 + i];
    lse[i] = lse_g[row0 + i];
    yh[i] = min(max(argmax_g[row0 + i], 0), vocab - 1);  // a caller-supplied prediction outside the vocabulary is clamped into it
    e = tokens[tok0 + i] == mask_id;
  }
  if (own) c[i] = ci;
  publish(s_elig, e);
  for (int k = i; k < L * (WORDS + 1); k += TPB) ((uint32_t*)bits)[k] = 0;
  if (i == 0) { top_row = -1; second_row = -1; }
  bool pool = false, sel = false;
  if (p.mode == 0) {
    if (e) margin = fminf(fabsf(ci - p.tau_low), fabsf(ci - p.tau_high));
    pool = e && ci >= p.tau_low;
    publish(s_pool, pool);
  } else if (p.mode == 1 && e) {
    margin = fabsf(ci - p.tau_high);
    sel = ci >= p.tau_high;
  }
  __syncthreads();

  // a row comes before another in the order of confidence: descending, ties by ascending row.  A wavefront takes every TPB/64-th
  // row against 64 others at a time.
  for (int r = wave; r < L; r += TPB / 64) {
    const float cr = c[r];
    for (int j0 = 0; j0 < L; j0 += 64) {
      const int j = j0 + (i & 63);
      const float cj = c[j];
      const unsigned long long m = __ballot(j < L && (cj > cr || (cj == cr && j < r)));
      if ((i & 63) < 2) ahead[r][(j0 >> 5) + (i & 1)] = (uint32_t)(m >> (32 * (i & 1)));
    }
  }
  __syncthreads();
  uint32_t before[WORDS];  // the rows before this one
  // most confident eligible row and the runner-up (for the safeguard and modes 1, 2)
  int rank = 0;
#pragma unroll
  for (int w = 0; w < WORDS; ++w) {
    before[w] = act && 32 * w < L ? ahead[i][w] : 0;
    rank += __popc(before[w] & s_elig.w[w]);
  }
  if (e && rank == 0) top_row = i;
  if (e && rank == 1) second_row = i;

  if (p.mode == 0) {
    int np = 0, at = 0;  // pooled rows, in ascending order
#pragma unroll
    for (int w = 0; w < RW; ++w) {
      const unsigned long long m = s_pool.q[w];
      if (w < wave) at += __popcll(m);
      else if (w == wave) at += __popcll(m & ((1ull << (i & 63)) - 1));
      np += __popcll(m);
    }
    if (pool) list[at] = i;
    __syncthreads();
    // conflict bit matrix over pooled pairs (Eq. 6), each unordered pair once
    constexpr int U = 4;
    for (int k0 = i; k0 < np * np; k0 += U * TPB) {
      int ra[U], rd[U];
      float za[U], zd[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k = k0 + u * TPB, ka = k / np, kd = k - ka * np;
        const bool ok = k < np * np && ka < kd;
        ra[u] = ok ? list[ka] : -1;
        rd[u] = ok ? list[kd] : -1;
        za[u] = zd[u] = 0.f;
        if (ok) {
          za[u] = to_f32(logits[(size_t)(row0 + ra[u]) * vocab + yh[rd[u]]]);
          zd[u] = to_f32(logits[(size_t)(row0 + rd[u]) * vocab + yh[ra[u]]]);
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        if (ra[u] < 0) continue;
        const float D = (za[u] - lse[ra[u]]) + (zd[u] - lse[rd[u]]);
        margin = fminf(margin, fabsf(D - p.gamma));
        if (D > p.gamma) {
          atomicOr(&bits[ra[u]][rd[u] >> 5], 1u << (rd[u] & 31));
          atomicOr(&bits[rd[u]][ra[u] >> 5], 1u << (ra[u] & 31));
        }
      }
    }
    // phase 1: every pooled row with conf >= tau_high; drop their conflicts from the pool
    const bool high = pool && ci >= p.tau_high;
    publish(s_high, high);
    __syncthreads();
    bool und = pool && !high;
    uint32_t blk[WORDS];  // the row's conflicts; then those of them that come before it in the order
#pragma unroll
    for (int w = 0; w < WORDS; ++w) {
      blk[w] = act ? bits[i][w] : 0;
      und = und && (blk[w] & s_high.w[w]) == 0;
    }
    publish(s_und, und);
    __syncthreads();
    sel = high;
    // the rows phase 2 starts with in their order: the margin includes the smallest step between two different confidences
    int at_und = 0, n_und = 0;
#pragma unroll
    for (int w = 0; w < WORDS; ++w) {
      blk[w] &= before[w] & s_und.w[w];
      at_und += __popc(before[w] & s_und.w[w]);
      n_und += __popc(s_und.w[w]);
    }
    if (und) sorted[at_und] = ci;
    __syncthreads();
    if (und && at_und + 1 < n_und) {
      const float next = sorted[at_und + 1];
      if (next < ci) margin = fminf(margin, ci - next);
    }
    // phase 2.  Every round decides at least the first undecided row of the order, so it ends after at most L of them.
    while (true) {
      unsigned long long left = 0;
#pragma unroll
      for (int w = 0; w < RW; ++w) left |= s_und.q[w];
      if (left == 0) break;  // (uniform: read between two barriers)
      bool take = und;
#pragma unroll
      for (int w = 0; w < WORDS; ++w) take = take && (blk[w] & s_und.w[w]) == 0;
      publish(s_new, take);
      __syncthreads();
      if (take) { sel = true; und = false; }
      if (und) {
#pragma unroll
        for (int w = 0; w < WORDS; ++w) und = und && (bits[i][w] & s_new.w[w]) == 0;
      }
      publish(s_und, und);
      __syncthreads();
    }
  }
  publish(s_sel, sel);
  __syncthreads();
  int n_sel = 0;
#pragma unroll
  for (int w = 0; w < RW; ++w) n_sel += __popcll(s_sel.q[w]);
  if (n_sel == 0 && top_row >= 0) {  // safeguard / top-1 rule: the most confident eligible row
    if (second_row >= 0 && c[top_row] != c[second_row]) margin = fminf(margin, c[top_row] - c[second_row]);
    if (i == top_row) sel = true;
  }
  if (act) {
    sel_out[row0 + i] = sel;
    if (apply && sel) tokens[tok0 + i] = yh[i];
  }
  margin = -wave_max(-margin);
  if ((i & 63) == 0) fbuf[wave] = margin;
  __syncthreads();
  if (i == 0) {
    for (int w = 1; w < TPB / 64; ++w) margin = fminf(margin, fbuf[w]);
    nsel_out[b] = n_sel ? n_sel : (top_row >= 0 ? 1 : 0);
    if (margin_out) margin_out[b] = margin;
  }
}

}  // namespace

template <typename T>
void launch_select(const T* logits, int vocab, const float* lse, const float* conf, const int32_t* argmax, int32_t* tokens,
                        const SelectMeta& meta, int n_seqs, int mask_id, dlm_select_params p, int apply, uint8_t* sel,
                        int32_t* nsel, float* margin, hipStream_t st) {
  int longest = 0;
  for (int b = 0; b < n_seqs; ++b) longest = meta.block_len[b] > longest ? meta.block_len[b] : longest;
  // Up to 32 rows: at most 1024 pairs, one trip of 256 threads; more threads would only make the barriers slower.  Up to 64 rows:
  // sets of two words instead of eight, as most of a short kernel's time is fetching its instructions.  Beyond that 1024 threads, also
  // where no pairs are scored (modes 1, 2): 16 wavefronts for the order's matrix of L x L bits, which with four is the longest part (one
  // sequence, 4 / 16 wavefronts: 65 rows 7.3 / 5.4 us, 128: 11.6 / 5.7, 256: 35.6 / 13.1).
#define GO(TPB, MAXL) \
  select_kernel<T, TPB, MAXL><<<n_seqs, TPB, 0, st>>>(logits, vocab, lse, conf, argmax, tokens, meta, mask_id, p, apply, sel, nsel, margin)
  if (longest > 64) GO(1024, 256);
  else if (longest > 32 && p.mode == 0) GO(1024, 64);
  else GO(256, 64);
#undef GO
}
template void launch_select<float>(const float*, int, const float*, const float*, const int32_t*, int32_t*, const SelectMeta&, int,
                                        int, dlm_select_params, int, uint8_t*, int32_t*, float*, hipStream_t);
template void launch_select<bf16_t>(const bf16_t*, int, const float*, const float*, const int32_t*, int32_t*, const SelectMeta&, int,
                                         int, dlm_select_params, int, uint8_t*, int32_t*, float*, hipStream_t);
