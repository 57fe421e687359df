// Macro-tile GEMM of a bf16 model for passes of more than a block's rows (a block with its look-ahead window, batched decoding,
// prefill): Y[M,N] = X[M,K] * W[N,K]^T, fp32 accumulation, epilogue fused.
//
// A workgroup of RW x CW wavefronts owns a tile of RW WM x CW WN matrix-core fragments (16 rows or columns each) and walks K:
//   * both operands are already stored as 1 KiB matrix-core fragments (16 rows x 32 k), so a stage of the pipeline is just
//     KB (RW WM + CW WN) fragments copied HBM/L2 -> LDS by direct-to-LDS loads (no registers, no LDS writes); S stages of KB
//     k-tiles rotate through up to 152 KiB of LDS;
//   * a wavefront owns WM x WN fragments of the output (fp32 accumulators) and reads its WM + WN operand fragments of the NEXT
//     k-tile from LDS into a second register set while the matrix cores work on the current one;
//   * one barrier per stage, in front of its last k-tile: by then every wavefront has the stage's last fragments in registers,
//     so the copies of stage s + S may overwrite it at once (S - 1 stages stay in flight), and they go out spread over the
//     KB k-tiles that follow;
//   * the waits on the direct-to-LDS loads are counted by hand (every stage is the same number of loads per wavefront; indices
//     past the end are clamped, so the count never varies), and so are the waits on the LDS reads (once per k-tile, behind the
//     products: the compiler counts the copies to LDS as possibly out of order on that counter and could only wait for all);
//   * the epilogue works straight from the accumulators.
// What bounds it: with operands of random values the chip's power limit and the L2 -> LDS fetch rate (16 .. 18 TB/s over the
// chip in this access pattern, loads alone) meet at about half of the published matrix-core rate for every tile from 128 x 128
// up (macro_tiles has the measured time per k-tile of each); below that, the fixed cost of a step.  So a larger tile is no
// faster per product than a 192 x 128 one, and what decides is how evenly the tiles divide the shape over 256 compute units:
// hence many tiles and a planner (gemm_macro.hip) instead of few large ones.  Two k-tiles per stage against one: 192 x 192
// 80 -> 76 us (gate/up of an 8B model at 384 rows), 128 x 128 -10 %; where only two such stages fit (256 x 192, 256 x 256) one
// k-tile per stage is the faster one.
#pragma once
#include <type_traits>

#include "gemm_epilogue.h"
#include "stats_part.h"

// {WM, WN, RW, CW, KB, ns1, ns4}: tile of 16 RW WM rows x 16 CW WN columns; nanoseconds per k-tile on a chip full of such
// workgroups when each streams a W of its own (one row block) and when four or more row blocks share it (operands of random
// values; fitted to 3500 launches of the layer and head matrices of an 8B and a 7B grouped-query model at 24 .. 2822 rows; but the first
// of 64 x 320 and 128 x 320, which serve single row blocks only, to the head of macro_product_only, and their second stands for nothing).
#define MACRO_TILES(X)                                                                                            \
  X(2, 2, 1, 8, 2, 683, 399) X(1, 5, 2, 4, 2, 822, 487) X(2, 5, 2, 4, 2, 823, 823) X(4, 5, 2, 4, 1, 834, 834)   \
  X(2, 1, 2, 4, 2, 174, 130) X(1, 3, 4, 2, 2, 262, 195) X(1, 5, 4, 2, 2, 429, 236) X(2, 4, 2, 4, 2, 696, 330)     \
  X(3, 2, 2, 4, 2, 348, 244) X(3, 4, 2, 4, 2, 706, 395)                                                           \
  X(2, 2, 4, 2, 2, 252, 193) X(2, 3, 4, 2, 2, 301, 232) X(4, 2, 2, 4, 2, 361, 278)                                \
  X(2, 5, 4, 2, 2, 481, 343) X(4, 3, 2, 4, 2, 536, 386) X(4, 4, 2, 4, 2, 714, 466)                                \
  X(5, 2, 2, 4, 2, 432, 338) X(5, 3, 2, 4, 2, 571, 443)                                                           \
  X(3, 3, 4, 2, 2, 389, 322) X(3, 5, 4, 2, 2, 532, 433) X(3, 6, 4, 2, 2, 615, 513)                                \
  X(4, 6, 4, 2, 1, 746, 695) X(4, 8, 4, 2, 1, 922, 831)
// rows:  32 (x 256, 320 columns), 64 (x 64, 96, 160, 256, 320), 96 (x 128, 256), 128 (x 64, 96, 128, 160, 192, 256, 320), 160 (x 128, 192),
//        192 (x 96, 160, 192), 256 (x 192, 256)

// 64 and 128 x 320, for the plain product only: a vocabulary whose 160-column blocks are a little under four rounds and whose 256-column
// ones a little over two takes two of these (head of a 7B model, 152064 columns, in the pass: 64 rows 200 -> 187 us, 96 rows 229 -> 189).  Never
// faster where row blocks share W: the planner leaves them out there.
constexpr bool macro_product_only(int wm, int wn, int cw) { return wm > 1 && wn * cw == 20; }

struct MacroTile {
  int wm, wn, rw, cw, kb;
  float ns1, ns4;
};
struct MacroPlan {
  int tile;  // index into MACRO_TILES
  int nblocks, mblocks, splits, kps;
  int fold;       // k-tiles after which a workgroup starts a second sum, added to the first at the end (0: one sum)
  int ssq_parts;  // EPI_RESID: chunks of the rows' sums of squares per column block (1 or 2)
};
// K is split only where a wavefront has at most this many output fragments: the last arriver holds two tiles of them
constexpr int MACRO_SPLIT_FRAGS = 16;
// tiles that also come with two sums of K, or two chunks of the squares, per workgroup: an instantiation of its own, so that the plain
// kernel keeps its loop and its registers (QKV, 96 x 128: 95 against 124, 128 x 256: 229 against 250)
constexpr bool macro_can_keep_order(int wm, int wn, int kb) { return kb == 2 && wm * wn >= 6 && wm * wn <= MACRO_SPLIT_FRAGS; }

// Tiles that also come with non-temporal copies of W, for launches of one row block (see issue): those with more than one whole round of W.
// With exactly one (96 x 128, 128 x 128, 160 x 128) it depends on the launch, and they are left plain.  Plain / non-temporal, K = 4096: in one
// round of workgroups gate/up of 28672 columns, 80 rows 47.5 / 43.4 us, 112 rows 48.8 / 44.8, 144 rows 55.9 / 52.8, down from 14336, split, 144 rows
// 42.6 / 32.3; in two the head of
// 51200 columns, 144 rows 105.8 / 100.4; in three that of 98304, 70 rows 150.2 / 148.9, 96 rows 149.0 / 154.6 (152064, K = 3584: 229 / 238).
constexpr bool macro_non_temporal(int rw, int cw, int wn) { return cw * wn > rw * cw; }

// gemm_macro_<epilogue>.hip: the launches of one epilogue's instantiations
template <int EPI>
void launch_macro_epi(const op_t* xt, const op_t* wt, int M, int N, int K, const MacroPlan& p, const GemmEpi& e, hipStream_t st);

#ifdef GEMM_MACRO_INSTANTIATE
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int SC1 = 16;  // cache-policy bit of the raw-buffer builtins: device scope
__device__ inline __amdgpu_buffer_rsrc_t part_rsrc(const float* base) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0x7fffffff, 0x00020000);
}

#define GLOBAL_PTR(p) ((const void __attribute__((address_space(1)))*)(p))
#define LDS_PTR(p) ((void __attribute__((address_space(3)))*)(p))

template <int WM, int WN, int RW, int CW, int KB>
struct MacroShape {
  static constexpr int NW = RW * CW, TPB = NW * 64;
  static constexpr int AT = RW * WM, BF = CW * WN;  // X (row) and W (column) fragments of a k-tile
  static constexpr int NFR = AT + BF;
  static constexpr int LPT = (NFR + NW - 1) / NW;   // direct-to-LDS loads per wavefront and k-tile (surplus ones repeat the last fragment)
  static constexpr int LPS = KB * LPT;              // ... and stage
  static constexpr int STAGE = KB * NFR * 1024;
  static constexpr int S_FIT = (152 * 1024) / STAGE, S_CNT = 63 / LPS + 1;  // what LDS holds, and what the memory counter counts
  static constexpr int S_ = S_FIT < S_CNT ? S_FIT : S_CNT;
  static constexpr int S = S_ > 6 ? 6 : S_;
  static constexpr int BODY = S * STAGE;            // (also holds the states of EPI_STATS, CW AT 256 bytes)
  static constexpr int LDS_BYTES = BODY + AT * 16 * 4 * (1 + BF);  // + 1/rms of the rows, sums of squares per row and column tile
  static_assert(S >= 2 && LDS_BYTES <= 160 * 1024, "pipeline shape");
};

// form: bit 0: the weights are packed in interleaved pairs of column tiles, not in single runs (weight_pack_rows - 1); and with ORDER
// bit 1: two chunks of the squares per column block, the other bits: k-tiles after which a second sum starts (0: one sum)
// NT: W is read once (a single row block) and is not kept from pass to pass, so most of its copies are non-temporal (see issue)
template <int WM, int WN, int RW, int CW, int KB, int EPI, bool ORDER, bool NT>
__global__ __launch_bounds__(RW * CW * 64, RW * CW / 4) void gemm_macro_kernel(const op8* __restrict__ xt, const op8* __restrict__ wt, int M, int N, int K,
                                                                               int form, int nblocks, int mblocks, int splits, int kt_per_split, GemmEpi e) {
  typedef MacroShape<WM, WN, RW, CW, KB> SH;
  constexpr int NW = SH::NW, TPB = SH::TPB, AT = SH::AT, BF = SH::BF, NFR = SH::NFR, LPT = SH::LPT, LPS = SH::LPS, STAGE = SH::STAGE, S = SH::S;
  const int prs = ORDER ? form & 1 : form, fold = ORDER ? form >> 2 : 0;
  const bool two_chunks = ORDER && (form & 2);
  extern __shared__ __align__(16) unsigned char lds[];
  float* s_rinv = (float*)(lds + SH::BODY);  // [AT * 16]
  float* s_ssq = s_rinv + AT * 16;           // [BF][AT * 16]
  __shared__ int s_ticket;

  // Workgroup id -> (K split, column block, row block), row blocks fastest.  Ids congruent mod 8 share an XCD: each XCD takes one
  // contiguous eighth of the tiles, so the row blocks of a column block (which stream the same W) meet in one L2 and no XCD has
  // more than its share; with a K split it walks one part of K (or few), so that X's other parts never enter its L2.
  const int tiles = nblocks * mblocks, lin = (blockIdx.x & 7) * ((tiles * splits + 7) >> 3) + (blockIdx.x >> 3);  // (the grid is a multiple of 8)
  if (lin >= tiles * splits) return;
  const int split = lin / tiles, tile = lin - split * tiles, cb = tile / mblocks, rb = tile - cb * mblocks;

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / CW, wn = wave % CW;
  const int KT = K >> 5, MTILES = (M + 15) >> 4, NTILES = N >> 4;
  const int mt0 = rb * AT, nt0 = cb * BF, m_lo = mt0 * 16;
  // the workgroup's k-tiles kb .. kb + nkt - 1; stage s holds k-tiles s KB .. s KB + KB - 1 of them
  const int kb = split * kt_per_split, nkt = min(KT, kb + kt_per_split) - kb, nstages = nkt / KB;

  // Copies lo .. hi - 1 (of this wavefront's LPS) of stage s -> buffer buf: of a k-tile's fragments, one operand's first and then the
  // other's, wavefront w moves the ones congruent w mod NW, in rounds of NW; a wavefront without a fragment of its own in the last round
  // moves the last one again.  The fragments' addresses at the first k-tile are kept, so that a copy costs one scalar shift and one add
  // (recomputing them from the tile indices each time took 3 .. 5 % of a wide launch).
  // Where W is read by one workgroup only, the rounds that are all W (which comes first then) are non-temporal: they do not enter the memory-side cache, in which
  // W does not stay from pass to pass unless the model is small (WEIGHTS_CACHED_BYTES; a plain read of HBM 6.2 -> 7.1 TB/s; the LM head of the 8B model, 8 rows 180 -> 158 us, 96 rows 196 ->
  // 185).  Where row blocks share W it loses what the L2 keeps for the second of them (two readers of a stream 5.1 -> 4.7 TB/s, four 3.6 ->
  // 2.9), and so does a fragment that several wavefronts move.
  constexpr bool W_FIRST = macro_non_temporal(RW, CW, WN);
  constexpr int FIRST_OP = W_FIRST ? BF : AT;
  static_assert(W_FIRST || !NT, "whole rounds of W come first");
  const unsigned lane16 = lane * 16;
  const char* fbase[LPT];
#pragma unroll
  for (int i = 0; i < LPT; ++i) {
    const int f = min(i * NW + wave, NFR - 1), fw = W_FIRST ? f : f - AT, fx = W_FIRST ? f - BF : f;
    const int ntile = min(nt0 + max(fw, 0), NTILES - 1), mtile = min(mt0 + max(fx, 0), MTILES - 1);
    fbase[i] = (W_FIRST ? fx >= 0 : fw < 0) ? (const char*)xt + ((size_t)mtile * KT + kb) * 1024
                                            : (const char*)wt + ((((size_t)(ntile >> prs) * KT + kb) << prs) + (ntile & prs)) * 1024;
  }
  auto issue = [&](int s, int buf, int lo, int hi) __attribute__((always_inline)) {
#pragma unroll
    for (int c = lo; c < hi; ++c) {
      const int sub = c / LPT, i = c % LPT, f = min(i * NW + wave, NFR - 1);
      const unsigned t = min(s * KB + sub, nkt - 1);
      const bool first = FIRST_OP % NW == 0 ? i < FIRST_OP / NW : f < FIRST_OP, is_x = first != W_FIRST;  // (uniform in the wavefront)
      const char* src = fbase[i] + (is_x ? t << 10 : t << (10 + prs));
      unsigned char* dst = lds + buf * STAGE + (sub * NFR + (!W_FIRST ? f : first ? AT + f : f - BF)) * 1024;  // (X lies in front)
      if (NT && (i + 1) * NW <= BF) __builtin_amdgcn_global_load_lds(GLOBAL_PTR(src + lane16), LDS_PTR(dst), 16, 0, 2);
      else __builtin_amdgcn_global_load_lds(GLOBAL_PTR(src + lane16), LDS_PTR(dst), 16, 0, 0);
    }
  };

  f32x4 acc[WN][WM];
#pragma unroll
  for (int j = 0; j < WN; ++j)
#pragma unroll
    for (int i = 0; i < WM; ++i) acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
  op8 xf[2][WM], wf[2][WN];
  auto read_frags = [&](int set, int buf, int sub) __attribute__((always_inline)) {
    const op8* st = (const op8*)(lds + buf * STAGE + sub * NFR * 1024) + lane;
#pragma unroll
    for (int i = 0; i < WM; ++i) xf[set][i] = st[(wm * WM + i) * 64];
#pragma unroll
    for (int j = 0; j < WN; ++j) wf[set][j] = st[(AT + wn * WN + j) * 64];
  };
  auto multiply = [&](int set) __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
      for (int i = 0; i < WM; ++i) acc[j][i] = mfma_op(wf[set][j], xf[set][i], acc[j][i]);
  };

  // EPI_RESID: residual and gain of the outputs are fetched here too where the registers hold them (only this workgroup touches them);
  // of a split tile by the workgroup that finishes it, while it waits for the others
  constexpr bool H_EARLY = EPI == EPI_RESID && (ORDER ? 12 : 10) * WM * WN + 8 * (WM + WN) <= 200;
  f32x4 h_ahead[WN][WM], g_ahead[WN];
  auto fetch_resid = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int j = 0; j < WN; ++j) {
      const int n = min(nt0 + wn * WN + j, NTILES - 1) * 16 + 4 * (lane >> 4);
      g_ahead[j] = *(const f32x4*)(e.gain + n);
#pragma unroll
      for (int i = 0; i < WM; ++i) h_ahead[j][i] = *(const f32x4*)(e.h + (size_t)min(m_lo + (wm * WM + i) * 16 + (lane & 15), M - 1) * N + n);
    }
  };
  // The first stage's copies go out before anything is read from memory (the arguments in front of e arrive in registers), then what
  // the epilogue reads, then the other stages: the wait for the first stage waits for these loads too, whatever their number.  Not where
  // 1/rms has to be published in front of the loop, for which the compiler waits for every load in flight.
  typedef RinvBatch<TPB, AT * 16> Rinv;
  constexpr bool RINV_LATE = 4 * WM * WN + 8 * (WM + WN) + 4 * Rinv::RPT <= 210;
  constexpr bool FIRST = EPI == EPI_RESID || RINV_LATE;
  if (FIRST) {
    issue(0, 0, 0, LPS);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (H_EARLY && splits == 1) fetch_resid();

  // K split: a ticket per workgroup and tile, taken here, where its trip to memory hides behind the pipeline's start
  int my_ticket = 0;
  if constexpr (WM * WN <= MACRO_SPLIT_FRAGS) {
    if (splits > 1 && tid == 0) my_ticket = __hip_atomic_fetch_add(e.counters + 2 * tile, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }

  // 1/rms of the workgroup's input rows, needed only by the epilogue: fetched behind the first stage's copies and ahead of the others, in one
  // trip where a row has up to 64 chunks (wide passes).  Where the registers hold what was fetched, it stays there until the loop is over (touching
  // it while copies to LDS are in flight would make the compiler wait for all of them); published to the other wavefronts by
  // the barrier of the epilogue, or by the loop's.
  const int rows = max(0, min(M, m_lo + AT * 16) - m_lo);
  const bool rinv_batched = EPI != EPI_RESID && Rinv::fits(e.rs);
  Rinv rinv;
  if (EPI != EPI_RESID) {
    if (rinv_batched) {
      rinv.fetch(e.rs, m_lo, rows);
      if (!RINV_LATE) rinv.publish(e.rs, rows, s_rinv);
    } else {
      block_rinv<TPB>(e.rs, m_lo, rows, s_rinv);
    }
  }

  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int s = FIRST ? 1 : 0; s < S - 1; ++s) issue(s, s, 0, LPS);
  issue(S - 1, S - 1, 0, LPS / KB);  // (the rest of it goes out during stage 0, as for every later stage)
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S - 2) * LPS + LPS / KB) : "memory");  // stage 0 has landed (this wavefront's share)
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
  read_frags(0, 0, 0);
  __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): as at the end of every k-tile below
  // K-tile SUB of stage s (in LDS buffer buf), whose operands are in register set `set`; stages up to s + S - 1 have been issued
  auto ktile = [&](auto SUBc, int set, int s, int buf, int nbuf) __attribute__((always_inline)) {
    constexpr int SUB = decltype(SUBc)::value;
    constexpr bool LAST = SUB == KB - 1;
    constexpr int LO = LAST ? 0 : LPS * (SUB + 1) / KB, HI = LAST ? LPS / KB : LPS * (SUB + 2) / KB;
    if (LAST) {
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"((S - 2) * LPS) : "memory");  // stage s + 1 has landed
      __builtin_amdgcn_s_barrier();  // ... for every wavefront, and every wavefront has read the last of stage s
      asm volatile("" ::: "memory");
    }
    __builtin_amdgcn_sched_barrier(0);
    if (LAST) issue(s + S, buf, LO, HI);
    else issue(s + S - 1, buf == 0 ? S - 1 : buf - 1, LO, HI);
    if (LAST) read_frags(set ^ 1, nbuf, 0);
    else read_frags(set ^ 1, buf, SUB + 1);
    multiply(set);
    // Issue order, fixed by hand: the products (which depend on registers only) start right away, and the copies and the LDS
    // reads of the next k-tile go out between them.  Left alone, the scheduler puts the reads next to their uses, and all
    // wavefronts of a SIMD, which leave the barrier together, would issue their loads while its matrix core idles.
    constexpr int NM = WN * WM, RF = WM + WN, LI = HI - LO;
    constexpr int OPS = 2 * (LI + RF) <= NM ? 1 : LI + RF <= NM ? 2 : 4;  // copies / reads per product: out by the middle of the products where they are many enough
    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
#pragma unroll
    for (int i = 0; i < LI; i += OPS) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);    // one product
      __builtin_amdgcn_sched_group_barrier(0x010, OPS, 0);  // copies to LDS
    }
#pragma unroll
    for (int i = 0; i < RF; i += OPS) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, OPS, 0);  // LDS reads
    }
    __builtin_amdgcn_sched_group_barrier(0x008, NM, 0);  // what is left of the products
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(0xc07f);  // lgkmcnt(0): the reads have had the products' time to complete
  };
  // two k-tiles per trip, unconditionally: a fragment read that is used only behind a branch would be moved behind it, next to
  // its use, and the matrix cores would wait for LDS
  static_assert(KB == 1 || KB == 2, "k-tiles per stage");
  int buf = 0;
  auto next = [&](int b) { return b + 1 == S ? 0 : b + 1; };
  if constexpr (KB == 2 && !ORDER) {
    for (int s = 0; s < nstages; ++s, buf = next(buf)) {
      ktile(std::integral_constant<int, 0>{}, 0, s, buf, next(buf));
      ktile(std::integral_constant<int, 1>{}, 1, s, buf, next(buf));
    }
    if (nkt & 1) multiply(0);  // the odd last k-tile: its operands were read with the stage before it
  } else if constexpr (KB == 2) {
    int s = 0;
    auto walk = [&](int end) __attribute__((always_inline)) {
      for (; s < end; ++s, buf = next(buf)) {
        ktile(std::integral_constant<int, 0>{}, 0, s, buf, next(buf));
        ktile(std::integral_constant<int, 1>{}, 1, s, buf, next(buf));
      }
    };
    walk(fold ? fold / KB : nstages);
    if (!fold) {
      if (nkt & 1) multiply(0);
    } else {  // (uniform) a second sum: what a K split over two workgroups adds, in the same order, without the hand-off
      f32x4 first[WN][WM];
#pragma unroll
      for (int j = 0; j < WN; ++j)
#pragma unroll
        for (int i = 0; i < WM; ++i) {
          first[j][i] = acc[j][i];
          acc[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
      walk(nstages);
      if (nkt & 1) multiply(0);
#pragma unroll
      for (int j = 0; j < WN; ++j)
#pragma unroll
        for (int i = 0; i < WM; ++i) acc[j][i] = first[j][i] + acc[j][i];
    }
  } else {
    int s = 0;
    for (; s + 1 < nstages; s += 2) {
      ktile(std::integral_constant<int, 0>{}, 0, s, buf, next(buf));
      buf = next(buf);
      ktile(std::integral_constant<int, 0>{}, 1, s + 1, buf, next(buf));
      buf = next(buf);
    }
    if (s < nstages) ktile(std::integral_constant<int, 0>{}, 0, s, buf, next(buf));
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // the surplus loads of the last stages: LDS must be quiet before it is reused

  const int g = lane >> 4, ml = lane & 15;
  if constexpr (WM * WN <= MACRO_SPLIT_FRAGS) if (splits > 1) {
    // K split (shapes whose tiles cover less than the chip).  The workgroup that took a tile's last ticket finishes it; the others
    // write their partial tile to the fp32 workspace, whole fragments in the accumulator layout, and then raise the tile's count
    // of finished partials.  The last one keeps its own in registers, waits for that count (every workgroup it waits for took its
    // ticket before, so it is running and finishes without waiting for anyone), adds the partial tiles in split order, its own in
    // its place (deterministic whoever is last), and runs the epilogue.
    // The hand-off crosses XCDs, whose L2s are separate.  Partials and counts are written and read at device scope themselves (SC1;
    // relaxed atomics), and a wavefront waits for the acknowledgement of its stores before the barrier in front of the count, so
    // neither side needs a fence: a release would write back the L2's dirty lines and an acquire drop its clean ones, under
    // the feet of the workgroups that still multiply.  From the end of the loop to the epilogue 10 us with fences, tickets taken
    // behind the loop and row-major partials (half lines), 3 to 4 now: down of an 8B model at 384 rows 71 -> 62 us.
    const unsigned slot = (unsigned)(AT * BF) * 256;  // floats of a tile's partial
    auto offset = [&](int j, int i) { return (unsigned)((((wm * WM + i) * BF + wn * WN + j) * 64 + lane) * 16); };
    auto exists = [&](int j, int i) { return nt0 + wn * WN + j < NTILES && mt0 + wm * WM + i < MTILES; };  // (uniform in the wavefront)
    int* ticket = e.counters + 2 * tile;
    if (tid == 0) s_ticket = my_ticket;
    __syncthreads();
    if (s_ticket != splits - 1) {
      const __amdgpu_buffer_rsrc_t mine = part_rsrc(e.part + (size_t)(split * tiles + tile) * slot);
#pragma unroll
      for (int j = 0; j < WN; ++j)
#pragma unroll
        for (int i = 0; i < WM; ++i)
          if (exists(j, i)) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[j][i]), mine, offset(j, i), 0, SC1);
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if (tid == 0) (void)__hip_atomic_fetch_add(ticket + 1, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return;
    }
    if (H_EARLY) fetch_resid();
    if (tid == 0) {
      while (__hip_atomic_load(ticket + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) != splits - 1) __builtin_amdgcn_s_sleep(1);
      __hip_atomic_store(ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // ready for the next launch
      __hip_atomic_store(ticket + 1, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    asm volatile("" ::: "memory");
    f32x4 sum[WN][WM];
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
      for (int i = 0; i < WM; ++i) sum[j][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int s0 = 0; s0 < splits; ++s0) {
      if (s0 == split) {
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
          for (int i = 0; i < WM; ++i) sum[j][i] += acc[j][i];
        continue;
      }
      const __amdgpu_buffer_rsrc_t theirs = part_rsrc(e.part + (size_t)(s0 * tiles + tile) * slot);
      u32x4 t[WN][WM];
#pragma unroll
      for (int j = 0; j < WN; ++j)
#pragma unroll
        for (int i = 0; i < WM; ++i) t[j][i] = __builtin_amdgcn_raw_buffer_load_b128(theirs, exists(j, i) ? offset(j, i) : 0u, 0, SC1);
#pragma unroll
      for (int j = 0; j < WN; ++j)
#pragma unroll
        for (int i = 0; i < WM; ++i) sum[j][i] += __builtin_bit_cast(f32x4, t[j][i]);
    }
#pragma unroll
    for (int j = 0; j < WN; ++j)
#pragma unroll
      for (int i = 0; i < WM; ++i) acc[j][i] = sum[j][i];
  }

  // ---- epilogue, straight from the accumulators.  What bounds it is the instructions it issues, then the trips to memory of what
  // it reads: so every lane finishes outputs of its own, values move between lanes by permlane and DPP, and loads go out ahead
  // of the stores before them (the memory counter retires in order).  From the end of the loop to the end of the kernel, 8B model
  // at 384 rows, with fragments staged through LDS, exchanged there and finished by half of the lanes / now: QKV 8.3 / 5.1 us,
  // gate/up 8.8 / 3.9, down (the finishing workgroup) 5.0 / 2.2, a 256 x 256 gate/up tile 9.1 / 4.2.
  if (RINV_LATE && rinv_batched) rinv.publish(e.rs, rows, s_rinv);
  if (EPI != EPI_RESID) __syncthreads();
  float ri[WM];  // 1/rms of the lane's row of each row tile
#pragma unroll
  for (int i = 0; i < WM; ++i) ri[i] = EPI == EPI_RESID ? 1.f : s_rinv[(wm * WM + i) * 16 + ml];
  const int nt_w = nt0 + wn * WN, mt_w = mt0 + wm * WM;  // the wavefront's first column and row tile
  const bool hi = lane >= 32;
  auto row = [&](int i) { return (mt_w + i) * 16 + ml; };
  if constexpr (EPI == EPI_SWIGLU) {
    // two fragments at a time (column tiles fastest): the lower 32 lanes finish the first's outputs, the upper ones the second's
    constexpr int F = WM * WN;
#pragma unroll
    for (int f = 0; f < F; f += 2) {
      const int f1 = f + 1 < F ? f + 1 : f, i0 = f / WN, j0 = f % WN, i1 = f1 / WN, j1 = f1 % WN;
      const bool there = hi ? (f1 != f && nt_w + j1 < NTILES && row(i1) < M) : (nt_w + j0 < NTILES && row(i0) < M);
      const Halves v = pair_halves(acc[j0][i0], acc[j1][i1]);
      const float r = hi ? ri[i1] : ri[i0];
      const int second = i1 == i0 ? 128 * (j1 - j0) : 16 * e.ffn + 128 * (j1 - j0);  // from the first fragment's outputs to the second's
      op_t* dst = e.act + ((size_t)(mt_w + i0) * e.ffn * 16 + (size_t)(nt_w + j0) * 128) + ((hi ? second : 0) + ml * 8 + 4 * (g & 1));
      if (there) *(op4*)dst = to_f16x4_sat(gated(v.lo * r, v.hi * r));
    }
  } else if constexpr (EPI == EPI_QKV) {
    const int hd = e.hd, tph = hd >> 4, half = hd >> 1, heads_rot = e.n_q + e.n_kv;
    constexpr int PR = (WM + 1) / 2;  // pairs of row tiles of a column tile: rotated two at a time, the lower lanes the first's outputs
    int pos[WM], slot[WM];
    if ((min(nt_w + WN, NTILES) - 1) / tph >= e.n_q) {
#pragma unroll
      for (int i = 0; i < WM; ++i) {
        const int m = min(row(i), M - 1);
        pos[i] = e.row_pos[m];
        slot[i] = e.row_slot[m];
      }
    }
    f32x4 rc[2][PR], rsn[2][PR];  // rotary cosines and sines of a column tile's pairs: the next tile's are in flight
    auto fetch_rope = [&](int j) __attribute__((always_inline)) {
      const int nt = nt_w + j;
      if (nt >= NTILES || nt / tph >= heads_rot) return;
#pragma unroll
      for (int p = 0; p < PR; ++p) {
        const int m = min(row(2 * p + (hi && 2 * p + 1 < WM)), M - 1);
        const size_t o = (size_t)m * half + 8 * (nt % tph) + 4 * (g & 1);
        rc[j & 1][p] = *(const f32x4*)(e.rope_cos + o);
        rsn[j & 1][p] = *(const f32x4*)(e.rope_sin + o);
      }
    };
    fetch_rope(0);
#pragma unroll
    for (int j = 0; j < WN; ++j) {
      if (j + 1 < WN) fetch_rope(j + 1);
      const int nt = nt_w + j, head = nt / tph, bt = nt % tph;  // (uniform)
      if (nt >= NTILES) continue;
      if (head < heads_rot) {
#pragma unroll
        for (int p = 0; p < PR; ++p) {
          const int i0 = 2 * p, i1 = 2 * p + 1 < WM ? 2 * p + 1 : i0, i = hi ? i1 : i0;
          const Halves v = pair_halves(acc[j][i0], acc[j][i1]);
          const float r = hi ? ri[i1] : ri[i0];
          const f32x4 x = v.lo * r, y = v.hi * r, c = rc[j & 1][p], sn = rsn[j & 1][p];
          // the lane's four dims 4 (g & 1) .. of the tile's eight, and their partners half a head up; then eight consecutive dims
          // per lane: even lane groups the tile's, odd ones their partners
          const op8 o = join_slots(to_f16x4_sat(x * c - y * sn), to_f16x4_sat(y * c + x * sn));
          const int m = row(i), d = 8 * bt + ((g & 1) ? half : 0);
          if (m < M && !(hi && i1 == i0)) {
            if (head < e.n_q) {
              *(op8*)(e.q + ((size_t)(mt_w + i) * e.n_q * hd + head * hd + d) * 16 + ml * 8) = o;
            } else {
              const size_t region = (size_t)(hi ? slot[i1] : slot[i0]) * e.slot_stride + (size_t)(head - e.n_q) * e.head_stride;
              *(op8*)(e.kcache + region + kv_k_index(hi ? pos[i1] : pos[i0], d, hd)) = o;
            }
          }
        }
      } else {
#pragma unroll
        for (int i = 0; i < WM; ++i) {
          // V keeps eight positions of a dim together: 4 x 4 transposed within each quad of lanes, so that a lane has one dim of the
          // quad's four rows; one store where these are four aligned positions of one sequence, four of one value each elsewhere
          const op4 t = transpose_quad(to_f16x4_sat(acc[j][i] * ri[i]));
          const int d = ((g & 2) ? half : 0) + 8 * bt + 4 * (g & 1) + (ml & 3), m_quad = row(i) & ~3;
          int qp[4], qs[4];
          quad_rows(pos[i], qp);
          quad_rows(slot[i], qs);
          f16_t* v = e.vcache + (size_t)(head - heads_rot) * e.head_stride;
          if ((qp[0] & 3) == 0 && qp[3] == qp[0] + 3 && qs[3] == qs[0] && m_quad + 3 < M) {
            *(op4*)(v + (size_t)qs[0] * e.slot_stride + kv_v_index(qp[0], d, hd)) = t;
          } else {
#pragma unroll
            for (int k = 0; k < 4; ++k)
              if (m_quad + k < M) v[(size_t)qs[k] * e.slot_stride + kv_v_index(qp[k], d, hd)] = t[k];
          }
        }
      }
    }
  } else if constexpr (EPI == EPI_RESID) {
    // (without H_EARLY) residual and gain of a column tile: the next three tiles' are in flight (one: O of an 8B model at 2048 rows 73.0 us
    // against 71.3)
    constexpr int RING = 4;
    f32x4 hc[RING][WM], gc[RING];
    auto fetch_col = [&](int j) __attribute__((always_inline)) {
      if (nt_w + j >= NTILES) return;
      gc[j % RING] = *(const f32x4*)(e.gain + (nt_w + j) * 16 + 4 * g);
#pragma unroll
      for (int i = 0; i < WM; ++i) hc[j % RING][i] = *(const f32x4*)(e.h + (size_t)min(row(i), M - 1) * N + (nt_w + j) * 16 + 4 * g);
    };
    if (!H_EARLY)
#pragma unroll
      for (int j = 0; j < RING - 1 && j < WN; ++j) fetch_col(j);
#pragma unroll
    for (int j = 0; j < WN; ++j) {
      if (!H_EARLY && j + RING - 1 < WN) fetch_col(j + RING - 1);
      const int nt = nt_w + j;
#pragma unroll
      for (int i = 0; i < WM; ++i) {
        const int m = row(i);
        float ss = 0.f;  // (a column tile that does not exist adds nothing)
        if (m < M && nt < NTILES) ss = finish_resid(e, m, nt * 16 + 4 * g, N, acc[j][i], EpiAhead{H_EARLY ? h_ahead[j][i] : hc[j % RING][i], H_EARLY ? g_ahead[j] : gc[j % RING], true, -1, -1});
        ss = sum_row4(ss);
        if (g == 0) s_ssq[(wn * WN + j) * AT * 16 + (wm * WM + i) * 16 + ml] = ss;
      }
    }
  } else if constexpr (EPI != EPI_STATS) {  // the product in bf16: two column tiles at a time, eight consecutive columns per lane
#pragma unroll
    for (int i = 0; i < WM; ++i) {
      const int m = row(i);
      bf16_t* out = e.out_bf16 + (size_t)m * N + nt_w * 16;
#pragma unroll
      for (int j = 0; j < WN; j += 2) {
        if (j + 1 < WN && nt_w + j + 1 < NTILES) {
          const bf16x8 o = join_slots(to_bf16x4(acc[j][i] * ri[i]), to_bf16x4(acc[j + 1 < WN ? j + 1 : j][i] * ri[i]));
          if (m < M) *(bf16x8*)(out + (j + (g & 1)) * 16 + 8 * (g >> 1)) = o;
        } else if (nt_w + j < NTILES && m < M) {
          *(bf16x4*)(out + j * 16 + 4 * g) = to_bf16x4(acc[j][i] * ri[i]);
        }
      }
    }
  }
  LiteState state[WM];  // EPI_STATS: the logits, and the states of their values as written
  if constexpr (EPI == EPI_STATS) {
#pragma unroll
    for (int i = 0; i < WM; ++i) {
      state[i] = lite_init();
#pragma unroll
      for (int j = 0; j < WN; ++j) {
        const int m = row(i), n = (nt_w + j) * 16 + 4 * g;
        if (nt_w + j >= NTILES) continue;
        const f32x4 v = acc[j][i] * ri[i];
        if (m < M) *(bf16x4*)(e.out_bf16 + (size_t)m * N + n) = to_bf16x4(v);
        state[i] = lite_merge(state[i], lite_of(v, n, e.skip_col));
      }
    }
  }
  if (EPI == EPI_STATS) {  // one state per row: the four lanes of a row, then the wavefronts' column ranges, each in a fixed order
    LiteState* s_state = (LiteState*)lds;  // [CW][AT * 16]
    __syncthreads();
#pragma unroll
    for (int i = 0; i < WM; ++i) {
      state[i] = lite_merge(state[i], lite_from(state[i], 16));  // (of the lanes' groups 0 and 2, then of group 0)
      state[i] = lite_merge(state[i], lite_from(state[i], 32));
      if (g == 0) s_state[wn * AT * 16 + (wm * WM + i) * 16 + ml] = state[i];
    }
    __syncthreads();
    for (int r = tid; r < AT * 16 && m_lo + r < M; r += TPB) {
      LiteState t = s_state[r];
#pragma unroll
      for (int c = 1; c < CW; ++c) t = lite_merge(t, s_state[c * AT * 16 + r]);
      f32x4* dst = (f32x4*)((Part*)e.stat_parts + (size_t)(m_lo + r) * nblocks + cb);  // Part{m, s, t, w = 0, bv = m, bi, pm, ps = 0}
      static_assert(sizeof(Part) == 32 && offsetof(Part, bv) == 16 && offsetof(Part, bi) == 20, "Part is written as two vectors");
      dst[0] = f32x4{t.m, t.s, t.t, 0.f};
      dst[1] = f32x4{t.m, __int_as_float(t.bi), NEG_BIG, 0.f};
    }
  }
  if (EPI == EPI_RESID) {  // the workgroup's share of sum h^2 per row, in one chunk or two: each half of its column tiles in ascending order, then the two
    __syncthreads();
    const bool two = two_chunks && BF % 4 == 0;
    const int nch = two ? (NTILES + BF / 2 - 1) / (BF / 2) : nblocks;
    for (int r = tid; r < AT * 16 && m_lo + r < M; r += TPB) {
      float* dst = e.ssq_out + (size_t)(m_lo + r) * nch + (two ? cb * 2 : cb);
      if (!two) {
        float ss[2] = {0.f, 0.f};
#pragma unroll
        for (int j = 0; j < BF; ++j) ss[j >= BF / 2] += s_ssq[j * AT * 16 + r];
        dst[0] = ss[0] + ss[1];
      } else {
        float ss[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < BF; ++j) ss[j / ((BF + 3) / 4)] += s_ssq[j * AT * 16 + r];
        dst[0] = ss[0] + ss[1];
        if (cb * 2 + 1 < nch) dst[1] = ss[2] + ss[3];
      }
    }
  }
}

template <int WM, int WN, int RW, int CW, int KB, int EPI, bool ORDER, bool NT>
void launch_tile(const op_t* xt, const op_t* wt, int M, int N, int K, const MacroPlan& p, const GemmEpi& e, hipStream_t st) {
  typedef MacroShape<WM, WN, RW, CW, KB> SH;
  static bool configured = false;  // raise the dynamic LDS limit of this instantiation once
  if (!configured) {
    (void)hipFuncSetAttribute((const void*)gemm_macro_kernel<WM, WN, RW, CW, KB, EPI, ORDER, NT>, hipFuncAttributeMaxDynamicSharedMemorySize, SH::LDS_BYTES);
    configured = true;
  }
  const int grid = (p.nblocks * p.mblocks * p.splits + 7) / 8 * 8;
  DLM_LAUNCH((gemm_macro_kernel<WM, WN, RW, CW, KB, EPI, ORDER, NT>), grid, SH::TPB, SH::LDS_BYTES, st, (const op8*)xt, (const op8*)wt, M, N, K,
             (weight_pack_rows(N) - 1) | (p.ssq_parts == 2 ? 2 : 0) | p.fold << 2, p.nblocks, p.mblocks, p.splits, p.kps, e);
}

}  // namespace

template <int EPI>
void launch_macro_epi(const op_t* xt, const op_t* wt, int M, int N, int K, const MacroPlan& p, const GemmEpi& e, hipStream_t st) {
  int i = 0;
#define GO(WM, WN, RW, CW, KB, NS1, NS4)                                                                                       \
  if constexpr ((EPI != EPI_STATS || 16 * WM * RW <= GEMM_STATS_MAX_ROWS) && !(macro_product_only(WM, WN, CW) && EPI != EPI_STATS && EPI != EPI_SUM)) {                                                     \
    if constexpr (EPI != EPI_STATS && macro_can_keep_order(WM, WN, KB)) {                                                      \
      if (p.tile == i && (p.fold || p.ssq_parts > 1)) return launch_tile<WM, WN, RW, CW, KB, EPI, true, false>(xt, wt, M, N, K, p, e, st); \
    }                                                                                                                          \
    if constexpr (macro_non_temporal(RW, CW, WN)) {                                                                            \
      if (p.tile == i && p.mblocks == 1 && !e.w_cached) return launch_tile<WM, WN, RW, CW, KB, EPI, false, true>(xt, wt, M, N, K, p, e, st);  \
    }                                                                                                                          \
    if (p.tile == i) return launch_tile<WM, WN, RW, CW, KB, EPI, false, false>(xt, wt, M, N, K, p, e, st);                    \
  }                                                                                                                            \
  ++i;
  MACRO_TILES(GO)
#undef GO
}
#endif  // GEMM_MACRO_INSTANTIATE
