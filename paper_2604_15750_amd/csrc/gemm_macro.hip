// Macro-tile GEMM: which tile and K split serves a shape (the kernel is in gemm_macro_kernel.h).
#include "gemm_macro_kernel.h"

namespace {

#define ROW(WM, WN, RW, CW, KB, NS1, NS4) {WM, WN, RW, CW, KB, NS1, NS4},
const MacroTile g_tiles[] = {MACRO_TILES(ROW)};
#undef ROW
constexpr int CUS = 256, MAX_SPLITS = 4, MAX_SPLIT_TILES = 1024;

// The order of the sums of a wide launch: whether K is summed in one part or two, and how many 16-column tiles a chunk of the rows'
// sums of squares has.  Another order moves the last bits of everything downstream, and with them the confidences of the narrow
// passes that read a wide pass's cache: an exponential of a bf16 logit jumps by 6 or 12 % where the logit's rounding flips (in-block
// passes of 8 .. 37 rows behind prefills of 512 .. 1756 rows, 48 trials: the confidences moved by up to 3.7 % in the 2-norm).  So from
// 32 row tiles (497 rows) on the order is a function of the shape alone, apart from the choice of the tile and of the workgroups:
// the constants below say which order a shape has; they are no timings of this kernel's tiles.  Shapes for which they ask for more
// than two parts are left out: there the order is the plan's (the down projections of an 8B model at 513 .. 640 and 1025 .. 1280 rows,
// of a 7B one at 513 .. 1024 and 1153 .. 1536).
struct SumOrder {
  bool fixed;
  int splits, bt;
};
SumOrder sum_order(int mt, int N, int K, bool may_split) {
  // rows x columns; weight of a product; of two workgroups, and of one, that share a compute unit
  const struct { int bm, bn; double rel, pair, single; } tiles[] = {{256, 256, 0.63, 0, 0}, {128, 256, 1.0, 1.45, 1.15}, {128, 128, 0.96, 1.83, 1.12},
                                                                    {192, 256, 0.86, 0, 0}, {256, 192, 0.72, 0, 0},      {192, 192, 0.83, 0, 0}};
  const int M = mt * 16, KT = K >> 5;
  SumOrder best{false, 1, 1};
  double best_us = 1e300;
  for (auto& t : tiles) {
    const int n = ((M + t.bm - 1) / t.bm) * ((N + t.bn - 1) / t.bn);
    int sp = may_split ? CUS / n : 1;
    if (sp > MAX_SPLITS) sp = MAX_SPLITS;
    if (sp > KT / 32) sp = KT / 32;
    if (sp < 1) sp = 1;
    const int kps = (KT + sp - 1) / sp;
    sp = (KT + kps - 1) / kps;
    const int rounds = (n * sp + CUS - 1) / CUS;
    const double turns = t.pair > 0 && rounds >= 2 ? (rounds / 2) * t.pair + (rounds & 1) * t.single : rounds;
    const double us = turns * t.bm * t.bn * t.rel * K * 6.2e-7 / sp + (sp > 1 ? (double)n * sp * t.bm * t.bn * 3.2e-6 : 0.0) + (sp > 2 ? 4.0 * (sp - 2) : 0.0);
    if (us < best_us) { best_us = us; best = SumOrder{mt >= 32 && sp <= 2, sp, t.bn / 16}; }
  }
  return best;
}

// The tile and K split with the least estimated time, in microseconds.  A round is what 256 compute units take together, one
// workgroup each (the pipeline's stages fill a unit's LDS).  Its k-tiles take the tile's measured time, between ns1 and ns4 by
// the number of row blocks that share W; a chip that is partly full runs its workgroups up to a third faster.  Every round pays
// its pipeline's start and its epilogue (QKV most: rotary embedding and scattered cache writes).  A K split, for launches that
// leave compute units idle, adds the hand-off and the partial tiles' traffic.  M enters only through its 16-row tiles.
// The round's and the hand-off's terms (round_us, 4.6 + 0.6 ..) and the tiles' times were fitted to the kernel with a fenced hand-off and
// epilogues staged through LDS, against which the choice lost 0.7 % to the best candidate over 220 shapes; they are not refitted, and now
// charge splits and rounds too much.  On the present kernel, 127 shapes of both models' layers from 72 to 1024 rows, it loses 3.7 %:
// nothing for gate/up from 208 rows on and QKV of the 8B model from 336, most for O at 264 .. 384 rows (27.9 us, 24.0 with a two-way split),
// QKV of the 7B one at 208 .. 304 (25.0 / 20.9), down of the 8B one at 248 (54.6 / 42.7).  Below 497 rows the order of the sums is free.
// Where the order of the sums is fixed, two parts of K are either a split over two workgroups (as long as all of them are one
// round) or one workgroup that keeps two sums (fold), and a chunk of the squares is a column block or half of one; the tile is free.
// With the split and the block width pinned as well, narrow matrices ran a second round: O of an 8B model at 2048 rows 90 us against
// 74 now, its down 230 / 179, QKV of a 7B model at 945 rows 89 / 48, O of the 8B one at 512 rows 44 / 37.
MacroPlan macro_plan(int M, int N, int K, int kind) {
  MacroPlan best{0, 1, 1, 1, 1, 0, 1};
  double best_us = 1e300;
  int best_full = 0;  // whole rounds before the last
  const bool may_split = kind != EPI_DIRECT && kind != EPI_STATS;  // the LM head's epilogues have no workspace
  const double round_us = kind == EPI_QKV ? 5.6 : kind == EPI_RESID ? 4.3 : kind == EPI_SWIGLU ? 1.8 : 3.4;
  const int KT = K >> 5, mt = (M + 15) >> 4, nt = N >> 4;
  SumOrder order = sum_order(mt, N, K, may_split);
  for (;; order.fixed = false) {
    int c = -1;
    for (const MacroTile& t : g_tiles) {
      ++c;
      if (kind == EPI_STATS && 16 * t.rw * t.wm > GEMM_STATS_MAX_ROWS) continue;  // (not instantiated)
      const int at = t.rw * t.wm, bt = t.cw * t.wn, mb = (mt + at - 1) / at, nb = (nt + bt - 1) / bt, tiles = mb * nb;
      // (never faster where row blocks share W, and not instantiated for the layer's epilogues)
      if (macro_product_only(t.wm, t.wn, t.cw) && (mb > 1 || !(kind == EPI_DIRECT || kind == EPI_STATS || kind == EPI_SUM))) continue;
      const int parts = order.fixed && kind == EPI_RESID && bt == 2 * order.bt ? 2 : 1;  // (two chunks of a block of 16 column tiles: bt % 4 == 0)
      const bool keeps = may_split && macro_can_keep_order(t.wm, t.wn, t.kb);
      if (order.fixed && kind == EPI_RESID && (bt != order.bt * parts || (parts == 2 && !(keeps && bt % 4 == 0)))) continue;
      const double own = mb == 1 ? 1.0 : mb == 2 ? 0.35 : mb == 3 ? 0.17 : 0.0, ns = t.ns4 + (t.ns1 - t.ns4) * own;
      for (int sp = 1; sp <= (may_split && t.wm * t.wn <= MACRO_SPLIT_FRAGS ? MAX_SPLITS : 1); ++sp) {
        if (sp > 1 && (tiles * sp > CUS || KT / sp < 16)) break;
        const bool fold = order.fixed && order.splits == 2 && sp == 1;
        if (order.fixed && !fold && sp != order.splits) continue;
        if (fold && !keeps) continue;
        const int kps = ((KT + sp - 1) / sp + t.kb - 1) / t.kb * t.kb;
        if ((KT + kps - 1) / kps != sp) continue;  // an empty split
        const int wgs = tiles * sp, full = (wgs - 1) / CUS, last = wgs - CUS * full;
        double us = kps * ns * 1e-3 * (full + 0.65 + 0.35 * last / CUS) + (full + 1) * round_us;
        if (parts > 1) us += 2.5;  // (the epilogue of a tile twice as wide: 2048 rows x 2048 columns, K = 512, 16.6 against 18.9 us)
        if (sp > 1) us += 4.6 + 0.6 * (sp - 1) + 0.62 * (sp - 1) * (mt * 16.0 * N * 8e-6);
        // gated launches (many rounds of wide matrices): fewer rounds where the estimates are within 1 %, as the estimate of a partly
        // filled round is the loosest part (gate/up of a 7B model at 481 .. 512 rows: 128 x 256 in three rounds 161 us, 256 x 192 in
        // two 149; of an 8B one at 2049 .. 2112 rows 389 / 384).  Only between equal splits: the order of the sums does not change.
        const double close = kind == EPI_SWIGLU && sp == best.splits && full != best_full ? (full < best_full ? 1.01 : 0.99) : 1.0;
        if (us < close * best_us) {
          best_us = us;
          best_full = full;
          best = MacroPlan{c, nb, mb, sp, kps, fold ? ((KT + 1) / 2 + 1) / 2 * 2 : 0, parts};
        }
      }
    }
    if (best_us < 1e300 || !order.fixed) return best;  // (an order that no tile has: any order)
  }
}

}  // namespace

int gemm_macro_ssq_chunks(int M, int N, int K) {  // (the plan of the launch itself)
  const MacroPlan p = macro_plan(M, N, K, EPI_RESID);
  const int ct = g_tiles[p.tile].cw * g_tiles[p.tile].wn / p.ssq_parts;
  return ((N >> 4) + ct - 1) / ct;
}
GemmPlan gemm_macro_plan(int M, int N, int K, int kind) {
  const MacroPlan p = macro_plan(M, N, K, kind);
  const MacroTile& t = g_tiles[p.tile];
  return GemmPlan{0, 16 * t.rw * t.wm, 16 * t.cw * t.wn, p.splits, p.fold ? 2 : p.splits, p.nblocks * p.mblocks * p.splits, p.ssq_parts};
}
size_t gemm_macro_part_elems(int M, int N, int K, int kind) {
  const MacroPlan p = macro_plan(M, N, K, kind);
  const MacroTile& t = g_tiles[p.tile];
  return p.splits > 1 ? (size_t)p.splits * p.nblocks * p.mblocks * (t.rw * t.wm) * (t.cw * t.wn) * 256 : 0;
}
int gemm_macro_stat_parts(int M, int N, int K) { return macro_plan(M, N, K, EPI_STATS).nblocks; }
int gemm_macro_counters() { return 2 * MAX_SPLIT_TILES; }  // two per tile of a launch that splits K

void launch_gemm_macro(const op_t* xt, const op_t* wt, int M, int N, int K, const GemmEpi& e, hipStream_t st) {
  const MacroPlan p = macro_plan(M, N, K, e.kind);
  switch (e.kind) {
    case EPI_QKV: launch_macro_epi<EPI_QKV>(xt, wt, M, N, K, p, e, st); break;
    case EPI_SWIGLU: launch_macro_epi<EPI_SWIGLU>(xt, wt, M, N, K, p, e, st); break;
    case EPI_RESID: launch_macro_epi<EPI_RESID>(xt, wt, M, N, K, p, e, st); break;
    case EPI_STATS: launch_macro_epi<EPI_STATS>(xt, wt, M, N, K, p, e, st); break;
    default: launch_macro_epi<EPI_SUM>(xt, wt, M, N, K, p, e, st); break;
  }
}
