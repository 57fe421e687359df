// Mid-size GEMM of a bf16 model (a few dozen to two hundred rows, where its column groups are one round over the compute units:
// choose_kernel in gemm_bf16.hip):
// Y[M,N] = X[M,K] * W[N,K]^T, fp32 accumulation, epilogue fused.
//
// At these row counts W is still the larger operand, but every column group re-reads X, so the groups
// have to be wide.  A workgroup of four wavefronts owns ALL the rows (MT row tiles) of CT adjacent
// column tiles (32 .. 128 columns) and a range of K; its wavefronts split that range among themselves,
// and each multiplies its k-tiles of the CT W fragments against all MT X fragments (CT MT products
// per CT + MT fragments fetched), everything in registers:
//   * W goes HBM -> registers, three steps at a time (a step is one k-tile, two for the narrowest groups; a wavefront keeps 8 .. 24 KiB
//     of W in flight, a workgroup 32 .. 96 KiB: what it takes to keep HBM busy with 128 .. 256 workgroups), non-temporally: one workgroup
//     reads a column group's W, once a pass, and the memory-side cache does not hold it until the next unless the model is small
//     (WEIGHTS_CACHED_BYTES; a plain read of HBM 6.2 -> 7.1 TB/s; gate/up of an 8B model at 8 rows, this and the loads' start below, 33.6 -> 31.4 us, at 37 rows 37.4 -> 33.2, QKV 19.0 -> 17.2);
//     X goes L2 -> registers as many steps ahead (one for more than four row tiles), issued BEFORE the W loads of
//     the same step, because the memory counter retires in order and a wait for X must not wait for younger W loads;
//   * the first loads need nothing from memory (their arguments arrive in registers), and what the rows' 1/rms needs is fetched behind them
//     and finished behind the loop (with three and four row tiles its 48 and 64 loads and the ring's are more than the memory counter's 63: the
//     wait for the first step then takes part of the second step in as well.  With batches that fit, half as large, the chunks left for
//     the end cost more: gate/up of an 8B model at 37 rows 32.3 -> 32.5 us, at 64 rows 34.0 -> 34.2);
//   * no barrier, no LDS inside the loop: a wavefront never waits for another.  (X through
//     direct-to-LDS loads would save a third of the registers, but the compiler then no longer counts
//     the register loads beside them and waits for every load in flight once per trip.)
//   * at the end the four partial accumulators meet in LDS (32 fragments per round), are added in
//     wavefront order, and each wavefront finishes every fourth output fragment.
// When the column groups are fewer than the compute units, K is split across workgroups as well:
// partial tiles go to an fp32 workspace written through to device scope, and the workgroup that takes
// the last ticket adds them in split order (a wavefront fetches the
// same split of all its output fragments in a single trip to memory).
#include "gemm_epilogue.h"
#include <type_traits>

namespace {

constexpr int TPB = 256, NWV = 4;
constexpr int MID_STEPS_MAX_MT = 4;  // row tiles up to which a launch may read the step-major copy of W

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
constexpr int SC1 = 16;  // cache-policy bit of the raw-buffer builtins: device scope

__device__ inline __amdgpu_buffer_rsrc_t part_rsrc(const float* base) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, 0x7fffffff, 0x00020000);
}

template <int MT, int CT>
struct MidShape {
  static constexpr int KB = CT <= 3 ? 2 : 1;  // k-tiles per step: narrow column groups take two, so that a step's loads are still 6 KiB of W
  // steps of W and of X per register ring (one in use, the others in flight).  Three of each: the memory counter retires in order, so X
  // one step ahead lets W be no more than two ahead either; with three or four steps of both ahead HBM serves the chip more slowly
  // (gate/up of an 8B model, 8 rows, W 3 / 4 / 5 deep: 31.4 / 32.0 / 31.7 us; X 2 deep and W 4: 32.2).  X two deep where its fragments are many.
  static constexpr int WD = 3, XD = MT <= 4 ? 3 : 2;
  static constexpr int TRIP = WD * XD / (WD == XD ? XD : 1);  // steps after which both rings are back where they started
  static constexpr int F = CT * MT;                 // output fragments of a workgroup
  static constexpr int FW = (F + NWV - 1) / NWV;    // ... finished by one wavefront
  static constexpr int FR = F < 32 ? (F + 3) / 4 * 4 : 32;  // fragments per reduction round (a multiple of 4: fragment f stays with wavefront f % 4)
  static constexpr int ROUNDS = (F + FR - 1) / FR;
  static constexpr int BODY = NWV * FR * 1024;
  static constexpr int LDS_BYTES = BODY + MT * 16 * 4 + CT * MT * 16 * 4;  // + 1/rms of the rows + every column tile's sum of squares per row
};

// grid.x = groups * splits; MT >= ceil(M / 16), and X has MT row tiles (the activation buffers are padded to 16 rows).
// STEPS: wt is the step-major copy of W.  NT: W is read non-temporally.
template <int MT, int CT, int PR, int EPI, bool STEPS, bool NT>
__global__ __launch_bounds__(TPB) void gemm_mid_kernel(const op8* __restrict__ xt, const op8* __restrict__ wt, int M, int N, int K,
                                                       int kt_per_split, int splits, GemmEpi e) {
  typedef MidShape<MT, CT> SH;
  constexpr int F = SH::F, FW = SH::FW, FR = SH::FR, ROUNDS = SH::ROUNDS;
  constexpr int KB = SH::KB, WD = SH::WD, XD = SH::XD, TRIP = SH::TRIP;
  static_assert(KB * ((XD - 1) * MT + (WD - 1) * CT) < 64, "the loop's loads in flight must fit the memory counter");
  extern __shared__ __align__(16) unsigned char lds[];
  __shared__ int s_last;
  float* s_rinv = (float*)(lds + SH::BODY);  // [MT * 16]
  float* s_ssq = s_rinv + MT * 16;           // [CT][MT * 16]

  // (nothing up to the first loads comes from memory: the arguments in front of e arrive in registers, and the grid's size is not asked for)
  const int group = STEPS ? blockIdx.x : blockIdx.x / splits, split = STEPS ? 0 : blockIdx.x - group * splits;  // (the copy: no K split)
  const int groups = (N + 16 * CT - 1) / (16 * CT);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int KT = K >> 5, NTILES = N >> 4;
  const int nt0 = group * CT;
  const int tb = split * kt_per_split, te = min(KT, tb + kt_per_split);
  const int per = (te - tb + NWV - 1) / NWV;
  const int t0 = tb + wave * per, t1 = min(te, t0 + per);  // this wavefront's k-tiles (possibly none)

  // fragment (nt0 + r, k-tile t) = wptr[r][(t - tsub) * wstep]; column tiles past the end repeat the last one.  With the step-major
  // copy (no K split, whole groups, KT a multiple of 4: the host checks) the wavefront's step s is at wptr[r][s * wstep]
  static_assert(!STEPS || MT <= MID_STEPS_MAX_MT, "the larger variants have no register to spare for a run-time stride");
  constexpr bool steps = STEPS;
  const size_t wstep = steps ? (size_t)groups * NWV * CT * 64 : (PR == 2 ? 128 : 64);
  const int tsub = steps ? t0 : 0;
  const op8* wptr[CT];
#pragma unroll
  for (int r = 0; r < CT; ++r) {
    const int nt = min(nt0 + r, NTILES - 1);
    wptr[r] = steps ? wt + ((size_t)(group * NWV + wave) * CT + r) * 64
                    : PR == 2 ? wt + ((size_t)(nt >> 1) * KT * 2 + (nt & 1)) * 64 : wt + (size_t)nt * KT * 64;
  }
  // In the last row tile, lanes whose row does not exist re-read row 0 of their k-group instead of fetching lines of their
  // own (a fragment's 128-byte lines hold 8 rows each: a block of 8 rows reads half of them); what they get is never stored.
  const int lane_last = (MT - 1) * 16 + (lane & 15) < M ? lane : (lane & ~15);

  f32x4 acc[CT][MT];
#pragma unroll
  for (int r = 0; r < CT; ++r)
#pragma unroll
    for (int j = 0; j < MT; ++j) acc[r][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  op8 w[WD][KB][CT], x[XD][KB][MT];
  const int nsteps = (t1 - t0 + KB - 1) / KB;
  const op8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};

  // step st of the wavefront (its k-tiles clamped to the wavefront's last one) -> register set `slot`
  auto load_x = [&](const int slot, int st) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < KB; ++i) {
      const int tc = min(t0 + st * KB + i, t1 - 1);
#pragma unroll
      for (int j = 0; j < MT; ++j) x[slot][i][j] = (xt + ((size_t)j * KT + tc) * 64)[j == MT - 1 ? lane_last : lane];
    }
  };
  auto load_w = [&](const int slot, int st) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < KB; ++i) {
      const int tc = min(t0 + st * KB + i, t1 - 1);
#pragma unroll
      for (int r = 0; r < CT; ++r) w[slot][i][r] = load_weight<NT>(wptr[r] + (size_t)(tc - tsub) * wstep + lane);
    }
  };
  auto compute = [&](const int ws, const int xs, int st) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < KB; ++i) {
      const bool past = KB > 1 && t0 + st * KB + i >= t1;  // the surplus k-tile of a ragged last step multiplies zeros
#pragma unroll
      for (int j = 0; j < MT; ++j) {
        const op8 xv = past ? zero8 : x[xs][i][j];
#pragma unroll
        for (int r = 0; r < CT; ++r) acc[r][j] = mfma_op(w[ws][i][r], xv, acc[r][j]);
      }
    }
  };
  // step S of a trip: X of the step XD - 1 ahead first, then W of the step WD - 1 ahead, so that the wait for this step's operands
  // (the oldest loads) leaves XD - 1 steps of both in flight; the scheduling barriers keep the compiler from sinking the loads down to
  // their uses (which it does under register pressure, undoing the prefetch)
  auto step = [&](auto Sc, int st) __attribute__((always_inline)) {
    constexpr int S = decltype(Sc)::value;
    load_x((S + XD - 1) % XD, st + XD - 1);
    load_w((S + WD - 1) % WD, st + WD - 1);
    __builtin_amdgcn_sched_barrier(0);
    compute(S % WD, S % XD, st);
    __builtin_amdgcn_sched_barrier(0);
  };
  // (every lambda here is forced inline: left to its own judgement the compiler keeps the largest variants' steps as
  // functions, and the operand rings, passed by reference, then live in scratch memory)
  // whole trips: TRIP steps in a row; the steps left over: nested, not skippable one by one (a path around a step's loads is
  // one the compiler's count of outstanding loads cannot follow: it would wait for all of them)
  auto trip = [&](auto self, auto Ic, int st) __attribute__((always_inline)) {
    constexpr int I = decltype(Ic)::value;
    if constexpr (I < TRIP) {
      step(Ic, st + I);
      self(self, std::integral_constant<int, I + 1>{}, st);
    }
  };
  auto rest = [&](auto self, auto Ic, int st) __attribute__((always_inline)) {
    constexpr int I = decltype(Ic)::value;
    if constexpr (I < TRIP - 1) {
      if (st + I < nsteps) {
        step(Ic, st + I);
        self(self, std::integral_constant<int, I + 1>{}, st);
      }
    }
  };
  const bool any = STEPS || nsteps > 0;  // (the copy: every wavefront has k-tiles)
  if (any) {
#pragma unroll
    for (int i = 0; i < WD - 1; ++i) {
      if (i < XD - 1) load_x(i, i);
      load_w(i, i);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
  // 1/rms of the input rows, needed only by the epilogue: fetched behind the first k-tiles, and kept until the loop is over (published
  // by the barriers of the reduction)
  typedef RinvBatch<TPB, MT * 16, ((MT > 1 && EPI == EPI_QKV) || MT > 4) ? 4 : 16> Rinv;  // (down's chunks are few from 17 rows on)
  const int rows = min(M, MT * 16);
  Rinv rinv;
  if (EPI != EPI_RESID) rinv.fetch_always(e.rs, rows, xt);
  __builtin_amdgcn_sched_barrier(0);
  // ... and so is what the epilogue of the fragment this wavefront finishes first (fragment `wave`) reads from memory, in the
  // variants of narrow passes, which are short enough for that round trip to show
  EpiAhead ahead = epi_none();
  if constexpr (MT <= 2 && (EPI == EPI_RESID || EPI == EPI_QKV)) {
    if (splits == 1 && wave < F && nt0 + wave / MT < NTILES)
      ahead = epi_ahead<EPI>(e, M, N, (wave % MT) * 16 + (lane & 15), (nt0 + wave / MT) * 16, lane >> 4);
  }
  if (any) {
    int st = 0;
    for (; st + TRIP <= nsteps; st += TRIP) trip(trip, std::integral_constant<int, 0>{}, st);
    rest(rest, std::integral_constant<int, 0>{}, st);
  }

  if (EPI != EPI_RESID) rinv.publish_all(e.rs, rows, s_rinv);
  // ---- the four partial accumulators -> one finished (or, with a K split, one partial) value per output fragment
  const int g = lane >> 4, ml = lane & 15;
  f32x4* red = (f32x4*)lds;  // [NWV][FR][64]
  // K split: partial tiles lie fragment by fragment in the accumulator layout, [split][group][fragment][lane]
  auto partial = [&](int s) { return part_rsrc(e.part + (size_t)(s * groups + group) * (F * 256)); };
  // fragment f = r * MT + j (column tile r, row tile j) in the accumulator layout -> its epilogue
  auto finish = [&](int f, f32x4 v) {
    const int r = f / MT, j = f - r * MT;
    const int nt = nt0 + r, m = j * 16 + ml;
    float ss = 0.f;
    if (nt < NTILES) ss = finish_frag<EPI>(e, M, N, m, nt * 16, g, v, EPI == EPI_RESID ? 1.f : s_rinv[m], f == wave ? ahead : epi_none());  // uniform in the wavefront
    if (EPI == EPI_RESID && g == 0) s_ssq[r * MT * 16 + m] = ss;
  };
#pragma unroll
  for (int rd = 0; rd < ROUNDS; ++rd) {
    if (rd) __syncthreads();  // the previous round has been read
#pragma unroll
    for (int i = 0; i < FR; ++i)
      if (rd * FR + i < F) red[(wave * FR + i) * 64 + lane] = acc[min(rd * FR + i, F - 1) / MT][min(rd * FR + i, F - 1) % MT];
    __syncthreads();
    for (int i = wave; i < FR && rd * FR + i < F; i += NWV) {
      const f32x4 v = ((red[i * 64 + lane] + red[(FR + i) * 64 + lane]) + red[(2 * FR + i) * 64 + lane]) + red[(3 * FR + i) * 64 + lane];
      const int f = rd * FR + i;
      if (splits == 1) {
        finish(f, v);
      } else {  // partial tile -> workspace, written through to device scope
        const int r = f / MT, j = f - r * MT;
        if (nt0 + r < NTILES && j * 16 < M) __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), partial(split), (unsigned)(f * 64 + lane) * 16u, 0, SC1);
      }
    }
  }
  if (splits > 1) {
    // Hand-off across workgroups (possibly across XCDs, whose L2s are separate): every wavefront waits until its own partial
    // stores, written through to device scope, have been acknowledged; then the workgroup takes its ticket, and the last
    // arriver reads the partial tiles at device scope.  Tickets and data are device-scope accesses themselves, so neither side
    // needs a fence: a release would write back the L2's dirty lines, an acquire drop its clean ones.
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) {
      int* ticket = e.counters + group;
      const int last = __hip_atomic_fetch_add(ticket, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == splits - 1;
      if (last) __hip_atomic_store(ticket, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);  // ready for the next launch
      s_last = last;
    }
    __syncthreads();
    if (!s_last) return;
    asm volatile("" ::: "memory");
    // the finished tile = the partial tiles added in split order; a wavefront fetches one split of all its fragments per trip
    f32x4 v[FW];
    unsigned off[FW];
#pragma unroll
    for (int i = 0; i < FW; ++i) {
      const int f = wave + NWV * i, r = f / MT, j = f - r * MT;
      off[i] = (f < F && nt0 + r < NTILES && j * 16 < M) ? (unsigned)(f * 64 + lane) * 16u : 0u;  // fragments that do not exist re-read element 0
      v[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    for (int s = 0; s < splits; s += 2) {  // two splits per trip to memory
      const int s1 = min(s + 1, splits - 1);
      u32x4 ta[FW], tb[FW];
#pragma unroll
      for (int i = 0; i < FW; ++i) ta[i] = __builtin_amdgcn_raw_buffer_load_b128(partial(s), off[i], 0, SC1);
#pragma unroll
      for (int i = 0; i < FW; ++i) tb[i] = __builtin_amdgcn_raw_buffer_load_b128(partial(s1), off[i], 0, SC1);
#pragma unroll
      for (int i = 0; i < FW; ++i) v[i] += __builtin_bit_cast(f32x4, ta[i]);
      if (s + 1 < splits)
#pragma unroll
        for (int i = 0; i < FW; ++i) v[i] += __builtin_bit_cast(f32x4, tb[i]);
    }
#pragma unroll
    for (int i = 0; i < FW; ++i)
      if (wave + NWV * i < F) finish(wave + NWV * i, v[i]);
  }
  if (EPI == EPI_RESID) {  // the workgroup's share of sum h^2 per row: its column tiles in order
    __syncthreads();
    if (tid < MT * 16 && tid < M) {
      float ss = 0.f;
#pragma unroll
      for (int r = 0; r < CT; ++r) ss += s_ssq[r * MT * 16 + tid];
      e.ssq_out[(size_t)tid * groups + group] = ss;
    }
  }
}

struct MidPlan {
  int ct, pr, mt, groups, splits, kps;
};

// What the compute units can load through their L2s (W once, X once per column group; about 45 GB/s each, 10 .. 12 TB/s
// together) bounds these shapes before HBM does, and a K split costs a round trip of partial tiles through memory plus a
// serial tail.  Wide matrices: of the group widths 128, 96 and 48 columns, the one that fills the chip's 256
// compute units best, without a K split if it can (QKV of an 8B model: 256 groups of 48; gate/up: 256 groups of 96).
// Narrow ones (O, down; at most 256 column tiles): 64-column groups and a four-way K split when K is long (down), 32-column
// groups and a two-way split when it is short (O); all measured against their alternatives.
MidPlan mid_plan(int M, int N, int K) {
  MidPlan best;
  double best_fill = -1.;
  const int pr = weight_pack_rows(N), mt = (M + 15) >> 4, KT = K >> 5;
  // short K: the partial tiles of a four-way split cost more than X re-read by twice the groups
  const int narrow = K >= 8192 && mt > 1 ? 4 : 2;
  // (a wide matrix beyond four row tiles comes here only for its 48-column groups)
  const int cts[3] = {pr == 2 ? (mt <= 4 ? 8 : 3) : narrow, pr == 2 ? (mt <= 4 ? 6 : 3) : narrow, pr == 2 ? 3 : narrow};
  for (int c = 0; c < 3; ++c) {
    MidPlan p;
    p.pr = pr; p.mt = mt; p.ct = cts[c];
    p.groups = (N + 16 * p.ct - 1) / (16 * p.ct);
    int s = pr == 2 ? 256 / p.groups : (256 + p.groups / 2) / p.groups;
    if (pr == 1 && mt == 1) s = 1;  // one row tile of a narrow matrix comes here only to avoid a second round of 16-column workgroups
    if (s > (pr == 2 ? 2 : 4)) s = pr == 2 ? 2 : 4;  // a short serial tail for the last arriver, and little traffic of partial tiles
    if (s > KT / 16) s = KT / 16;     // at least four k-tiles per wavefront
    if (s < 1) s = 1;
    p.kps = (KT + s - 1) / s;
    p.splits = (KT + p.kps - 1) / p.kps;  // no empty split
    // as many groups of the widest kind as compute units, or more: the widest re-reads X least (more than one round of them is not
    // launched: choose_kernel gives such a shape to another kernel)
    if (c == 0 && p.groups >= 256) return p;
    // otherwise, of the group widths, the one whose workgroups fill the chip's 256 compute units best; on a near tie the
    // one without a K split, then the wider
    const int wgs = p.groups * p.splits;
    const double fill = (double)wgs / ((wgs + 255) / 256 * 256) + (p.splits == 1 ? 0.01 : 0.);
    if (fill > best_fill + 0.005) { best_fill = fill; best = p; }
  }
  return best;
}

template <int MT, int CT, int PR, int EPI, bool STEPS, bool NT>
void launch_kernel(const op_t* xt, const op_t* wt, int M, int N, int K, const MidPlan& p, const GemmEpi& e, hipStream_t st) {
  typedef MidShape<MT, CT> SH;
  static bool configured = false;  // raise the dynamic LDS limit of this instantiation once
  if (!configured) {
    (void)hipFuncSetAttribute((const void*)gemm_mid_kernel<MT, CT, PR, EPI, STEPS, NT>, hipFuncAttributeMaxDynamicSharedMemorySize, SH::LDS_BYTES);
    configured = true;
  }
  DLM_LAUNCH((gemm_mid_kernel<MT, CT, PR, EPI, STEPS, NT>), p.groups * p.splits, TPB, SH::LDS_BYTES, st, (const op8*)xt, (const op8*)wt, M, N, K,
             p.kps, p.splits, e);
}
template <int MT, int CT, int PR, int EPI, bool NT>
void launch_layout(const op_t* xt, const op_t* wt, int M, int N, int K, const MidPlan& p, const GemmEpi& e, hipStream_t st) {
  if constexpr (MT <= MID_STEPS_MAX_MT) {
    if (e.w_steps) return launch_kernel<MT, CT, PR, EPI, true, NT>(xt, e.w_steps, M, N, K, p, e, st);
  }
  launch_kernel<MT, CT, PR, EPI, false, NT>(xt, wt, M, N, K, p, e, st);
}
template <int MT, int CT, int PR, int EPI>
void launch_one(const op_t* xt, const op_t* wt, int M, int N, int K, const MidPlan& p, const GemmEpi& e, hipStream_t st) {
  // (a layer's matrix, not a plain product's, which is not read again; beyond four row tiles W is the smaller part: a pass of 96 rows
  // through 4 layers of 1024 x 3584 takes 201 us with every W non-temporal, 195 with none)
  if constexpr (EPI != EPI_SUM && MT <= 4) {
    if (e.w_cached) return launch_layout<MT, CT, PR, EPI, false>(xt, wt, M, N, K, p, e, st);
  }
  launch_layout<MT, CT, PR, EPI, true>(xt, wt, M, N, K, p, e, st);
}

template <int MT, int EPI>
void launch_mt(const op_t* xt, const op_t* wt, int M, int N, int K, const MidPlan& p, const GemmEpi& e, hipStream_t st) {
  if (p.pr == 1) {
    if (p.ct == 2) { if constexpr (MT <= 13) launch_one<MT, 2, 1, EPI>(xt, wt, M, N, K, p, e, st); }
    else if constexpr (MT >= 2 && MT <= 8) launch_one<MT, 4, 1, EPI>(xt, wt, M, N, K, p, e, st);
  } else if (p.ct == 3) {
    if constexpr (MT <= 6) launch_one<MT, 3, 2, EPI>(xt, wt, M, N, K, p, e, st);
  } else if (p.ct == 8) {
    if constexpr (MT <= 4) launch_one<MT, 8, 2, EPI>(xt, wt, M, N, K, p, e, st);
  } else {
    if constexpr (MT <= 4) launch_one<MT, 6, 2, EPI>(xt, wt, M, N, K, p, e, st);
  }
}

template <int EPI>
void launch_epi(const op_t* xt, const op_t* wt, int M, int N, int K, const MidPlan& p, const GemmEpi& e, hipStream_t st) {
  switch (p.mt) {  // the dispatcher sends only row counts that have an instantiation
    case 1: launch_mt<1, EPI>(xt, wt, M, N, K, p, e, st); break;
    case 2: launch_mt<2, EPI>(xt, wt, M, N, K, p, e, st); break;
    case 3: launch_mt<3, EPI>(xt, wt, M, N, K, p, e, st); break;
    case 4: launch_mt<4, EPI>(xt, wt, M, N, K, p, e, st); break;
    case 5: launch_mt<5, EPI>(xt, wt, M, N, K, p, e, st); break;
    case 6: launch_mt<6, EPI>(xt, wt, M, N, K, p, e, st); break;
    case 7: launch_mt<7, EPI>(xt, wt, M, N, K, p, e, st); break;
    case 8: launch_mt<8, EPI>(xt, wt, M, N, K, p, e, st); break;
    case 9: launch_mt<9, EPI>(xt, wt, M, N, K, p, e, st); break;
    case 10: launch_mt<10, EPI>(xt, wt, M, N, K, p, e, st); break;
    case 11: launch_mt<11, EPI>(xt, wt, M, N, K, p, e, st); break;
    case 12: launch_mt<12, EPI>(xt, wt, M, N, K, p, e, st); break;
    default: launch_mt<13, EPI>(xt, wt, M, N, K, p, e, st); break;
  }
}

}  // namespace

// whole rounds of workgroups without a K split, whatever the width of the groups: the shapes the mid kernel takes even below 17 rows
bool gemm_mid_fills_chip(int M, int N, int K) {
  const MidPlan p = mid_plan(M, N, K);
  return p.splits == 1 && p.groups % 256 == 0;
}
bool gemm_mid_one_round(int M, int N, int K) {
  const MidPlan p = mid_plan(M, N, K);
  return p.groups * p.splits <= 256;
}
GemmPlan gemm_mid_plan(int M, int N, int K) {
  const MidPlan p = mid_plan(M, N, K);
  return GemmPlan{0, 16 * p.mt, 16 * p.ct, p.splits, p.splits, p.groups * p.splits, 1};
}
size_t gemm_mid_part_elems(int M, int N, int K) {
  const MidPlan p = mid_plan(M, N, K);
  return p.splits > 1 ? (size_t)p.splits * p.groups * p.ct * p.mt * 256 : 0;
}
int gemm_mid_ssq_chunks(int M, int N, int K) { return mid_plan(M, N, K).groups; }
int gemm_mid_counters(int max_n) { return (max_n + 31) / 32; }  // 32-column groups are the narrowest

int gemm_mid_steps_ct(int N, int K) {
  const MidPlan p = mid_plan(16, N, K);
  return (p.splits == 1 && N % (16 * p.ct) == 0 && (K >> 5) % NWV == 0) ? p.ct : 0;
}

void launch_gemm_mid(const op_t* xt, const op_t* wt, int M, int N, int K, const GemmEpi& e_in, hipStream_t st) {
  const MidPlan p = mid_plan(M, N, K);
  GemmEpi e = e_in;
  // the step-major copy serves exactly the launches it was laid out for
  if (!(e.w_steps && p.mt <= MID_STEPS_MAX_MT && e.w_steps_ct == p.ct && p.splits == 1 && N % (16 * p.ct) == 0 && (K >> 5) % NWV == 0)) e.w_steps = nullptr;
  switch (e.kind) {
    case EPI_QKV: launch_epi<EPI_QKV>(xt, wt, M, N, K, p, e, st); break;
    case EPI_SWIGLU: launch_epi<EPI_SWIGLU>(xt, wt, M, N, K, p, e, st); break;
    case EPI_RESID: launch_epi<EPI_RESID>(xt, wt, M, N, K, p, e, st); break;
    default: launch_epi<EPI_SUM>(xt, wt, M, N, K, p, e, st); break;
  }
}
