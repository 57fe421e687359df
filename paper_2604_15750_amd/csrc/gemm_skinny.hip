// Skinny GEMM of a bf16 model (M <= 64 rows): Y[M,N] = X[M,K] * W[N,K]^T, fp32 accumulation, epilogue fused.
//
// One workgroup per 16- or 32-column output tile over the whole of K.  Its wavefronts split K among
// themselves; each keeps 8 KiB of W fragments (and the matching X fragments) in flight, HBM ->
// registers, and multiplies them on the matrix cores; the accumulators are added through LDS in
// wavefront order (deterministic).  No workgroup waits for another: no workspace, no counter, no
// serial tail.  With 256 .. 768 workgroups all resident at once, HBM stays busy from the first load
// to the last.  Every workgroup re-reads X through its L2, which costs as much of the compute units'
// load bandwidth as W itself for the narrow matrices, so lanes whose row does not exist fetch no line of
// their own (they re-read a row that exists): a fragment's 128-byte lines hold 8 rows each, and a block
// of 8 rows (the minimum block length) reads half of them.  W is read non-temporally: once a pass, by one workgroup, and the memory-side
// cache does not hold it until the next pass unless the model is small (WEIGHTS_CACHED_BYTES; a plain read of HBM 6.2 -> 7.1 TB/s); with both first batches in flight before anything else is
// read, O and down of an 8B model at 8 rows 12.8 -> 12.0 us on average, gate/up of a 7B one at 16 rows 46.8 -> 43.1.
#include "gemm_epilogue.h"

namespace {

// grid.x = N / (16 R) workgroups of NWV wavefronts; wavefront w multiplies k-tiles [w*per, (w+1)*per) of the
// workgroup's R column tiles against all MT row tiles, D k-tiles per batch, two batches of registers.
// STEPS: wt is the step-major copy of W.  NT: W is read non-temporally.
// TWO: registers for two workgroups on a compute unit.
template <int MT, int R, int NWV, int D, int EPI, bool NT, bool STEPS = false, bool TWO = false>
__global__ __launch_bounds__(NWV * 64, TWO ? NWV / 2 : 1) void gemm_skinny_kernel(const op8* __restrict__ xt, const op8* __restrict__ wt, int M, int N,
                                                               int K, GemmEpi e) {
  __shared__ f32x4 red[NWV][R * MT][64];
  __shared__ float s_rinv[MT * 16];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = MT == 2 ? tid >> 6 : __builtin_amdgcn_readfirstlane(tid >> 6);  // (a scalar but for two row tiles: see load)
  const int KT = K >> 5;
  const int per = (KT + NWV - 1) / NWV;
  const int t_begin = wave * per, t_end = min(KT, t_begin + per);
  const op8 zero8 = {0, 0, 0, 0, 0, 0, 0, 0};
  // lanes of the last row tile whose row does not exist re-read row 0 of their k-group (whatever they get is never stored)
  const int xlane_last = (MT - 1) * 16 + (lane & 15) < M ? lane : (lane & ~15);
  // the workgroup's R tiles are one interleaved run; in the step-major copy (KT a multiple of NWV: the host checks) the
  // wavefront's step s is the R fragments from ((s * workgroups + this workgroup) * NWV + wave) * R on
  const op8* wbase = STEPS ? wt + ((size_t)blockIdx.x * NWV + wave) * R * 64 : wt + (size_t)blockIdx.x * KT * R * 64;
  const size_t wstride = STEPS ? (size_t)(N >> 4) * NWV * 64 : R * 64;
  const int tsub = STEPS ? t_begin : 0;

  f32x4 acc[R][MT];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int j = 0; j < MT; ++j) acc[r][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  op8 wreg[2][D][R], xreg[2][D][MT];

  // k-tiles past the wavefront's last one re-read that: the loads are unconditional, as a path around them is one the compiler's count
  // of outstanding loads cannot follow, and scalar in everything but the lane, as a short kernel is bound by the fetching of its
  // instructions first (a test per fragment and addresses in vectors: 2.4 us from the start
  // to the last load of the first batch, 1.0 now; down of an 8B model at 8 rows 18.6 -> 18.0).  With two row tiles addresses in vectors
  // and batches of two are faster (O of 20 rows, K = 3584 10.2 -> 9.6 us, K = 4096 10.3 -> 10.1).
  auto load = [&](int buf, int tb) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < D; ++i) {
      const int t = min(tb + i, t_end - 1);
#pragma unroll
      for (int r = 0; r < R; ++r) wreg[buf][i][r] = load_weight<NT>(wbase + (size_t)(t - tsub) * wstride + r * 64 + lane);
#pragma unroll
      for (int j = 0; j < MT; ++j) xreg[buf][i][j] = (xt + ((size_t)j * KT + t) * 64)[j == MT - 1 ? xlane_last : lane];
    }
    __builtin_amdgcn_sched_barrier(0);
  };
  auto compute = [&](int buf, int tb, bool whole) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < D; ++i) {
      const bool past = !whole && tb + i >= t_end;  // (multiplies zeros)
#pragma unroll
      for (int j = 0; j < MT; ++j) {
        const op8 x = past ? zero8 : xreg[buf][i][j];
#pragma unroll
        for (int r = 0; r < R; ++r) acc[r][j] = mfma_op(wreg[buf][i][r], x, acc[r][j]);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  const bool any = t_begin < t_end;  // (uniform: a wavefront beyond a short K has no k-tiles)
  if (any) {
    load(0, t_begin);
    load(1, t_begin + D);
  }
  // 1/rms of the input rows, needed only by the epilogue: fetched behind the first batches; so is what the epilogue of the tile this
  // wavefront finishes first reads from memory (tile rj = wave of the R * MT)
  typedef RinvBatch<NWV * 64, MT * 16, (MT > 1 && EPI == EPI_QKV ? 4 : 16)> Rinv;  // (down's chunks are few from 17 rows on)
  const int rows = min(M, MT * 16);
  Rinv rinv;
  if (EPI != EPI_RESID) rinv.fetch_always(e.rs, rows, xt);
  EpiAhead ahead = epi_none();
  if ((EPI == EPI_RESID || EPI == EPI_QKV) && wave < R * MT)
    ahead = epi_ahead<EPI>(e, M, N, (wave % MT) * 16 + (lane & 15), (blockIdx.x * R + wave / MT) * 16, lane >> 4);
  __builtin_amdgcn_sched_barrier(0);
  if (any) {
    int tb = t_begin;
    for (; tb + 3 * D < t_end; tb += 2 * D) {
      compute(0, tb, true);
      load(0, tb + 2 * D);
      compute(1, tb + D, true);
      load(1, tb + 3 * D);
    }
    if (tb + 2 * D < t_end) {  // three batches are left, else two (the second of which may be empty)
      compute(0, tb, true);
      load(0, tb + 2 * D);
      compute(1, tb + D, true);
      compute(0, tb + 2 * D, false);
    } else {
      compute(0, tb, false);
      compute(1, tb + D, false);
    }
  }

  if (EPI != EPI_RESID) rinv.publish_all(e.rs, rows, s_rinv);
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int j = 0; j < MT; ++j) red[wave][r * MT + j][lane] = acc[r][j];
  __syncthreads();

  const int g = lane >> 4, ml = lane & 15;
  for (int rj = wave; rj < R * MT; rj += NWV) {  // one wavefront finishes one 16 x 16 tile
    const int r = rj / MT, j = rj % MT;
    const int m = j * 16 + ml;
    const int nt = blockIdx.x * R + r;
    f32x4 v = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NWV; ++w) v += red[w][rj][lane];
    const float ss = finish_frag<EPI>(e, M, N, m, nt * 16, g, v, EPI == EPI_RESID ? 1.f : s_rinv[j * 16 + ml], rj == wave ? ahead : epi_none());
    if (EPI == EPI_RESID && g == 0 && m < M) e.ssq_out[(size_t)m * (N >> 4) + nt] = ss;
  }
}

// batch depth: 8 KiB of W in flight per wavefront for up to 32 rows, half of that beyond (the X fragments take the registers);
// the step-major copy reads best with batches of four (measured: deeper batches add queueing, not bandwidth), of two with two row
// tiles, where a wavefront has few k-tiles and those past its last are read again.  Interleaved pairs
// of column tiles (wide matrices) come here with one row tile only: from 17 rows on the mid or the macro kernel has them.
template <int MT, int EPI, bool NT>
void launch_layout(const op_t* xt, const op_t* wt, int pr, int M, int N, int K, const GemmEpi& e, hipStream_t st) {
  if (pr == 1 && e.w_steps) {
    DLM_LAUNCH((gemm_skinny_kernel<MT, 1, 8, (MT == 2 ? 2 : 4), EPI, NT, true>), N / 16, 512, 0, st, (const op8*)xt, (const op8*)e.w_steps, M, N, K, e);
  } else if (pr == 1) {
    // 257 to 384 column tiles (and more where there is no step-major copy): two workgroups a unit, with batches that leave them the registers,
    // instead of a second round of few (QKV of a 7B model, 288 tiles: 24 rows 16.9 -> 13.7 us, 32 rows 18.7 -> 15.7, 48 rows 22.4 -> 19.2, 64
    // rows 26.3 -> 22.4; O of 272 tiles, K = 4352, 20 / 64 rows 18.6 -> 16.2 / 26.8 -> 24.5; gate/up of 320, K = 6144, 22.7 -> 21.8 / 37.2 -> 34.7).
    // From 385 tiles on, nearly two full rounds, the copy's workgroups are as fast or faster (two a unit / the copy: O of 448 tiles, K =
    // 7168, 20 rows 28.0 / 26.5, 64 rows 41.2 / 40.3; QKV of 448, K = 5120, 20.4 / 19.7, 29.7 / 30.1).
    if constexpr (MT > 1) {
      if (N / 16 > 256) {
        DLM_LAUNCH((gemm_skinny_kernel<MT, 1, 8, (MT == 2 || (MT == 3 && EPI == EPI_QKV) ? 2 : 1), EPI, NT, false, true>), N / 16, 512, 0, st, (const op8*)xt, (const op8*)wt, M, N, K, e);
        return;
      }
    }
    DLM_LAUNCH((gemm_skinny_kernel<MT, 1, 8, (MT <= 2 ? 8 : 4), EPI, NT>), N / 16, 512, 0, st, (const op8*)xt, (const op8*)wt, M, N, K, e);
  } else if constexpr (MT == 1) {
    if (e.w_steps) DLM_LAUNCH((gemm_skinny_kernel<MT, 2, 4, 4, EPI, NT, true>), N / 32, 256, 0, st, (const op8*)xt, (const op8*)e.w_steps, M, N, K, e);
    else DLM_LAUNCH((gemm_skinny_kernel<MT, 2, 4, 4, EPI, NT>), N / 32, 256, 0, st, (const op8*)xt, (const op8*)wt, M, N, K, e);
  }
}

template <int MT, int EPI>
void launch_skinny(const op_t* xt, const op_t* wt, int pr, int M, int N, int K, const GemmEpi& e, hipStream_t st) {
  if constexpr (EPI != EPI_SUM) {  // (of a layer's matrix: a plain product's is not read again)
    if (e.w_cached) return launch_layout<MT, EPI, false>(xt, wt, pr, M, N, K, e, st);
  }
  launch_layout<MT, EPI, true>(xt, wt, pr, M, N, K, e, st);
}

template <int EPI>
void launch_epi(const op_t* xt, const op_t* wt, int pr, int M, int N, int K, const GemmEpi& e, hipStream_t st) {
  if (M <= 16) launch_skinny<1, EPI>(xt, wt, pr, M, N, K, e, st);
  else if (M <= 32) launch_skinny<2, EPI>(xt, wt, pr, M, N, K, e, st);
  else if (M <= 48) launch_skinny<3, EPI>(xt, wt, pr, M, N, K, e, st);
  else launch_skinny<4, EPI>(xt, wt, pr, M, N, K, e, st);
}

}  // namespace

void launch_gemm_skinny(const op_t* xt, const op_t* wt, int pr, int M, int N, int K, const GemmEpi& e_in, hipStream_t st) {
  GemmEpi e = e_in;
  // the step-major copy serves the launches it was laid out for: pr column tiles per workgroup, 8 wavefronts (pr 1) or 4 (pr 2)
  if (!(e.w_steps && e.w_steps_ct == pr && (K >> 5) % (pr == 1 ? 8 : 4) == 0 && N % (16 * pr) == 0)) e.w_steps = nullptr;
  switch (e.kind) {
    case EPI_QKV: launch_epi<EPI_QKV>(xt, wt, pr, M, N, K, e, st); break;
    case EPI_SWIGLU: launch_epi<EPI_SWIGLU>(xt, wt, pr, M, N, K, e, st); break;
    case EPI_RESID: launch_epi<EPI_RESID>(xt, wt, pr, M, N, K, e, st); break;
    default: launch_epi<EPI_SUM>(xt, wt, pr, M, N, K, e, st); break;
  }
}
