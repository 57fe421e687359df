// Fused vocabulary reduction (paper Sec. 4.2: Eq. 3 and the entropy signal; Sec. 4.3: confidence
// and prediction).  One pass over each row of logits gives, with the mask token excluded,
//   m = max z, y = argmax, s = sum e^(z-m), t = sum e^(z-m) (z-m), w = sum e^(z-m) (z-z')
// and from those  lse = m + ln s,  conf = 1/s,  H = ln s - t/s,  KL(p||p') = w/s - lse + lse'.
// The kernel is a pure HBM stream: 16-byte loads, several in flight per lane, rows split over
// enough workgroups to fill 256 CUs; partial states are merged in a fixed order (deterministic).
#include "stats_part.h"

namespace {

template <typename T> struct Vec;
template <> struct Vec<bf16_t> { static constexpr int N = 8; typedef bf16x8 type; };
template <> struct Vec<float> { static constexpr int N = 4; typedef f32x4 type; };

constexpr float LOG2E = 1.4426950408889634f, LN2 = 0.6931471805599453f;

// Running state of a wavefront while it streams its share of a row.  The reference of the exponentials is the maximum of
// ALL the wavefront's elements so far (m, the same in every lane), not each lane's own: a new maximum then turns up a few
// times per row instead of in some lane at nearly every step, so the rescaling and the search for the maximum's token id sit
// in a wavefront-uniform branch that is almost never taken, and the common path is straight-line: per element a subtract and
// a multiply for the exponent, one exp2, one add and one fma (two more for KL).  The exponent-weighted sum
// t2 = sum e^(z-m) (z-m) log2(e) is kept in base-2 units.  bi = lowest token id of the maximum (elements are visited in
// ascending id order within a lane, lanes of one load hold ascending ids, and a later element must be strictly greater).
struct Run {
  float m;          // uniform: running maximum (= the best logit)
  int bi;           // uniform: its token id
  float s, t2, w;   // per lane, relative to m
  float pm, ps;     // previous-step row when its lse is not stored: uniform maximum, per-lane sum e^(z'-pm)
};
constexpr float RUN_MIN = -2.0e38f;  // start of the running maximum: (RUN_MIN - m) * log2(e) stays finite for real maxima m
__device__ inline Run run_init() { return Run{RUN_MIN, 0x7fffffff, 0.f, 0.f, 0.f, RUN_MIN, 0.f}; }

// (wave_sum and wave_max of common.h, and the same for the least token id: a wavefront makes these trips at its end and at every new
// maximum, and a chunk is short: 384 rows of 126464 bf16 logits from memory, without / with a previous row, 28.3 / 43.5 us through LDS, 24.7 /
// 40.2 now.)
__device__ inline int lanes_min(int v) {
  return (int)butterfly((unsigned)v, [](unsigned a, unsigned b) { return (unsigned)min((int)a, (int)b); });
}

// The 64 lane states -> the wavefront's Part (valid in every lane): the lanes share m, so the sums are plain butterflies in a
// fixed order (deterministic).
__device__ inline Part run_finish(const Run& r) {
  Part p;
  p.m = r.m;
  p.s = wave_sum(r.s);
  p.t = wave_sum(r.t2) * LN2;
  p.w = wave_sum(r.w);
  p.bv = r.m;
  p.bi = r.bi;
  p.pm = r.pm > RUN_MIN ? r.pm : NEG_BIG;
  p.ps = wave_sum(r.ps);
  return p;
}

// A new maximum somewhere in the wavefront (vm = each lane's maximum of its N elements, RUN_MIN if it has none): move the
// reference.  Called by all 64 lanes together, from a wavefront-uniform branch.
template <int N>
__device__ inline void new_maximum(Run& p, const float (&z)[N], unsigned valid, float vm, int v0) {
  const float wmax = wave_max(vm);
  int cand = 0x7fffffff;
#pragma unroll
  for (int i = N - 1; i >= 0; --i)
    if (((valid >> i) & 1u) && z[i] == wmax) cand = v0 + i;
  const float d2 = (p.m - wmax) * LOG2E, a = __builtin_amdgcn_exp2f(d2);
  p.t2 = a * fmaf(d2, p.s, p.t2);
  p.s *= a;
  p.w *= a;
  p.m = wmax;
  p.bi = lanes_min(cand);
}
template <int N>
__device__ inline void new_prev_maximum(Run& p, float vm) {
  const float wmax = wave_max(vm);
  p.ps *= __builtin_amdgcn_exp2f((p.pm - wmax) * LOG2E);
  p.pm = wmax;
}

// Absorb N consecutive logits (first token id v0) of every lane; bit i of `valid` says that element i takes part (the mask
// token and elements past the end do not).  ALL: every element of every lane is valid (the common path: no selects).
// Called by all 64 lanes of a wavefront together.
template <int N, bool KL, bool PREV_SUMS, bool ALL>
__device__ inline void absorb(Run& p, const float (&z)[N], const float (&zp)[N], int v0, unsigned valid) {
  float vm = RUN_MIN;
#pragma unroll
  for (int i = 0; i < N; ++i) vm = fmaxf(vm, (ALL || ((valid >> i) & 1u)) ? z[i] : RUN_MIN);
  if (__builtin_amdgcn_ballot_w64(vm > p.m) != 0) new_maximum<N>(p, z, ALL ? 0xffffffffu : valid, vm, v0);
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const float d2 = (z[i] - p.m) * LOG2E;  // the difference first: exact for nearby values
    float e = __builtin_amdgcn_exp2f(d2);
    if (!ALL) e = ((valid >> i) & 1u) ? e : 0.f;
    p.s += e;
    p.t2 = fmaf(e, ALL ? d2 : (((valid >> i) & 1u) ? d2 : 0.f), p.t2);
    if (KL) p.w = fmaf(e, ALL ? z[i] - zp[i] : (((valid >> i) & 1u) ? z[i] - zp[i] : 0.f), p.w);
  }
  if (KL && PREV_SUMS) {
    float pv = RUN_MIN;
#pragma unroll
    for (int i = 0; i < N; ++i) pv = fmaxf(pv, (ALL || ((valid >> i) & 1u)) ? zp[i] : RUN_MIN);
    if (__builtin_amdgcn_ballot_w64(pv > p.pm) != 0) new_prev_maximum<N>(p, pv);
#pragma unroll
    for (int i = 0; i < N; ++i) {
      const float e = __builtin_amdgcn_exp2f((zp[i] - p.pm) * LOG2E);
      p.ps += (ALL || ((valid >> i) & 1u)) ? e : 0.f;
    }
  }
}

__device__ inline void finalize(const Part& p, int row, bool has_prev, float prev_lse, const StatsOut& o, float* save_lse_slot) {
  float ls = __logf(p.s);
  float lse = p.m + ls;
  o.max_logit[row] = p.m;
  o.lse[row] = lse;
  o.conf[row] = 1.0f / p.s;
  o.entropy[row] = ls - p.t / p.s;
  o.argmax[row] = p.bi;
  o.kl[row] = has_prev ? (p.w / p.s - lse + prev_lse) : 0.f;
  if (save_lse_slot) *save_lse_slot = lse;
}

// One wavefront's share of elements [lo, hi) of a row (the workgroup walks them together: lane l of the workgroup takes the
// l-th vector of every stride).  Whole trips of U vectors (16 bytes each) per lane are loaded together and absorbed one after
// the other without a bounds or mask test; the trip that holds the mask token and the ragged last one take the path with
// per-element validity.  AHEAD: a trip's loads go out before the trip in front of it is absorbed (loads_ahead).  Loop bounds are uniform
// in the workgroup: the absorb steps exchange values between lanes.
template <typename T, int TPB, bool VECTOR, bool AHEAD, bool KL, bool PREV_SUMS>
__device__ inline void stream_chunk(Run& run, const T* __restrict__ z_row, const T* __restrict__ p_row, T* __restrict__ s_row, int lo,
                                    int hi, int mask_id) {
  constexpr int N = Vec<T>::N;
  typedef typename Vec<T>::type V;
  if (VECTOR) {
    constexpr int U = TPB > 256 ? 2 : 4, STRIDE = TPB * N, TRIP = U * STRIDE;
    const int base = lo + threadIdx.x * N;
    const int nfull = (hi - lo) / TRIP;
    auto fetch = [&](V (&zv)[U], V (&pv)[U], int t) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        zv[u] = *(const V*)(z_row + base + t * TRIP + u * STRIDE);
        if (KL) pv[u] = *(const V*)(p_row + base + t * TRIP + u * STRIDE);
      }
    };
    auto take = [&](const V (&zv)[U], const V (&pv)[U], int t) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int v = base + t * TRIP + u * STRIDE;
        float z[N], zp[N];
#pragma unroll
        for (int i = 0; i < N; ++i) { z[i] = to_f32(zv[u][i]); zp[i] = KL ? to_f32(pv[u][i]) : 0.f; }
        if (s_row) *(V*)(s_row + v) = zv[u];
        absorb<N, KL, PREV_SUMS, true>(run, z, zp, v, 0xffffffffu);
      }
    };
    const int mask_trip = mask_id >= lo ? (mask_id - lo) / TRIP : -1;  // (a trip of another chunk where it is past the end)
    for (int t = 0; t * TRIP < hi - lo;) {
      const int end = mask_trip >= t && mask_trip < nfull ? mask_trip : nfull;  // whole trips without the mask token
      V zv[U], pv[U];
      if constexpr (AHEAD) {
        if (t < end) {
          V zw[U], pw[U];
          fetch(zv, pv, t);
          for (; end - t > 2; t += 2) {
            fetch(zw, pw, t + 1);
            __builtin_amdgcn_sched_barrier(0);
            take(zv, pv, t);
            fetch(zv, pv, t + 2);
            __builtin_amdgcn_sched_barrier(0);
            take(zw, pw, t + 1);
          }
          if (end - t == 2) {
            fetch(zw, pw, t + 1);
            __builtin_amdgcn_sched_barrier(0);
            take(zv, pv, t);
            take(zw, pw, t + 1);
          } else {
            take(zv, pv, t);
          }
          t = end;
          continue;
        }
      } else {
        if (t < end) {
          for (; t < end; ++t) {
            fetch(zv, pv, t);
            take(zv, pv, t);
          }
          continue;
        }
      }
      const int t0 = lo + t * TRIP;  // first element of the trip (uniform)
#pragma unroll 1
      for (int u = 0; u < U; ++u) {
        const int v = base + t * TRIP + u * STRIDE;
        if (t0 + u * STRIDE >= hi) break;  // uniform
        const bool in = v < hi;            // vocab % N == 0 and lo % N == 0: a vector is inside or outside as a whole
        float z[N], zp[N];
        V a, b;
        if (in) { a = *(const V*)(z_row + v); if (KL) b = *(const V*)(p_row + v); }
#pragma unroll
        for (int i = 0; i < N; ++i) { z[i] = in ? to_f32(a[i]) : 0.f; zp[i] = (KL && in) ? to_f32(b[i]) : 0.f; }
        if (s_row && in) *(V*)(s_row + v) = a;
        unsigned valid = in ? (1u << N) - 1u : 0u;
        if (mask_id >= v && mask_id < v + N) valid &= ~(1u << (mask_id - v));  // the mask token takes no part
        absorb<N, KL, PREV_SUMS, false>(run, z, zp, v, valid);
      }
      ++t;
    }
  } else {
    for (int v0 = lo; v0 < hi; v0 += TPB) {  // uniform bounds; a lane past the end or on the mask token feeds an invalid element
      const int v = v0 + threadIdx.x;
      const bool in = v < hi;
      float z[1] = {in ? to_f32(z_row[v]) : 0.f}, zp[1] = {(KL && in) ? to_f32(p_row[v]) : 0.f};
      if (s_row && in) s_row[v] = z_row[v];
      absorb<1, KL, PREV_SUMS, false>(run, z, zp, v, (in && v != mask_id) ? 1u : 0u);
    }
  }
}

// Workgroups of 256 threads of the vector path on a compute unit, held (stats_plan) where the registers would let one more in
template <typename T> constexpr int HELD = sizeof(T) == 2 ? 5 : 6;

template <typename T, int TPB, bool VECTOR, int PER_UNIT, bool AHEAD>
__global__ __launch_bounds__(TPB) __attribute__((amdgpu_waves_per_eu(1, TPB == 256 ? PER_UNIT : 8))) void vocab_stats_kernel(const T* __restrict__ logits, int vocab, int mask_id, int chunk,
                                                          int nchunks, StatsRows sr, StatsOut o, Part* __restrict__ parts) {
  __shared__ Part sh[TPB / 64];
  const int row = blockIdx.x / nchunks, c = blockIdx.x - row * nchunks;
  const T* z_row = logits + (size_t)row * vocab;
  const int64_t prow = sr.prev_row ? sr.prev_row[row] : (sr.prev_base ? (int64_t)row * vocab : -1);
  const int64_t srow = sr.save_row ? sr.save_row[row] : -1;
  const T* p_row = prow >= 0 ? (const T*)sr.prev_base + prow : nullptr;
  T* s_row = srow >= 0 ? (T*)sr.save_base + srow : nullptr;
  const bool kl = p_row != nullptr;
  const bool prev_sums = kl && sr.prev_lse == nullptr;
  const int lo = c * chunk, hi = min(vocab, lo + chunk);

  Run run = run_init();
  if (!kl) stream_chunk<T, TPB, VECTOR, AHEAD, false, false>(run, z_row, p_row, s_row, lo, hi, mask_id);
  else if (!prev_sums) stream_chunk<T, TPB, VECTOR, AHEAD, true, false>(run, z_row, p_row, s_row, lo, hi, mask_id);
  else stream_chunk<T, TPB, VECTOR, AHEAD, true, true>(run, z_row, p_row, s_row, lo, hi, mask_id);
  const Part p = run_finish(run);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = p;
  __syncthreads();
  if (threadIdx.x == 0) {
    Part r = sh[0];
    for (int i = 1; i < TPB / 64; ++i) r = part_merge(r, sh[i]);
    if (nchunks == 1) {
      float pl = 0.f;
      if (kl) pl = sr.prev_lse ? sr.prev_lse[prow / vocab] : r.pm + __logf(r.ps);
      finalize(r, row, kl, pl, o, srow >= 0 && sr.save_lse ? sr.save_lse + srow / vocab : nullptr);
    } else {
      parts[(size_t)row * nchunks + c] = r;
    }
  }
}

// one wavefront per row: lane c holds the partial state of chunk c (of chunks c, c + 64, ... merged in that order); fixed butterfly order
__global__ __launch_bounds__(64) void vocab_stats_merge_kernel(const Part* __restrict__ parts, int rows, int nchunks, int vocab, StatsRows sr,
                                                               StatsOut o) {
  const int row = blockIdx.x, lane = threadIdx.x;
  // (what the row's results need besides, read beside its states: two trips and a division that would come after the merge)
  const int64_t prow = sr.prev_row ? sr.prev_row[row] : (sr.prev_base ? (int64_t)row * vocab : -1);
  const int64_t srow = sr.save_row ? sr.save_row[row] : -1;
  Part r = lane < nchunks ? parts[(size_t)row * nchunks + lane] : part_init();
  for (int c0 = 64; c0 < nchunks; c0 += 512) {  // more states than lanes (the LM-head epilogue's): eight loads in flight, added in order
    Part q[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) q[i] = c0 + 64 * i + lane < nchunks ? parts[(size_t)row * nchunks + c0 + 64 * i + lane] : part_init();
#pragma unroll
    for (int i = 0; i < 8; ++i) r = part_merge(r, q[i]);
  }
  const float prev_lse = prow >= 0 && sr.prev_lse ? sr.prev_lse[prow / vocab] : 0.f;
  float* save_slot = srow >= 0 && sr.save_lse ? sr.save_lse + srow / vocab : nullptr;
#pragma unroll
  for (int ofs = 32; ofs > 0; ofs >>= 1) r = part_merge(r, part_from(r, ofs));
  if (lane != 0) return;
  const float pl = prow < 0 ? 0.f : sr.prev_lse ? prev_lse : r.pm + __logf(r.ps);
  finalize(r, row, prow >= 0, pl, o, save_slot);
}

constexpr int MAX_CHUNKS = 32;
constexpr int ROW_MIN = 136, ROW_MAX = 256;  // rows that can get a workgroup of 1024 threads each (stats_plan)

template <typename T, int TPB, bool VECTOR, int PER_UNIT = 8, bool AHEAD = false>
void launch_items(const T* logits, int rows, int vocab, int mask_id, const StatsPlan& p, const StatsRows& sr, const StatsOut& o, void* workspace, hipStream_t st) {
  // (the hardware dispatcher balances better than a resident grid walking the items)
  vocab_stats_kernel<T, TPB, VECTOR, PER_UNIT, AHEAD><<<rows * p.chunks, TPB, 0, st>>>(logits, vocab, mask_id, p.chunk, p.chunks, sr, o, (Part*)workspace);
  if (p.chunks > 1) vocab_stats_merge_kernel<<<rows, 64, 0, st>>>((const Part*)workspace, rows, p.chunks, vocab, sr, o);
}

}  // namespace

size_t stats_workspace_bytes(int rows) { return (size_t)rows * MAX_CHUNKS * sizeof(Part); }

void launch_stats_merge(const void* parts, int rows, int nparts, int vocab, const StatsRows& sr, const StatsOut& o, hipStream_t st) {
  vocab_stats_merge_kernel<<<rows, 64, 0, st>>>((const Part*)parts, rows, nparts, vocab, sr, o);
}

// How a row is cut.  The reduction is bound by its reads; what the cut decides is how evenly they lie on the chip and whether a
// second launch has to merge.  Chunks for about 1536 workgroups of 256 threads, each at least two vectors per lane, merged by a second
// kernel (4 us at 384 rows), are the general form; one chunk (a vocabulary of up to 4096 bf16 or 2048 fp32 logits) needs no merge.
// Where a merge would be needed, rows are read in 16-byte vectors and there is a row for most of the 256 compute units but no
// second round, one workgroup of 1024 threads takes a whole row and writes its results itself.  Microseconds of GPU time per call
// on logits in the memory-side cache, chunks -> whole rows, without / with a previous row:
//   bf16, 126464 tokens: 96 rows 13.0 -> 16.6 / 15.8 -> 20.4, 128: 16.2 -> 17.3 / 20.1 -> 20.8, 160: 18.2 -> 17.8 / 22.6 -> 20.9,
//   192: 17.6 -> 17.9 / 22.6 -> 21.6, 256: 22.2 -> 18.3 / 28.8 -> 24.9; 272 rows: 22.7 -> 31.2 / 31.4 -> 42.9 (a second round of
//   workgroups, as two of 1024 threads don't fit into a unit's registers).  These are with lane exchanges through LDS, which cost chunks more.
//   With the present ones and logits from memory: 136 rows 15.6 -> 17.6 / 20.0 -> 21.2, 152: 17.2 -> 17.8 / 21.9 -> 21.3, 192: 16.0 -> 18.1 /
//   23.1 -> 22.6, 256: 20.7 -> 18.5 / 29.7 -> 27.5; the mean of whole / chunks over 4 vocabularies, both types, without / with, is 0.99 at 136 rows,
//   0.96 at 152, 0.92 at 176, 0.94 at 192, 0.90 at 208, 0.87 at 224.  Single shapes lose up to 13 % below 200 rows; the line
//   stands where the mean first is ahead, and a row's values depend on it (the cut is the order of the sums).
// Without 16-byte vectors a lane has one scalar load in flight, and fewer lanes are what it loses by: 126463 tokens, bf16, 96 rows
//   20.5 -> 34.6 / 23.5 -> 58.9, 256: 44.2 -> 55.2 / 48.0 -> 60.0.  With one chunk the larger workgroup has nothing to save:
//   1024 tokens, fp32, 96 .. 256 rows 4.4 -> 6.4.
// A compute unit holds five workgroups of 256 threads (fp32: six), one more where that puts all of them on the chip at once.  One more
// always would leave other counts with a last round of few: 126464 tokens from memory, with a previous row, six a unit -> five: bf16,
// 384 rows (1536 workgroups) 40.3 -> 41.9, 768: 73.2 -> 77.0, 1536: 133.6 -> 141.1, but 896 (1792): 88.0 -> 83.4, 1756: 159.3 -> 152.8; seven ->
// six: fp32, 448 rows (1792) 81.6 -> 84.5, 896: 155.6 -> 161.3, but 1024 (2048): 182.1 -> 175.6, 2048: 355.3 -> 343.0.
// More rows keep their chunks.  A workgroup of 256 threads per row saves the merge there, but a lane then walks five times as far: each
// addend straight into the running sum, KL left 1e-5 of its value behind; a partial sum per vector first, all values were others than
// those of the same row in a call of fewer rows, and units that got a row more than the mean took longer (528 rows with a
// previous row, logits from memory: 57 -> 62 us).
StatsPlan stats_plan(int rows, int vocab, int elem_size) {
  const int n = 16 / elem_size;  // elements of a vector
  const int want = (1536 + rows - 1) / rows, most = (vocab + 512 * n - 1) / (512 * n);
  int nch = want < most ? want : most;
  if (nch > MAX_CHUNKS) nch = MAX_CHUNKS;
  if (nch < 1) nch = 1;
  StatsPlan p;
  p.vector = vocab % n == 0;
  p.threads = p.vector && nch > 1 && rows >= ROW_MIN && rows <= ROW_MAX ? 1024 : 256;
  if (p.threads == 1024) nch = 1;
  const int unit = p.threads * n;  // chunks are whole strides of the workgroup
  p.chunk = ((vocab + nch - 1) / nch + unit - 1) / unit * unit;
  p.chunks = (vocab + p.chunk - 1) / p.chunk;
  const int held = elem_size == 2 ? HELD<bf16_t> : HELD<float>;
  const int64_t workgroups = (int64_t)rows * p.chunks;
  p.per_unit = workgroups > 256 * held && workgroups <= 256 * (held + 1) ? held + 1 : held;
  return p;
}

// Whether a whole row's workgroup has the next trip's loads in flight while it absorbs one: where the wait for a trip shows, that is where
// the rows read, those of z and of z', are few; with more of them the reads are bound by bandwidth and more in flight only queue.
// us a call, waiting for each trip -> a trip ahead:
//   bf16, nothing compared, 126464 tokens: 136 rows 16.6 -> 15.7, 200: 17.0 -> 16.0, 256: 17.4 -> 17.2; 152064: 17.9 -> 16.5, 18.2 -> 16.9, 18.6 -> 17.9
//   bf16, all compared, 126464: 136 rows 20.0 -> 19.5, 152: 19.8 -> 19.9, 176: 20.2 -> 21.2, 208: 21.6 -> 22.5, 256: 24.8 -> 25.6; their
//     log-sum-exp recomputed, more arithmetic per byte: 136 rows 25.9 -> 24.8, 192: 26.0 -> 26.0, 224: 26.3 -> 26.8, 256: 27.1 -> 28.0
//   bf16, some compared, in a pass of a small model: 152 rows, 64 of them, 93.9 -> 93.3, 176, 64: 97.6 -> 96.9, 192, 128: 100.3 -> 100.8, 224,
//     64: 81.4 -> 82.2, 256, 64: 82.9 -> 85.0; of a 7B one 152, 64: 28.0 -> 24.3 the launch
//   fp32, nothing compared, 126464: 136 rows 16.8 -> 15.9, 192: 19.1 -> 18.9, 224: 20.9 -> 21.2, 256: 23.3 -> 24.4; any compared (136 .. 256
//     rows, 32 to all of them) loses 1 to 9 %: all of 152 26.0 -> 28.1, of 256 41.1 -> 41.3.
// The same additions in the same order, and so the same values, either way.
template <typename T>
bool loads_ahead(int rows, int compared, bool lse_given) {
  if (sizeof(T) == 4) return compared == 0 && rows <= 200;
  return compared == 0 || (rows <= 192 && rows + compared <= (lse_given ? 304 : 384));
}

template <typename T>
void launch_vocab_stats(const T* logits, int rows, int compared, int vocab, int mask_id, const StatsRows& sr, const StatsOut& o, void* workspace, hipStream_t st) {
  const StatsPlan p = stats_plan(rows, vocab, sizeof(T));
  if (p.threads == 1024 && loads_ahead<T>(rows, compared, sr.prev_lse != nullptr)) launch_items<T, 1024, true, 8, true>(logits, rows, vocab, mask_id, p, sr, o, workspace, st);
  else if (p.threads == 1024) launch_items<T, 1024, true>(logits, rows, vocab, mask_id, p, sr, o, workspace, st);
  else if (p.vector && p.per_unit > HELD<T>) launch_items<T, 256, true, HELD<T> + 1>(logits, rows, vocab, mask_id, p, sr, o, workspace, st);
  else if (p.vector) launch_items<T, 256, true, HELD<T>>(logits, rows, vocab, mask_id, p, sr, o, workspace, st);
  else launch_items<T, 256, false>(logits, rows, vocab, mask_id, p, sr, o, workspace, st);
}

template void launch_vocab_stats<float>(const float*, int, int, int, int, const StatsRows&, const StatsOut&, void*, hipStream_t);
template void launch_vocab_stats<bf16_t>(const bf16_t*, int, int, int, int, const StatsRows&, const StatsOut&, void*, hipStream_t);
