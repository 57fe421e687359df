// Epilogues of a bf16 model's GEMM kernels, on finished values in the accumulator layout of
// v_mfma_f32_16x16x32_f16 (transposed product): in a 16 x 16 output tile, lane ml + 16 g holds
// columns 4g .. 4g+3 of row ml.
#pragma once
#include <type_traits>

#include "common.h"

__device__ inline bf16x4 to_bf16x4(f32x4 v) { return bf16x4{(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]}; }
__device__ inline f16x4 to_f16x4_sat(f32x4 v) { return f16x4{to_f16_sat(v[0]), to_f16_sat(v[1]), to_f16_sat(v[2]), to_f16_sat(v[3])}; }

// a fragment's 16 bytes of this lane; NT: past the memory-side cache
template <bool NT>
__device__ __attribute__((always_inline)) inline op8 load_weight(const op8* p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}

// ---- exchanges between the lanes of a wavefront, on fragments in the accumulator layout (all 64 lanes together)
// The halves of two fragments: lo = the lower 32 lanes' values of u and, in the upper 32 lanes, of v; hi = the upper 32 lanes'.  So
// where a fragment's columns 0 .. 7 meet its columns 8 .. 15 (gate and up, rotary partners), each lane gets one pair.
struct Halves { f32x4 lo, hi; };
__device__ __attribute__((always_inline)) inline Halves pair_halves(f32x4 u, f32x4 v) {
  Halves r;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    const auto x = __builtin_amdgcn_permlane32_swap(__float_as_uint(u[t]), __float_as_uint(v[t]), false, false);
    r.lo[t] = __uint_as_float(x[0]);
    r.hi[t] = __uint_as_float(x[1]);
  }
  return r;
}
// Two groups of 16-bit values per lane -> 16 consecutive bytes per lane: the lanes of group g (16 lanes each) get group 2 (g / 2)'s
// and then group 2 (g / 2) + 1's values, of u where g is even and of v where it is odd.
template <typename V4>
__device__ __attribute__((always_inline)) inline auto join_slots(V4 u, V4 v) {
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  typedef unsigned int u32x4_ __attribute__((ext_vector_type(4)));
  typedef typename std::conditional<std::is_same<V4, bf16x4>::value, bf16x8, f16x8>::type V8;
  const u32x2 a = __builtin_bit_cast(u32x2, u), b = __builtin_bit_cast(u32x2, v);
  const auto x = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false), y = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
  const u32x4_ o = {x[0], y[0], x[1], y[1]};
  return __builtin_bit_cast(V8, o);
}
template <int CTRL>
__device__ __attribute__((always_inline)) inline unsigned dpp(unsigned v) {
  return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, false);
}
// 4 x 4 transpose within each quad of lanes: lane q of the quad gets element q of its four lanes
__device__ __attribute__((always_inline)) inline f16x4 transpose_quad(f16x4 v) {
  typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
  const u32x2 a = __builtin_bit_cast(u32x2, v);
  const bool up = threadIdx.x & 2, odd = threadIdx.x & 1;
  const unsigned got = dpp<0x4e>(up ? a[0] : a[1]);  // quad_perm [2, 3, 0, 1]
  const unsigned r0 = up ? got : a[0], r1 = up ? a[1] : got;
  const unsigned sel = odd ? 0x03020706u : 0x05040100u;
  const u32x2 o = {__builtin_amdgcn_perm(dpp<0xb1>(r0), r0, sel), __builtin_amdgcn_perm(dpp<0xb1>(r1), r1, sel)};  // quad_perm [1, 0, 3, 2]
  return __builtin_bit_cast(f16x4, o);
}
__device__ __attribute__((always_inline)) inline void quad_rows(int v, int (&out)[4]) {  // the quad's four values, in every lane of it
  out[0] = (int)dpp<0x00>((unsigned)v);
  out[1] = (int)dpp<0x55>((unsigned)v);
  out[2] = (int)dpp<0xaa>((unsigned)v);
  out[3] = (int)dpp<0xff>((unsigned)v);
}
// sum over the four lanes of a row: lanes 16 apart, then lanes 32 apart
__device__ __attribute__((always_inline)) inline float sum_row4(float v) {
  auto x = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  const float s = __uint_as_float(x[0]) + __uint_as_float(x[1]);
  x = __builtin_amdgcn_permlane32_swap(__float_as_uint(s), __float_as_uint(s), false, false);
  return __uint_as_float(x[0]) + __uint_as_float(x[1]);
}

// 1/rms of rows [m_lo, m_lo + rows) from the producer's partial sums of squares into s_rinv, by the whole workgroup of NT
// threads: sixteen lanes per row, each adding every sixteenth chunk in ascending order, then a fixed butterfly
// (deterministic).  A lane's sixteen loads of a block of 256 chunks are issued together and waited for once: one trip to
// memory per block instead of one per chunk.
template <int NT>
__device__ inline void block_rinv(const RowScale& rs, int m_lo, int rows, float* s_rinv) {
  const int sub = threadIdx.x & 15;
  for (int row = threadIdx.x >> 4; row < rows; row += NT / 16) {
    float ss = 0.f;
    if (rs.ssq) {
      const float* src = rs.ssq + (size_t)(m_lo + row) * rs.nch;
      for (int c0 = 0; c0 < rs.nch; c0 += 256) {
        float v[16];
#pragma unroll
        for (int k = 0; k < 16; ++k) {
          const int c = c0 + sub + 16 * k;
          v[k] = c < rs.nch ? src[c] : 0.f;
        }
#pragma unroll
        for (int k = 0; k < 16; ++k) ss += v[k];
      }
    }
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
    if (sub == 0) s_rinv[row] = rs.ssq ? rsqrtf(ss * rs.inv_d + rs.eps) : 1.f;
  }
}

// block_rinv in two parts, for a workgroup of NT threads and at most ROWS rows of up to 16 CH chunks each, so that a kernel can do its
// work in between: fetch issues all of a thread's loads and touches none of what they bring, publish adds the values (sixteen lanes per
// row, each every sixteenth chunk in ascending order, then block_rinv's butterfly, here by lane rotation: after the first step the
// values repeat every eight lanes, and so on, so the sums are the same) and writes the rows' values.  (block_rinv in front of a loop,
// which the compiler makes a chain of up to sixteen trips, kept the wavefronts that run it from their weights.)
template <int NT, int ROWS, int CH = 4>
struct RinvBatch {
  static constexpr int RPT = (ROWS + NT / 16 - 1) / (NT / 16);  // rows per thread
  static constexpr int LOADS = RPT * CH;
  float v[RPT][CH];
  static __device__ inline bool fits(const RowScale& rs) { return rs.nch <= 16 * CH; }
  __device__ __attribute__((always_inline)) inline void fetch(const RowScale& rs, int m_lo, int rows) {
    if (rs.ssq) fetch(rs.ssq, rs.nch, m_lo, rows);
  }
  // ... with no path around the loads, which the compiler's count of loads in flight could not follow (it would let the first products
  // wait for all of them): where there are no sums of squares, `any_floats` (at least one of them) is read instead
  __device__ __attribute__((always_inline)) inline void fetch_always(const RowScale& rs, int rows, const void* any_floats) {
    const bool there = rs.ssq != nullptr;
    fetch(there ? rs.ssq : (const float*)any_floats, there ? rs.nch : 1, 0, there ? rows : 1);
  }
  __device__ __attribute__((always_inline)) inline void fetch(const float* ssq, int nch, int m_lo, int rows) {
    const int sub = threadIdx.x & 15;
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      const int row = (threadIdx.x >> 4) + r * (NT / 16);
      const float* src = ssq + (size_t)(m_lo + min(row, rows - 1)) * nch;
#pragma unroll
      for (int k = 0; k < CH; ++k) v[r][k] = src[min(sub + 16 * k, nch - 1)];  // (past the end: the last one, left out below)
    }
  }
  template <int CTRL>
  static __device__ inline float rotate_add(float a) { return a + __uint_as_float(dpp<CTRL>(__float_as_uint(a))); }
  __device__ __attribute__((always_inline)) inline void publish(const RowScale& rs, int rows, float* s_rinv) const {
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      const int row = (threadIdx.x >> 4) + r * (NT / 16);
      float ss = 0.f;
#pragma unroll
      for (int k = 0; k < CH; ++k) ss += (int)(threadIdx.x & 15) + 16 * k < rs.nch ? v[r][k] : 0.f;
      finish(rs, row, rows, ss, s_rinv);
    }
  }
  // ... for rows of any number of chunks (a model of d_model > 4096 has more than 256 from a skinny product, more than 64 from a mid one):
  // those beyond the batch are read here, four of every row in a trip, and added behind the batch's.  d_model 5120, 64 rows, gate/up behind
  // 320 chunks and QKV behind 320: 56.0 and 31.7 us with the batch left unused and block_rinv behind the loop, 52.0 and 30.0 so (with
  // eight in a trip 52.3 and 30.2); 20 rows 50.0 and 20.0 -> 48.5 and 19.7.
  __device__ __attribute__((always_inline)) inline void publish_all(const RowScale& rs, int rows, float* s_rinv) const {
    constexpr int TAIL = 4;
    const int sub = threadIdx.x & 15;
    float ss[RPT];
#pragma unroll
    for (int r = 0; r < RPT; ++r) {
      ss[r] = 0.f;
#pragma unroll
      for (int k = 0; k < CH; ++k) ss[r] += sub + 16 * k < rs.nch ? v[r][k] : 0.f;
    }
    if (rs.ssq)
      for (int c0 = 16 * CH; c0 < rs.nch; c0 += 16 * TAIL) {
        float t[RPT][TAIL];
#pragma unroll
        for (int r = 0; r < RPT; ++r) {
          const float* src = rs.ssq + (size_t)min((int)(threadIdx.x >> 4) + r * (NT / 16), rows - 1) * rs.nch;
#pragma unroll
          for (int k = 0; k < TAIL; ++k) t[r][k] = src[min(c0 + sub + 16 * k, rs.nch - 1)];
        }
#pragma unroll
        for (int r = 0; r < RPT; ++r)
#pragma unroll
          for (int k = 0; k < TAIL; ++k) ss[r] += c0 + sub + 16 * k < rs.nch ? t[r][k] : 0.f;
      }
#pragma unroll
    for (int r = 0; r < RPT; ++r) finish(rs, (threadIdx.x >> 4) + r * (NT / 16), rows, ss[r], s_rinv);
  }

 private:
  static __device__ __attribute__((always_inline)) inline void finish(const RowScale& rs, int row, int rows, float ss, float* s_rinv) {
    // row_ror:8, 4, 2, 1
    ss = rotate_add<0x121>(rotate_add<0x122>(rotate_add<0x124>(rotate_add<0x128>(ss))));
    if ((threadIdx.x & 15) == 0 && row < rows) s_rinv[row] = rs.ssq ? rsqrtf(ss * rs.inv_d + rs.eps) : 1.f;
  }
};

// What an epilogue reads from memory besides the product, fetched ahead (at the start of the kernel, while the first weights
// are in flight) for the fragment a wavefront finishes first, so that the end of a short kernel does not wait for a round
// trip: EPI_RESID the four residual values and gains of the lane, EPI_QKV the lane's rotary cosines and sines and, for the
// K and V heads, the row's position and cache slot.
struct EpiAhead {
  f32x4 a, b;
  bool have;
  int pos, slot;  // EPI_QKV, K and V heads: the row's position and cache slot (-1: not fetched)
};
__device__ inline EpiAhead epi_none() { return EpiAhead{f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}, false, -1, -1}; }
template <int EPI>
__device__ inline EpiAhead epi_ahead(const GemmEpi& e, int M, int N, int m, int nc, int g) {
  EpiAhead r = epi_none();
  if (EPI == EPI_RESID) {
    if (m < M && nc < N) {
      r.a = *(const f32x4*)(e.h + (size_t)m * N + nc + 4 * g);
      r.b = *(const f32x4*)(e.gain + nc + 4 * g);
      r.have = true;
    }
  } else if (EPI == EPI_QKV) {
    const int hd = e.hd, half = hd >> 1;
    if (m < M && nc < N && g < 2) {
      const int head = nc / hd;
      if (head < e.n_q + e.n_kv) {
        const int i = 8 * ((nc % hd) >> 4) + 4 * g;
        r.a = *(const f32x4*)(e.rope_cos + (size_t)m * half + i);
        r.b = *(const f32x4*)(e.rope_sin + (size_t)m * half + i);
        r.have = true;
      }
      if (head >= e.n_q) {
        r.pos = e.row_pos[m];
        r.slot = e.row_slot[m];
      }
    }
  }
  return r;
}

// Rotary pair group: a = packed columns nc+4gp .. +3 of a 16-column tile starting at packed column nc,
// b = the same + 8; they are dims i .. i+3 and i+half .. i+half+3 of one head (weights packed with PERM_ROTARY).
__device__ inline void finish_qkv(const GemmEpi& e, int m, int nc, int gp, f32x4 a, f32x4 b, const EpiAhead ahead = epi_none()) {
  const int hd = e.hd, half = hd >> 1;
  const int head = nc / hd, i = 8 * ((nc % hd) >> 4) + 4 * gp;
  if (head < e.n_q + e.n_kv) {
    const bool pre = ahead.have;
    const f32x4 c = pre ? ahead.a : *(const f32x4*)(e.rope_cos + (size_t)m * half + i);
    const f32x4 sn = pre ? ahead.b : *(const f32x4*)(e.rope_sin + (size_t)m * half + i);
    const f32x4 ra = a * c - b * sn, rb = b * c + a * sn;
    a = ra;
    b = rb;
  }
  const f16x4 ab = to_f16x4_sat(a), bb = to_f16x4_sat(b);
  if (head < e.n_q) {
    *(f16x4*)(e.q + tile_index(m, head * hd + i, e.n_q * hd)) = ab;
    *(f16x4*)(e.q + tile_index(m, head * hd + i + half, e.n_q * hd)) = bb;
    return;
  }
  const bool is_k = head < e.n_q + e.n_kv;
  const int kvh = is_k ? head - e.n_q : head - e.n_q - e.n_kv;
  // (a load here, between the stores of two fragments, has to wait for every store before it: the memory counter retires in order)
  const int pos = ahead.pos >= 0 ? ahead.pos : e.row_pos[m];
  const int slot = ahead.pos >= 0 ? ahead.slot : e.row_slot[m];
  f16_t* dst = (is_k ? e.kcache : e.vcache) + (size_t)slot * e.slot_stride + (size_t)kvh * e.head_stride;
  if (is_k) {  // four consecutive dims share a lane slot of the K tiling
    *(f16x4*)(dst + kv_k_index(pos, i, hd)) = ab;
    *(f16x4*)(dst + kv_k_index(pos, i + half, hd)) = bb;
  } else {
    // dims i .. i+3 (i a multiple of 4) lie in one 16-dim tile: consecutive dims are 8 elements apart (kv_v_index)
    const size_t va = kv_v_index(pos, i, hd), vb = kv_v_index(pos, i + half, hd);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      dst[va + 8 * j] = ab[j];
      dst[vb + 8 * j] = bb[j];
    }
  }
}

// gate = packed columns nc+4gp .. +3, up = the same + 8: output columns 8 (nc/16) + 4gp .. +3 (weights packed with PERM_GATED)
__device__ inline f32x4 gated(f32x4 g, f32x4 u) {
  f32x4 a;
#pragma unroll
  for (int t = 0; t < 4; ++t) a[t] = g[t] * __builtin_amdgcn_rcpf(1.f + __expf(-g[t])) * u[t];  // (the hardware reciprocal: 1 ulp)
  return a;
}
__device__ inline void finish_swiglu(const GemmEpi& e, int m, int nc, int gp, f32x4 g, f32x4 u) {
  *(op4*)(e.act + tile_index(m, 8 * (nc >> 4) + 4 * gp, e.ffn)) = to_f16x4_sat(gated(g, u));
}

// residual add and next norm's x for columns n .. n+3 of row m; returns the four columns' share of sum h^2
__device__ inline float finish_resid(const GemmEpi& e, int m, int n, int N, f32x4 y, const EpiAhead ahead = epi_none()) {
  const size_t o = (size_t)m * N + n;
  const bool pre = ahead.have;
  const f32x4 v = (pre ? ahead.a : *(const f32x4*)(e.h + o)) + y;
  *(f32x4*)(e.h + o) = v;
  const f32x4 g = pre ? ahead.b : *(const f32x4*)(e.gain + n);
  *(op4*)(e.x + tile_index(m, n, N)) = to_f16x4_sat(v * g);
  return v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
}

__device__ inline void finish_sum(const GemmEpi& e, int m, int n, int N, f32x4 v) {
  *(bf16x4*)(e.out_bf16 + (size_t)m * N + n) = to_bf16x4(v);
}

// One 16 x 16 tile starting at packed column nc: v = this lane's four finished columns of row m, rinv = 1/rms of the input row.
// Called by all 64 lanes of a wavefront together (it exchanges values between lanes).  EPI_RESID returns the tile's share of
// sum h^2 of row m (in every lane of the row), the others 0.
template <int EPI>
__device__ inline float finish_frag(const GemmEpi& e, int M, int N, int m, int nc, int g, f32x4 v, float rinv, const EpiAhead ahead = epi_none()) {
  if (EPI == EPI_QKV || EPI == EPI_SWIGLU) {
    const f32x4 b = pair_halves(v, v).hi;  // the partner group, columns + 8, sits 32 lanes up
    if (g < 2 && m < M) {
      if (EPI == EPI_QKV) finish_qkv(e, m, nc, g, v * rinv, b * rinv, ahead);
      else finish_swiglu(e, m, nc, g, v * rinv, b * rinv);
    }
    return 0.f;
  }
  if (EPI == EPI_RESID) {
    return sum_row4(m < M ? finish_resid(e, m, nc + 4 * g, N, v, ahead) : 0.f);
  }
  if (m < M) finish_sum(e, m, nc + 4 * g, N, v * rinv);
  return 0.f;
}
