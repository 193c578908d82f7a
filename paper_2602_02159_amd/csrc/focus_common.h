// Shared device helpers for the gfx950 kernels: bf16 packing, wavefront (64-lane) and workgroup
// reductions / scans, MFMA operand types.  Device code only; wavefront size is 64 throughout.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace focus {

constexpr int kWave = 64;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// ---- bf16 <-> fp32 -------------------------------------------------------------------------------
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// round-to-nearest-even fp32 -> bf16 bits (NaN stays NaN)
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7fffffffu) > 0x7f800000u) return (u >> 16) | 0x40u;
  return (u + 0x7fffu + ((u >> 16) & 1u)) >> 16;
}
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  return f32_to_bf16_bits(lo) | (f32_to_bf16_bits(hi) << 16);
}

// 8 bf16 (one 16-byte vector) widened into 8 floats, added into acc
__device__ __forceinline__ void add_bf16x8(float (&acc)[8], const uint4& v) {
  acc[0] += bf16_lo(v.x); acc[1] += bf16_hi(v.x);
  acc[2] += bf16_lo(v.y); acc[3] += bf16_hi(v.y);
  acc[4] += bf16_lo(v.z); acc[5] += bf16_hi(v.z);
  acc[6] += bf16_lo(v.w); acc[7] += bf16_hi(v.w);
}

__device__ __forceinline__ bf16x8 as_bf16x8(const uint4& v) { return __builtin_bit_cast(bf16x8, v); }

// 16-byte streaming load with the non-temporal hint: the data is read once and should not displace reusable
// lines from the caches (measured +7% read bandwidth on a pure scan).
__device__ __forceinline__ uint4 load_stream16(const void* p) {
  typedef unsigned v4u __attribute__((ext_vector_type(4)));
  const v4u t = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(p));
  return make_uint4(t.x, t.y, t.z, t.w);
}

// ---- wavefront reductions ------------------------------------------------------------------------
// Fixed butterfly order, so results do not depend on scheduling.
__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}
__device__ __forceinline__ uint32_t wave_sum_u32(uint32_t v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, kWave);
  return v;
}

template <int CTRL>
__device__ __forceinline__ float lane_dpp(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, 0xF, 0xF, false));
}

// sum of x over the 16 lanes of a DPP row (the lanes that hold the 16 queries of a tile for the same keys); every
// lane of the row receives the total
__device__ __forceinline__ float row_sum16(float x) {
  x += lane_dpp<0xB1>(x);   // quad_perm [1,0,3,2]
  x += lane_dpp<0x4E>(x);   // quad_perm [2,3,0,1]
  x += lane_dpp<0x141>(x);  // row_half_mirror
  x += lane_dpp<0x140>(x);  // row_mirror
  return x;
}

// op over the 16 lanes of a DPP row / over the wavefront (op commutative and associative); every lane receives the result
template <class Op>
__device__ __forceinline__ uint32_t row_reduce_u32(uint32_t x, const Op op) {
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, false));   // quad_perm [1,0,3,2]
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, false));   // quad_perm [2,3,0,1]
  x = op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xF, 0xF, false));  // row_half_mirror
  return op(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x140, 0xF, 0xF, false));  // row_mirror
}
template <class Op>
__device__ __forceinline__ uint32_t wave_reduce_u32(uint32_t x, const Op op) {
  typedef unsigned v2u __attribute__((ext_vector_type(2)));
  x = row_reduce_u32(x, op);
  const v2u a = __builtin_amdgcn_permlane32_swap(x, x, false, false);
  x = op(a.x, a.y);
  const v2u b = __builtin_amdgcn_permlane16_swap(x, x, false, false);
  return op(b.x, b.y);
}

// Reductions over the 4 lanes with the same lane % 16, via v_permlane32_swap / v_permlane16_swap:
// swap(x, x) returns {value of the partner in the even half/row, value of the partner in the odd half/row}.
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ float group_max(float v) {
  uintx2 a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a.x), __uint_as_float(a.y));
  uintx2 b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b.x), __uint_as_float(b.y));
}
__device__ __forceinline__ float group_sum(float v) {
  uintx2 a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a.x) + __uint_as_float(a.y);
  uintx2 b = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b.x) + __uint_as_float(b.y);
}

// Workgroup exclusive scan of one uint32 per thread.  `wsum` is shared memory of at least
// blockDim/64 + 1 words.  Returns the exclusive prefix; *total gets the sum over the workgroup.
// Contains two barriers: every thread of the workgroup must call it.
__device__ __forceinline__ uint32_t block_exclusive_scan(uint32_t v, uint32_t* wsum, uint32_t* total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  uint32_t incl = v;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    uint32_t t = __shfl_up(incl, o, kWave);
    if (lane >= o) incl += t;
  }
  __syncthreads();  // wsum may still be read from a previous call
  if (lane == 63) wsum[wid] = incl;
  __syncthreads();
  uint32_t base = 0, tot = 0;
  for (int w = 0; w < nw; ++w) {
    uint32_t s = wsum[w];
    if (w < wid) base += s;
    tot += s;
  }
  *total = tot;
  return base + incl - v;
}

// Workgroup exclusive prefix COUNT of one flag per thread, from wavefront ballots: one LDS write, one barrier
// pair and at most blockDim/64 LDS reads per thread.  `wsum` is shared memory of at least 2 * (blockDim/64)
// words.  Every thread of the workgroup must call it.
__device__ __forceinline__ uint32_t block_flag_scan(bool flag, uint32_t* wsum, uint32_t* total) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6, nw = (blockDim.x + 63) >> 6;
  const unsigned long long b = __ballot(flag);
  __syncthreads();  // wsum may still be read from a previous call
  if (lane == 0) wsum[wid] = (uint32_t)__popcll(b);
  __syncthreads();
  uint32_t base = 0, tot = 0;
  for (int w = 0; w < nw; ++w) {
    const uint32_t s = wsum[w];
    if (w < wid) base += s;
    tot += s;
  }
  *total = tot;
  return base + (uint32_t)__popcll(b & ((1ull << lane) - 1ull));
}

// Softmax statistics of the key splits: float2 (maximum, sum) [H, n_split, q_pad], so that neighbouring threads read neighbouring
// queries.  An empty split holds (-inf, 0).
struct RowState {
  float m, l;
};
// adds N of them without a branch; those without a positive sum (empty, NaN) count for nothing
template <int N>
__device__ __forceinline__ void add_splits(RowState& r, const float2 (&v)[N]) {
  float m = r.m;
#pragma unroll
  for (int u = 0; u < N; ++u) m = fmaxf(m, v[u].y > 0.f ? v[u].x : -INFINITY);
  const float z = m == -INFINITY ? 0.f : m;
  float l = r.l * __builtin_amdgcn_exp2f(r.m - z);
#pragma unroll
  for (int u = 0; u < N; ++u) l += v[u].y > 0.f ? v[u].y * __builtin_amdgcn_exp2f(v[u].x - z) : 0.f;
  r.m = m;
  r.l = l;
}
__device__ __forceinline__ float lse_of(const RowState& r) { return r.l > 0.f ? r.m + __builtin_amdgcn_logf(r.l) : INFINITY; }  // v_log_f32 is log2
// splits first, first + step, ... of one row, N loads at a time; `row` = its place in the first split, `stride` = rows per split.
// FENCE: a scheduling fence keeps the loads of a batch together.  Without it the compiler waited for each of them in the variants of
// column_mass_kernel that hold few heads, to stay within 64 registers, and a batch was eight memory round trips.  Where they are
// together anyway it costs a little (32 heads, 8256 keys, one-layer step: 0.3 of 41 us).
constexpr int kSplitsInFlight = 8;
template <int N = kSplitsInFlight, bool FENCE = false>
__device__ __forceinline__ RowState add_row_splits(const float2* row, int64_t stride, int first, int step, int n_split) {
  RowState r{-INFINITY, 0.f};
  for (int s0 = first; s0 < n_split; s0 += N * step) {
    float2 v[N];
#pragma unroll
    for (int u = 0; u < N; ++u) {
      const int s = s0 + u * step;
      v[u] = row[(int64_t)min(s, n_split - 1) * stride];
      if (!FENCE && s >= n_split) v[u] = make_float2(-INFINITY, 0.f);
    }
    if (FENCE) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < N; ++u)
        if (s0 + u * step >= n_split) v[u] = make_float2(-INFINITY, 0.f);
    }
    add_splits(r, v);
  }
  return r;
}

// =====================================================================================================
// Helpers shared by the block-relevance kernels and the attention kernel that works the relevances out itself, written once so that the
// K-scanning and the cached-means variants produce bit-identical partial relevances.
// =====================================================================================================
// Sum over the focus queries of Q[h, i, 8c .. 8c+7] by one wavefront, for the calling lane's chunk c = lane % (D/8): lane (r, c)
// adds up the list entries r, r + R, r + 2 R, ... (U row loads in flight at a time), then the R lanes of a chunk meet (fixed
// tree; every lane receives the total).  `entry` = focus_idx[lane], fetched by the caller ahead of time (any value past the list).
template <int D, int U>
__device__ __forceinline__ void add_focus_rows(float (&qs)[8], const uint16_t* __restrict__ qh, int64_t qsn,
                                               const int32_t* __restrict__ focus_idx, int entry, int n_f, int n_gen) {
  constexpr int CPR = D / 8, R = kWave / CPR;
  static_assert(kWave % (R * U) == 0, "a batch lies within the entries a wavefront holds, or behind them");
  const int lane = threadIdx.x & 63, c = lane % CPR, r = lane / CPR;
  for (int f0 = 0; f0 < n_f; f0 += R * U) {  // uniform
    int row[U];
    if (f0 < kWave) {
#pragma unroll
      for (int u = 0; u < U; ++u) row[u] = __shfl(entry, f0 + u * R + r, kWave);
    } else {
#pragma unroll
      for (int u = 0; u < U; ++u) row[u] = f0 + u * R + r < n_f ? focus_idx[f0 + u * R + r] : -1;
    }
    uint4 v[U];
#pragma unroll
    for (int u = 0; u < U; ++u)
      v[u] = (f0 + u * R + r < n_f && row[u] >= 0 && row[u] < n_gen) ? *reinterpret_cast<const uint4*>(qh + (int64_t)row[u] * qsn + c * 8)
                                                                     : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int u = 0; u < U; ++u) add_bf16x8(qs, v[u]);
  }
}
template <int D, bool MANY>  // MANY: twice the loads in flight for lists longer than 4 R entries
__device__ __forceinline__ void focus_row_sum(float (&qs)[8], const uint16_t* __restrict__ qh, int64_t qsn,
                                              const int32_t* __restrict__ focus_idx, int entry, int n_f, int n_gen) {
  constexpr int CPR = D / 8, R = kWave / CPR;
#pragma unroll
  for (int e = 0; e < 8; ++e) qs[e] = 0.f;
  if (MANY && n_f > 4 * R)
    add_focus_rows<D, 8>(qs, qh, qsn, focus_idx, entry, n_f, n_gen);
  else
    add_focus_rows<D, 4>(qs, qh, qsn, focus_idx, entry, n_f, n_gen);
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    if (CPR == 8)  // lanes 8 apart: a rotation of the DPP row
      qs[e] += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, qs[e]), 0x128, 0xF, 0xF, false));
    qs[e] = group_sum(qs[e]);
  }
}

// dot product of one 8-wide chunk, fixed fused-multiply-add order, then the sum over the CPR lanes of a block row
template <int CPR>
__device__ __forceinline__ float chunk_dot_reduce(const float (&qs)[8], const float4& k0, const float4& k1) {
  float dot = qs[0] * k0.x;
  dot = __builtin_fmaf(qs[1], k0.y, dot);
  dot = __builtin_fmaf(qs[2], k0.z, dot);
  dot = __builtin_fmaf(qs[3], k0.w, dot);
  dot = __builtin_fmaf(qs[4], k1.x, dot);
  dot = __builtin_fmaf(qs[5], k1.y, dot);
  dot = __builtin_fmaf(qs[6], k1.z, dot);
  dot = __builtin_fmaf(qs[7], k1.w, dot);
  if (CPR == 16) return row_sum16(dot);
  dot += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, dot), 0xB1, 0xF, 0xF, false));   // quad_perm [1,0,3,2]
  dot += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, dot), 0x4E, 0xF, 0xF, false));   // quad_perm [2,3,0,1]
  dot += __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, dot), 0x141, 0xF, 0xF, false));  // row_half_mirror
  return dot;
}

}  // namespace focus
