// Selection, block-mean, block-relevance and column-mass kernels: the stages of the step that are either
// pure HBM scans or a few KB of latency-bound integer work.  None of them is a dense contraction, so none
// uses MFMA; what matters is coalesced 16-byte loads, many loads in flight and fixed-order reductions.
#include "focus_cache.h"
#include "focus_common.h"
#include "focus_kernels.h"
#include "focus_topk.h"

namespace focus {

// =====================================================================================================
// Past-confidence-guided indicator (Sec. 5.2): Eq. 4 top-k over the still-masked positions, then the
// Eq. 5 window union clipped to [lo, hi).  One workgroup; everything stays in LDS.
// =====================================================================================================
// MAXN > 0: n_gen <= min(blockDim.x, MAXN) (the usual case, a generation block of 32..256 positions): the
// radix-select path and the strided window pass are not compiled in.
constexpr int kSelectMaxGen = 16384;

template <int MAXN>
__global__ __launch_bounds__(kTopkThreads) void select_queries_kernel(
    const float* __restrict__ conf, const uint8_t* __restrict__ masked, int n_gen, int k, int half, int lo, int hi,
    int32_t* __restrict__ focus_idx, int32_t* __restrict__ active_idx, int max_active, int32_t* __restrict__ counts) {
  __shared__ TopkShared sm;
  __shared__ uint8_t flags[MAXN > 0 ? MAXN : kSelectMaxGen];
  auto keyfn = [=](int i, uint32_t& key) -> bool {
    key = order_key(conf[i]);
    return masked == nullptr || masked[i] != 0;
  };
  block_topk<MAXN>(keyfn, n_gen, k, focus_idx, counts, flags, sm);  // ends with a barrier: flags are visible

  // window union: position p is active iff some focus position lies within `half` of it
  const int tid = threadIdx.x, nt = blockDim.x;
  const int n = hi - lo;
  const int chunk = (n + nt - 1) / nt;
  const int c0 = min(tid * chunk, n), c1 = min(c0 + chunk, n);
  auto is_active = [&](int p) -> bool {
    const int a = max(p - half, 0), b = min(p + half, n_gen - 1);
    for (int i = a; i <= b; ++i)
      if (flags[i]) return true;
    return false;
  };
  uint32_t total;
  if (MAXN > 0 || n <= nt) {
    const bool act = tid < n && is_active(lo + tid);
    const uint32_t pos = block_flag_scan(act, sm.wsum, &total);
    if (act) active_idx[pos] = lo + tid;
  } else {
    uint32_t cnt = 0;
    for (int j = c0; j < c1; ++j) cnt += is_active(lo + j);
    uint32_t pos = block_exclusive_scan(cnt, sm.wsum, &total);
    for (int j = c0; j < c1; ++j)
      if (is_active(lo + j)) active_idx[pos++] = lo + j;
  }
  for (int i = (int)total + tid; i < max_active; i += nt) active_idx[i] = -1;
  if (tid == 0) counts[1] = (int32_t)total;
}

// up to 64 positions: one wavefront, in registers (without LDS, flags and barriers: 64 positions, windows of nine
// 2.8 -> 2.2 us, of one 2.4 -> 2.1)
__global__ __launch_bounds__(64) void select_positions_kernel(const SelectArgs s, int n_gen, int max_active) {
  select_positions(s, n_gen, max_active, threadIdx.x, true);
}

hipError_t launch_select_queries(const float* conf, const uint8_t* masked, int n_gen, int k, int window, int lo,
                                 int hi, int32_t* focus_idx, int32_t* active_idx, int max_active, int32_t* counts,
                                 hipStream_t st) {
  const int threads = n_gen <= 256 ? 256 : kTopkThreads;
  if (n_gen <= kSelectInLogitsGen)
    hipLaunchKernelGGL(select_positions_kernel, dim3(1), dim3(64), 0, st, SelectArgs{conf, masked, k, window / 2, lo, hi, focus_idx, active_idx, counts},
                       n_gen, max_active);
  else if (n_gen <= 256)
    hipLaunchKernelGGL(select_queries_kernel<256>, dim3(1), dim3(threads), 0, st, conf, masked, n_gen, k, window / 2, lo, hi,
                       focus_idx, active_idx, max_active, counts);
  else if (n_gen <= threads)
    hipLaunchKernelGGL(select_queries_kernel<1024>, dim3(1), dim3(threads), 0, st, conf, masked, n_gen, k, window / 2, lo, hi,
                       focus_idx, active_idx, max_active, counts);
  else
    hipLaunchKernelGGL(select_queries_kernel<0>, dim3(1), dim3(threads), 0, st, conf, masked, n_gen, k, window / 2, lo,
                       hi, focus_idx, active_idx, max_active, counts);
  return hipGetLastError();
}

// Grouped-query attention: the `group` query heads that share a K/V head are presented to every other kernel as
// `group` times as many query rows of that head (row g * n_gen + i for position i of the g-th head of the group).
// This turns the index lists of the selection into lists of such rows: list entry a of head g lands at g * n + a,
// n the number of valid entries, so the output is ascending when the input is; the tail is filled with -1.
__global__ __launch_bounds__(256) void expand_groups_kernel(const int32_t* __restrict__ focus_idx, int max_focus,
                                                            const int32_t* __restrict__ active_idx, int max_active,
                                                            const int32_t* __restrict__ counts, int n_gen, int group,
                                                            int32_t* __restrict__ focus_out, int32_t* __restrict__ active_out,
                                                            int32_t* __restrict__ counts_out) {
  const int n_f = counts ? min(max(counts[0], 0), max_focus) : max_focus;
  const int n_a = counts ? min(max(counts[1], 0), max_active) : max_active;
  const int t = blockIdx.x * blockDim.x + threadIdx.x;
  if (t < group * max_focus) {
    int v = -1;
    if (t < group * n_f) {
      const int i = focus_idx[t % n_f];
      if (i >= 0 && i < n_gen) v = (t / n_f) * n_gen + i;
    }
    focus_out[t] = v;
  }
  if (t < group * max_active) {
    int v = -1;
    if (t < group * n_a) {
      const int i = active_idx[t % n_a];
      if (i >= 0 && i < n_gen) v = (t / n_a) * n_gen + i;
    }
    active_out[t] = v;
  }
  if (t == 0) {
    counts_out[0] = group * n_f;
    counts_out[1] = group * n_a;
  }
}

hipError_t launch_expand_groups(const int32_t* focus_idx, int max_focus, const int32_t* active_idx, int max_active,
                                const int32_t* counts, int n_gen, int group, int32_t* focus_out, int32_t* active_out,
                                int32_t* counts_out, hipStream_t st) {
  const int n = group * std::max(max_focus, max_active);
  hipLaunchKernelGGL(expand_groups_kernel, dim3(ceil_div(n, 256)), dim3(256), 0, st, focus_idx, max_focus, active_idx,
                     max_active, counts, n_gen, group, focus_out, active_out, counts_out);
  return hipGetLastError();
}

// =====================================================================================================
// Top-k over a float array that may first have to be assembled from partial sums:
//   values[j] = sum_{i < n_parts} part[i * n + j] / (|I_focus| n_heads)   (fixed order, see sum_partials), written to values_out,
// then Top-k over values[0..n).  With part == nullptr the values are read as they are.  One workgroup.
// Used for Top-C over R_b (partial relevances) and Top-N_sink over S_j (n_parts = 0).
// =====================================================================================================
template <int MAXN>  // MAXN > 0: n <= min(blockDim.x, MAXN), no radix-select code
__global__ __launch_bounds__(kTopkThreads) void reduce_topk_kernel(const float* __restrict__ part, int n_parts,
                                                                   int n_heads, const int32_t* __restrict__ counts, int n_focus_max,
                                                                   float* __restrict__ values, int n, int k,
                                                                   int32_t* __restrict__ out) {
  __shared__ TopkShared sm;
  const int tid = threadIdx.x, nt = blockDim.x;
  float mine = 0.f;
  if (part != nullptr) {
    const int n_f = counts ? min(max(counts[0], 0), n_focus_max) : n_focus_max;
    const float scale = n_f > 0 ? 1.f / ((float)n_f * (float)n_heads) : 0.f;
    for (int j = tid; j < n; j += nt) {
      float acc = sum_partials(part, n_parts, n_parts != n_heads, n, j);
      acc *= scale;
      values[j] = acc;
      mine = acc;  // the value of element tid when n <= nt
    }
    if (MAXN == 0 && n > nt) {  // the radix path re-reads values written by other threads of the workgroup
      __threadfence_block();
      __syncthreads();
    }
  } else if (tid < n) {
    mine = values[tid];
  }
  if (k <= 0) return;
  if (MAXN > 0 || n <= nt) {
    auto keyfn = [=](int, uint32_t& key) -> bool {  // only ever asked for i == tid on this path
      key = order_key(mine);
      return true;
    };
    block_topk<(MAXN > 0 ? MAXN : kTopkThreads)>(keyfn, n, k, out, nullptr, nullptr, sm);
  } else {
    auto keyfn = [=](int i, uint32_t& key) -> bool {
      key = order_key(values[i]);
      return true;
    };
    const bool aligned = (reinterpret_cast<uintptr_t>(values) & 15u) == 0;
    block_topk(keyfn, n, k, out, nullptr, nullptr, sm, aligned ? values : nullptr);
  }
}

// Per-head partial relevances [H, n_b] -> sums of groups of kRelGroup heads [ceil(H / 4), n_b], in the same place (a thread owns a block's column)
// and in the order of sum_partials.  Between a K scan and an attention kernel that ranks more than 256 blocks itself: one memory round trip in a
// launch of many workgroups, where a launch of one read all parts and ranked them (16 heads, 2048 blocks, whole layer with the scan 139.5 -> 125
// us; 32 heads, 512 blocks 60.8 -> 59.3).  Up to eight heads the attention kernel takes the parts as they are (with this launch and without: 8
// heads, 1870 blocks 62.8 and 61.2, 74.8 before; 4 heads, 512 blocks 21.4 and 19.7, 22.3 before; d = 64, 313 blocks 17.9 and 16.2, 18.4).
__global__ __launch_bounds__(64) void group_heads_kernel(float* __restrict__ part, int H, int n_b) {
  constexpr int kHeads = 32;
  const int b = blockIdx.x * 64 + (int)threadIdx.x;
  if (b >= n_b) return;
  for (int h0 = 0; h0 < H; h0 += kHeads) {
    float v[kHeads];
#pragma unroll
    for (int u = 0; u < kHeads; ++u) v[u] = part[(int64_t)min(h0 + u, H - 1) * n_b + b];
#pragma unroll
    for (int u = 0; u < kHeads; u += kRelGroup) {
      float g = v[u];
#pragma unroll
      for (int i = 1; i < kRelGroup; ++i) g = h0 + u + i < H ? g + v[u + i] : g;
      if (h0 + u < H) part[(int64_t)((h0 + u) / kRelGroup) * n_b + b] = g;
    }
  }
}
hipError_t launch_group_heads(float* part, int n_heads, int n_b, hipStream_t st) {
  hipLaunchKernelGGL(group_heads_kernel, dim3(ceil_div(n_b, 64)), dim3(64), 0, st, part, n_heads, n_b);
  return hipGetLastError();
}

hipError_t launch_reduce_topk(const float* part, int n_parts, int n_heads, const int32_t* counts, int n_focus_max, float* values, int n,
                              int k, int32_t* out, hipStream_t st) {
  const int threads = n <= 64 ? 64 : (n <= 256 ? 256 : kTopkThreads);
  if (n <= 256)
    hipLaunchKernelGGL(reduce_topk_kernel<256>, dim3(1), dim3(threads), 0, st, part, n_parts, n_heads, counts, n_focus_max, values, n, k,
                       out);
  else if (n <= threads)
    hipLaunchKernelGGL(reduce_topk_kernel<1024>, dim3(1), dim3(threads), 0, st, part, n_parts, n_heads, counts, n_focus_max, values, n,
                       k, out);
  else
    hipLaunchKernelGGL(reduce_topk_kernel<0>, dim3(1), dim3(threads), 0, st, part, n_parts, n_heads, counts, n_focus_max, values, n,
                       k, out);
  return hipGetLastError();
}

// =====================================================================================================
// Representative keys (Sec. 5.3): kbar[h, b, :] = mean of the prompt rows of block b.  A pure HBM scan:
// one workgroup per (block, head); every wave instruction reads 1 KB of consecutive bytes; eight
// independent 16-byte non-temporal loads per thread are in flight before the first add.
// WITH_REL: the same scan also emits the block's partial relevance part[h, b] = qsum^h . kbar^h_b (Eq. 7), so that
// scoring blocks from raw K needs one launch and never writes or re-reads kbar (kbar may then be null).
// =====================================================================================================
template <int D, bool WITH_REL>
__global__ __launch_bounds__(256, 8) void block_means_kernel(const uint16_t* __restrict__ K, int64_t sh, int64_t sn,
                                                          int M, int B, int n_b, float* __restrict__ kbar,
                                                          const uint16_t* __restrict__ Q, int64_t qsh, int64_t qsn,
                                                          const int32_t* __restrict__ focus_idx,
                                                          const int32_t* __restrict__ counts, int n_focus_max, int n_gen,
                                                          float* __restrict__ part) {
  constexpr int TPR = D / 8;      // threads per row (16 bytes each)
  constexpr int RPP = 256 / TPR;  // rows per pass of the workgroup
  constexpr int UNROLL = 8;
  __shared__ __attribute__((aligned(16))) float red[RPP][D];
  __shared__ __attribute__((aligned(16))) float kb_sh[WITH_REL ? D : 4];
  const int b = blockIdx.x, h = blockIdx.y;
  const int r0 = b * B;
  const int len = min(B, M - r0);
  const int c = threadIdx.x % TPR, rr = threadIdx.x / TPR;
  // the focus list that the first wavefront will need at the very end is fetched now, in the shadow of the K loads
  int entry = -1, n_f = 0;
  if (WITH_REL) {
    if ((int)threadIdx.x < min(n_focus_max, kWave)) entry = focus_idx[threadIdx.x];
    n_f = counts ? min(max(counts[0], 0), n_focus_max) : n_focus_max;
  }
  const uint16_t* base = K + (int64_t)h * sh + (int64_t)r0 * sn + c * 8;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int r = rr; r < len; r += RPP * UNROLL) {
    uint4 v[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const int row = r + u * RPP;
      v[u] = row < len ? load_stream16(base + (int64_t)row * sn) : make_uint4(0, 0, 0, 0);
    }
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) add_bf16x8(acc, v[u]);
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) red[rr][c * 8 + e] = acc[e];
  __syncthreads();
  if (threadIdx.x < D) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < RPP; ++i) s += red[i][threadIdx.x];
    const float mean = s / (float)len;
    if (kbar) kbar[((int64_t)h * n_b + b) * D + threadIdx.x] = mean;
    if (WITH_REL) kb_sh[threadIdx.x] = mean;
  }
  if (WITH_REL) {
    __syncthreads();  // kb_sh is complete
    if (threadIdx.x < kWave) {
      float qs[8];
      focus_row_sum<D, false>(qs, Q + (int64_t)h * qsh, qsn, focus_idx, entry, n_f, n_gen);
      const float4* kp = reinterpret_cast<const float4*>(kb_sh + c * 8);
      const float dot = chunk_dot_reduce<TPR>(qs, kp[0], kp[1]);
      if (threadIdx.x == 0) part[(int64_t)h * n_b + b] = dot;
    }
  }
}

hipError_t launch_block_means(const void* K, const focus_shape& s, float* kbar, hipStream_t st) {
  const int n_b = ceil_div(s.n_ctx, s.block);
  dim3 grid(n_b, s.n_heads);
  const uint16_t* k = static_cast<const uint16_t*>(K);
  if (s.head_dim == 128)
    hipLaunchKernelGGL((block_means_kernel<128, false>), grid, dim3(256), 0, st, k, s.k_stride_h, s.k_stride_n, s.n_ctx,
                       s.block, n_b, kbar, nullptr, 0, 0, nullptr, nullptr, 0, 0, nullptr);
  else
    hipLaunchKernelGGL((block_means_kernel<64, false>), grid, dim3(256), 0, st, k, s.k_stride_h, s.k_stride_n, s.n_ctx,
                       s.block, n_b, kbar, nullptr, 0, 0, nullptr, nullptr, 0, 0, nullptr);
  return hipGetLastError();
}

// block means and partial relevances in one scan of K (kbar may be null: the means are then not stored)
hipError_t launch_block_means_relevance(const void* K, const void* Q, const int32_t* focus_idx, const int32_t* counts,
                                        int n_focus_max, const focus_shape& s, float* kbar, float* part, hipStream_t st) {
  const int n_b = ceil_div(s.n_ctx, s.block);
  dim3 grid(n_b, s.n_heads);
  const uint16_t* k = static_cast<const uint16_t*>(K);
  const uint16_t* q = static_cast<const uint16_t*>(Q);
  if (s.head_dim == 128)
    hipLaunchKernelGGL((block_means_kernel<128, true>), grid, dim3(256), 0, st, k, s.k_stride_h, s.k_stride_n, s.n_ctx,
                       s.block, n_b, kbar, q, s.q_stride_h, s.q_stride_n, focus_idx, counts, n_focus_max, s.n_gen, part);
  else
    hipLaunchKernelGGL((block_means_kernel<64, true>), grid, dim3(256), 0, st, k, s.k_stride_h, s.k_stride_n, s.n_ctx,
                       s.block, n_b, kbar, q, s.q_stride_h, s.q_stride_n, focus_idx, counts, n_focus_max, s.n_gen, part);
  return hipGetLastError();
}

// The share of one workgroup in a cache update (cache_update_kernel): slots g kUpdateSlots .. of head h
template <int D>
constexpr int kUpdateSlots = 256 / (2 * (D / 8));
template <int D>
__device__ __forceinline__ void cache_update_part(const CacheUpdate& u, int g, int h) {
  constexpr int kChunks = D / 8, kPerSlot = 2 * kChunks;
  const int a = g * kUpdateSlots<D> + (int)threadIdx.x / kPerSlot;
  if (a >= u.max_active) return;
  const int t = (int)threadIdx.x % kPerSlot;
  const bool is_v = t >= kChunks;
  const int c = is_v ? t - kChunks : t;
  const uint4 x = *reinterpret_cast<const uint4*>((is_v ? u.Vn : u.Kn) + (int64_t)h * u.nsh + (int64_t)a * u.nsn + c * 8);
  const int i = u.active_idx[a];
  const int n_act = u.counts ? min(max(u.counts[1], 0), u.max_active) : u.max_active;
  const int64_t row = (int64_t)u.row_base + i;
  if (a >= n_act || i < 0 || row < 0 || row >= u.n_rows) return;
  uint16_t* dst = is_v ? u.Vc + (int64_t)h * u.vsh + row * u.vsn + c * 8 : u.Kc + (int64_t)h * u.ksh + row * u.ksn + c * 8;
  *reinterpret_cast<uint4*>(dst) = x;
}

// =====================================================================================================
// Block relevance (Eq. 7), partial sums: qsum^h . kbar^h_b with qsum^h the SUM of the focus queries of head h; the
// 1/(|I_focus| H) factor and the rest of the sum over heads are applied, in a fixed order, where the blocks are ranked.
// A wavefront owns one head and P R consecutive blocks (R = 4 at d = 128, 8 at 64), a lane one 8-wide slice of d of one block
// row; the focus indices and the kbar loads are issued first, then the focus rows of Q: two dependent memory round trips.
// PER_HEAD: part[h, b].  Otherwise the four heads of the workgroup meet in LDS and part[h / 4, b] is their sum, so that whoever
// ranks the blocks — every workgroup of the attention kernel, or a single one past kFusedMaxBlocks — has a quarter to read.
// Heads are the fast grid axis: workgroups go to the XCDs round-robin, so those of one head share an L2 and its focus rows.
// Sparse layer of 32 heads with 256 blocks 15.3 -> 14.9 us (a workgroup per head and 32 blocks, its 16 focus rows summed by all
// four wavefronts through LDS, and every attention workgroup adding 32 partial relevances per block), 4 heads at 1K 11.0 -> 10.4.
// Two passes: eight need fewer workgroups and read the focus rows less often, and take 0.3 us more from 64 to 1024 blocks.
// =====================================================================================================
constexpr int kRelPasses = 2;
template <int D, bool PER_HEAD>
__device__ __forceinline__ void relevance_partial(const int32_t* __restrict__ focus_idx, const float* __restrict__ kbar,
                                                  const int32_t* __restrict__ counts, const uint16_t* __restrict__ Q, int64_t qsh, int64_t qsn,
                                                  int n_b, int H, int n_focus_max, int n_gen, float* __restrict__ part) {
  constexpr int CPR = D / 8;        // lanes per block row
  constexpr int R = kWave / CPR;    // block rows per pass
  constexpr int P = kRelPasses;
  static_assert(kRelGroup * kWave == 256, "a wavefront per head of the group");
  __shared__ float dots[kRelGroup][P * R];
  const int lane = threadIdx.x & 63, c = lane % CPR, r = lane / CPR;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int h = blockIdx.x * kRelGroup + wave, b0 = grid_yz() * (P * R);
  if (h < H) {
    const int entry = lane < n_focus_max ? focus_idx[lane] : -1;
    const int n_f = counts ? min(max(counts[0], 0), n_focus_max) : n_focus_max;
    float4 k0[P], k1[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const float4* kp = reinterpret_cast<const float4*>(kbar + ((int64_t)h * n_b + min(b0 + p * R + r, n_b - 1)) * D + c * 8);
      k0[p] = kp[0];
      k1[p] = kp[1];
    }
    __builtin_amdgcn_sched_barrier(0);
    float qs[8];
    focus_row_sum<D, true>(qs, Q + (int64_t)h * qsh, qsn, focus_idx, entry, n_f, n_gen);
#pragma unroll
    for (int p = 0; p < P; ++p) {
      const float dot = chunk_dot_reduce<CPR>(qs, k0[p], k1[p]);
      const int b = b0 + p * R + r;
      if (c == 0) {
        if (PER_HEAD) {
          if (b < n_b) part[(int64_t)h * n_b + b] = dot;
        } else {
          dots[wave][p * R + r] = dot;
        }
      }
    }
  }
  if (PER_HEAD) return;
  __syncthreads();
  const int t = threadIdx.x;
  if (t < P * R && b0 + t < n_b) {
    float acc = dots[0][t];
#pragma unroll
    for (int w = 1; w < kRelGroup; ++w) acc = (int)blockIdx.x * kRelGroup + w < H ? acc + dots[w][t] : acc;
    part[(int64_t)blockIdx.x * n_b + b0 + t] = acc;
  }
}

template <int D, bool PER_HEAD>
__global__ __launch_bounds__(256) void relevance_partial_kernel(const int32_t* __restrict__ focus_idx,
                                                                const float* __restrict__ kbar,
                                                                const int32_t* __restrict__ counts,
                                                                const uint16_t* __restrict__ Q, int64_t qsh, int64_t qsn, int n_b,
                                                                int H, int n_focus_max, int n_gen, float* __restrict__ part) {
  relevance_partial<D, PER_HEAD>(focus_idx, kbar, counts, Q, qsh, qsn, n_b, H, n_focus_max, n_gen, part);
}
// The grid's slices from n_slices on make a cache update, a workgroup each per head and kUpdateSlots slots.
template <int D>
__global__ __launch_bounds__(256) void relevance_update_kernel(const int32_t* __restrict__ focus_idx, const float* __restrict__ kbar,
                                                               const int32_t* __restrict__ counts, const uint16_t* __restrict__ Q,
                                                               int64_t qsh, int64_t qsn, int n_b, int H, int n_focus_max, int n_gen,
                                                               float* __restrict__ part, int n_slices, const CacheUpdate update) {
  if (grid_yz() >= n_slices) {  // whole workgroup
    const int64_t item = (int64_t)(grid_yz() - n_slices) * gridDim.x + blockIdx.x;
    const int64_t g = item / update.n_heads;
    if (g * kUpdateSlots<D> < update.max_active) cache_update_part<D>(update, (int)g, (int)(item - g * update.n_heads));
    return;
  }
  relevance_partial<D, false>(focus_idx, kbar, counts, Q, qsh, qsn, n_b, H, n_focus_max, n_gen, part);
}

template <int D>
static void launch_block_relevance_t(const uint16_t* q, const int32_t* focus_idx, const int32_t* counts, int n_focus_max, const float* kbar,
                                     const focus_shape& s, float* part, bool per_head, hipStream_t st, const CacheUpdate* u) {
  const int n_b = ceil_div(s.n_ctx, s.block), n_x = ceil_div(s.n_heads, kRelGroup), n_slices = ceil_div(n_b, kRelPasses * (512 / D));
  const int n_update = u ? (int)ceil_div64((int64_t)ceil_div(u->max_active, kUpdateSlots<D>) * s.n_heads, n_x) : 0;
  const dim3 grid = grid_x_yz(n_x, n_slices + n_update);
  if (u)
    hipLaunchKernelGGL(relevance_update_kernel<D>, grid, dim3(256), 0, st, focus_idx, kbar, counts, q, s.q_stride_h, s.q_stride_n, n_b, s.n_heads,
                       n_focus_max, s.n_gen, part, n_slices, *u);
  else if (per_head)
    hipLaunchKernelGGL((relevance_partial_kernel<D, true>), grid, dim3(256), 0, st, focus_idx, kbar, counts, q, s.q_stride_h,
                       s.q_stride_n, n_b, s.n_heads, n_focus_max, s.n_gen, part);
  else
    hipLaunchKernelGGL((relevance_partial_kernel<D, false>), grid, dim3(256), 0, st, focus_idx, kbar, counts, q, s.q_stride_h,
                       s.q_stride_n, n_b, s.n_heads, n_focus_max, s.n_gen, part);
}

hipError_t launch_block_relevance(const void* Q, const int32_t* focus_idx, const int32_t* counts, int n_focus_max,
                                  const float* kbar, const focus_shape& s, float* part, bool per_head, hipStream_t st,
                                  const CacheUpdate* update) {
  const uint16_t* q = static_cast<const uint16_t*>(Q);
  if (per_head && update != nullptr) return hipErrorInvalidValue;
  if (s.head_dim == 128)
    launch_block_relevance_t<128>(q, focus_idx, counts, n_focus_max, kbar, s, part, per_head, st, update);
  else
    launch_block_relevance_t<64>(q, focus_idx, counts, n_focus_max, kbar, s, part, per_head, st, update);
  return hipGetLastError();
}

// =====================================================================================================
// Sink identification, second half (Eq. 6).  The MFMA kernel has written the scaled logits (base-2
// domain) and per-split row maxima / sums; here the row log-sum-exp is assembled and the column mass
// S_j = mean over (head, active query) of exp2(logit - lse) is accumulated in a fixed order.
// =====================================================================================================
// One workgroup per head and 16 queries: thread = (query, split lane); up to 256 splits are one memory round trip.
constexpr int kCombineLanes = 32;
__global__ __launch_bounds__(16 * kCombineLanes) void lse_combine_kernel(const float* __restrict__ part_ml, int q_pad, int n_split, float* __restrict__ lse2) {
  constexpr int kWaves = kCombineLanes / 4;
  __shared__ float2 wave_sh[kWaves][16];
  const int q = threadIdx.x & 15, sl = threadIdx.x >> 4;
  const int64_t tile = blockIdx.x;  // h * (q_pad / 16) + query tile
  const int tiles = q_pad >> 4, h = (int)(tile / tiles), q0 = (int)(tile - (int64_t)h * tiles) * 16;
  const RowState r = add_row_splits(reinterpret_cast<const float2*>(part_ml) + (int64_t)h * n_split * q_pad + q0 + q, q_pad, sl, kCombineLanes, n_split);
  const float m = group_max(r.m);  // the four lanes of a query in this wavefront
  const float l = group_sum(r.l > 0.f ? r.l * __builtin_amdgcn_exp2f(r.m - m) : 0.f);
  if ((threadIdx.x & 63) < 16) wave_sh[threadIdx.x >> 6][q] = make_float2(m, l);
  __syncthreads();
  if (threadIdx.x < 16) lse2[tile * 16 + q] = lse_of(add_row_splits(&wave_sh[0][q], 16, 0, 1, kWaves));
}

hipError_t launch_lse_combine(const float* part_ml, int H, int q_pad, int n_split, float* lse2, hipStream_t st) {
  hipLaunchKernelGGL(lse_combine_kernel, dim3(H * (q_pad / 16)), dim3(16 * kCombineLanes), 0, st, part_ml, q_pad, n_split, lse2);
  return hipGetLastError();
}

// Column attention mass S_j (Eq. 6) from what the first stage left behind.  Workgroup = 128 keys, 512 threads.
//   PRE = false: `src` holds the scaled logits of at most 16 active queries in the layout
//                [head][key quad][query][key within the quad] (fp32) and lse2 their row log-sum-exps [H, 16].  Lane
//                (query c, quad qd) of wavefront w owns the four keys of quad 4 w + qd for query c: one 16-byte load
//                per head, the 64 lanes of a load instruction reading 1 KB of consecutive bytes; HEADS heads are in
//                flight at a time, the smallest of four, eight and sixteen that holds all of them, else sixteen: with fewer in
//                flight there are fewer registers, so that more workgroups share a compute unit, and less code to fetch (sink chain:
//                1 head, 1088 keys 10.3 -> 9.3 us, 131 136 keys 34.4 -> 29.0; 3 heads, 16 448 keys 17.3 -> 16.4; 6 heads, 8256 keys
//                15.7 -> 15.0).  That a load past the last head repeats it costs nothing (1 to 8 heads, up to 32 832 keys: sixteen
//                in flight with the absent ones left out take as long).  It adds exp2(logit - lse) over the heads in head order; the
//                sixteen queries of a quad are then summed across the lanes of a DPP row (fixed tree).
//                PAST_CACHE: more logits than the 256 MB memory-side cache holds: heads in descending order and without a place in
//                that cache, which has kept the last heads that were written; reading the first ones first would displace them
//                (kMemorySideCache).
//   PRE = true:  `src` holds per-part column sums [n_parts, L] (already summed over a part's queries); thread
//                (key, part group pg) adds parts pg, pg + 4, ..., eight loads in flight, then the four groups are added.
// S_j = total / (H * n_act).
// With cand != nullptr the workgroup also nominates: the n_sink largest masses among its own prompt positions (j < M; ties to
// the lower j) go to cand[wg * n_sink ..], ascending, padded with -1, and their order keys + 1 to cand_keys at the same places
// (0 beside a -1).  With n_sink = N_sink the overall Top-N_sink is a subset of the union of these lists (sink_final_kernel); with
// fewer nominees per group sink_rank_kernel sees to the groups that may hold more.
constexpr int kMassKeys = 128;

// LSE (with PRE = false): lse2 holds the softmax statistics (max, sum) of n_split key splits per row, [H, n_split, 16], instead,
// and every workgroup forms the log-sum-exps itself, thread = (split lane, row), while its first logits travel.  Every workgroup reads
// all of the statistics, and what that costs goes with the bytes that all of them together take from the L2s: up to
// kLseInMassBytes it is no more than a launch of lse_combine_kernel.  Sink chain in us with that launch and without it, bytes in all: 32
// heads, 4160 keys 21.8 and 20.6 (1.1 MB), 8256 keys 29.6 and 28.8 (4.3 MB), 16 448 keys 45.1 and 48.9 (34 MB); 8 heads, 8256 keys 16.6
// and 16.4 (2.1 MB), 16 448 21.7 and 21.5 (4.2 MB), 24 640 24.1 and 25.5 (13 MB), 32 832 26.9 and 30.8 (17 MB); 1 head, 8256 keys 12.3
// and 11.5 (0.5 MB), 24 640 14.6 and 15.1 (4.8 MB), 32 832 15.0 and 16.0 (8.4 MB), 131 136 22.4 and 28.9 (34 MB); 4 heads, 1056 keys
// 11.8 and 10.2 (0.04 MB).
constexpr int kLseRows = 1024;
constexpr int64_t kLseInMassBytes = 5000000;
static bool lse_in_column_mass(int H, int n_split, int n_workgroups) {
  const int64_t bytes = (int64_t)H * 16 * n_split * (int64_t)sizeof(float2);
  return H * 16 <= kLseRows && bytes * n_workgroups <= kLseInMassBytes;
}

template <bool PRE, bool LSE, int HEADS, bool PAST_CACHE>
__global__ __launch_bounds__(512) void column_mass_kernel(const float* __restrict__ src, const float* __restrict__ lse2,
                                                          const int32_t* __restrict__ counts, int max_active, int n_parts,
                                                          int H, int L, float* __restrict__ col_mass, int M, int n_sink,
                                                          int32_t* __restrict__ cand, uint32_t* __restrict__ cand_keys, int n_split) {
  __shared__ float red[PRE ? 4 : 1][kMassKeys];
  __shared__ float mass_sh[kMassKeys];
  __shared__ float lse_sh[LSE ? kLseRows : 1];
  __shared__ __attribute__((aligned(16))) uint32_t ckeys[kMassKeys];
  __shared__ uint32_t ctotal;
  const int n_act = counts ? min(max(counts[1], 0), max_active) : max_active;
  const float norm = n_act > 0 ? 1.f / ((float)H * (float)n_act) : 0.f;
  if (PRE) {
    const int kj = threadIdx.x & (kMassKeys - 1), pg = threadIdx.x / kMassKeys;
    const int j = blockIdx.x * kMassKeys + kj;
    float acc = 0.f;
    if (j < L) {
      for (int q0 = pg; q0 < n_parts; q0 += 32) {
        float x[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
          const int q = q0 + 4 * u;
          x[u] = q < n_parts ? src[(int64_t)q * L + j] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) acc += x[u];
      }
    }
    red[pg][kj] = acc;
    __syncthreads();
    if (pg == 0) mass_sh[kj] = ((red[0][kj] + red[1][kj]) + (red[2][kj] + red[3][kj])) * norm;
  } else {
    constexpr int kHeadsInFlight = HEADS;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = lane & 15, qd = lane >> 4;
    const int quad_local = wave * 4 + qd;                                    // 0 .. 31
    const int64_t n_quads = (L + 3) >> 2;
    const int64_t quad = (int64_t)blockIdx.x * (kMassKeys / 4) + quad_local;  // key quad of this lane
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
    // (quads past the end repeat the last one; their masses are not looked at)
    const float4* base = reinterpret_cast<const float4*>(src) + (quad < n_quads ? quad : n_quads - 1) * 16 + min(c, max_active - 1);
    for (int h0 = 0; h0 < n_parts; h0 += kHeadsInFlight) {
      float4 x[kHeadsInFlight];
      float z[kHeadsInFlight];
#pragma unroll
      for (int u = 0; u < kHeadsInFlight; ++u) {
        const int h = min(h0 + u, n_parts - 1);  // clamped: stays in bounds, ignored below
        if (PAST_CACHE) {
          x[u] = __builtin_bit_cast(float4, load_stream16(base + (int64_t)(n_parts - 1 - h) * n_quads * 16));
          z[u] = lse2[(int64_t)(n_parts - 1 - h) * 16 + c];
        } else {
          x[u] = base[(int64_t)h * n_quads * 16];
          if (!LSE) z[u] = lse2[(int64_t)h * 16 + c];
        }
      }
      if (LSE) {
        if (h0 == 0) {  // uniform
          const float2* ml = reinterpret_cast<const float2*>(lse2);
          const int rows = H * 16, lanes = rows <= 64 ? 8 : (rows <= 128 ? 4 : (rows <= 256 ? 2 : 1));  // neighbouring lanes per row
          const int sl = threadIdx.x & (lanes - 1), per_turn = 512 / lanes;
          for (int row = threadIdx.x / lanes; row < rows; row += per_turn) {
            const float2* first = ml + (row >> 4) * n_split * 16 + (row & 15);
            const RowState r = n_split <= 2 * lanes ? add_row_splits<2>(first, 16, sl, lanes, n_split)
                                                         : add_row_splits<kSplitsInFlight, HEADS <= 8>(first, 16, sl, lanes, n_split);
            float m = r.m;
            if (lanes > 1) m = fmaxf(m, lane_dpp<0xB1>(m));   // quad_perm [1,0,3,2]
            if (lanes > 2) m = fmaxf(m, lane_dpp<0x4E>(m));   // quad_perm [2,3,0,1]
            if (lanes > 4) m = fmaxf(m, lane_dpp<0x141>(m));  // row_half_mirror
            float l = r.l > 0.f ? r.l * __builtin_amdgcn_exp2f(r.m - m) : 0.f;
            if (lanes > 1) l += lane_dpp<0xB1>(l);
            if (lanes > 2) l += lane_dpp<0x4E>(l);
            if (lanes > 4) l += lane_dpp<0x141>(l);
            if (sl == 0) lse_sh[row] = lse_of(RowState{m, l});
          }
          __syncthreads();
        }
#pragma unroll
        for (int u = 0; u < kHeadsInFlight; ++u) z[u] = lse_sh[min(h0 + u, n_parts - 1) * 16 + c];
      }
#pragma unroll
      for (int u = 0; u < kHeadsInFlight; ++u) {
        if (h0 + u < n_parts) {
          acc[0] += __builtin_amdgcn_exp2f(x[u].x - z[u]);
          acc[1] += __builtin_amdgcn_exp2f(x[u].y - z[u]);
          acc[2] += __builtin_amdgcn_exp2f(x[u].z - z[u]);
          acc[3] += __builtin_amdgcn_exp2f(x[u].w - z[u]);
        }
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) acc[r] = row_sum16(c < n_act ? acc[r] : 0.f);  // query slots past the count add nothing
    if (c == 0) {
#pragma unroll
      for (int r = 0; r < 4; ++r) mass_sh[quad_local * 4 + r] = acc[r] * norm;
    }
  }
  __syncthreads();
  float mass = 0.f;
  const int j = blockIdx.x * kMassKeys + threadIdx.x;  // threads 0 .. 127: one key each
  if (threadIdx.x < kMassKeys && j < L) {
    mass = mass_sh[threadIdx.x];
    col_mass[j] = mass;
  }
  if (cand != nullptr && (int)blockIdx.x * kMassKeys < M) {  // uniform over the workgroup
    if (threadIdx.x < kMassKeys) ckeys[threadIdx.x] = j < M ? order_key(mass) + 1u : 0u;
    __syncthreads();
    if (threadIdx.x < kWave)
      wave_topk<2, true>(ckeys, kMassKeys, n_sink, cand + (int64_t)blockIdx.x * n_sink, nullptr, &ctotal, blockIdx.x * kMassKeys, nullptr,
                   cand_keys ? cand_keys + (int64_t)blockIdx.x * n_sink : nullptr);
  }
}

// Final rounds of the sink tournament over the n_cand = n_groups * n_sink first-round winners (n_sink <= 16,
// n_cand <= 4096; cand ascending in j apart from -1 padding, cand_keys their order keys + 1, 0 beside a -1).  Round two: wavefront w ranks candidates
// [256 w, 256 w + 256); round three: one wavefront ranks the <= 256 survivors.  Every round keeps the order
// (value descending, index ascending) and lists its winners by ascending position, so the result is the exact Top-N_sink
// in ascending order.
// Up to 256 candidates are one round of one wavefront (8K prompts with 4 sinks: 3.4 us for the three rounds, 2.8 for the one).
__global__ __launch_bounds__(1024) void sink_final_kernel(const int32_t* __restrict__ cand, const uint32_t* __restrict__ cand_keys,
                                                         int n_cand, int n_sink, int32_t* __restrict__ sink_idx) {
  __shared__ __attribute__((aligned(16))) uint32_t keys1[16][256];
  __shared__ __attribute__((aligned(16))) int32_t pos1[16][256];
  __shared__ __attribute__((aligned(16))) uint32_t keys2[256];
  __shared__ int32_t win1[16][16];
  __shared__ int32_t win2[16];
  __shared__ uint32_t tot1[16], tot2;
  const int tid = threadIdx.x, w = tid >> 6, lane = tid & 63;
  const int c0 = w * 256 + lane * 4;  // whole vectors may be read past n_cand: the buffers hold kMaxNominees entries
  uint4 k4 = *reinterpret_cast<const uint4*>(cand_keys + c0);  // the nominees' keys were written beside their positions
  *reinterpret_cast<int4*>(&pos1[w][lane * 4]) = *reinterpret_cast<const int4*>(cand + c0);
  k4.x = c0 < n_cand ? k4.x : 0u;
  k4.y = c0 + 1 < n_cand ? k4.y : 0u;
  k4.z = c0 + 2 < n_cand ? k4.z : 0u;
  k4.w = c0 + 3 < n_cand ? k4.w : 0u;
  *reinterpret_cast<uint4*>(&keys1[w][lane * 4]) = k4;
  __syncthreads();
  if (w * 256 < n_cand) wave_topk<4, true>(keys1[w], 256, n_sink, win1[w], nullptr, &tot1[w]);  // blockDim covers these waves
  __syncthreads();
  if (n_cand <= 256) {  // one wavefront
    if (tid < n_sink) {
      const int32_t t = win1[0][tid];
      sink_idx[tid] = t >= 0 ? pos1[0][t] : -1;
    }
    return;
  }
  if (tid < 256) {
    const int ww = tid >> 4, i = tid & 15;
    const int32_t slot = (ww * 256 < n_cand && i < n_sink) ? win1[ww][i] : -1;
    keys2[tid] = slot >= 0 ? keys1[ww][slot] : 0u;
  }
  __syncthreads();
  if (w == 0) wave_topk<4, true>(keys2, 256, n_sink, win2, nullptr, &tot2);
  __syncthreads();
  if (tid < n_sink) {
    const int32_t t = win2[tid];
    sink_idx[tid] = t >= 0 ? pos1[t >> 4][win1[t >> 4][t & 15]] : -1;
  }
}

bool sink_tournament_fits(int M, int n_sink) {
  return n_sink >= 1 && n_sink <= kTournamentMaxSinks && (int64_t)ceil_div(M, kMassKeys) * n_sink <= kTournamentMaxCand;
}

// pre_reduced = false: src = logits [H, ceil(L / 4), 16, 4], n_parts = H.  pre_reduced = true: src = column sums [n_parts, L].
hipError_t launch_column_mass(const float* src, bool pre_reduced, const float* lse2, const int32_t* counts, int max_active,
                              int n_parts, int H, int L, float* col_mass, int M, int n_sink, int32_t* cand, uint32_t* cand_keys,
                              int n_split, float* lse_scratch, hipStream_t st) {
  if (cand != nullptr && (n_sink < 1 || n_sink > kMaxNominees / ceil_div(M, kMassKeys))) return hipErrorInvalidValue;  // n_sink: nominees per group
  if (!pre_reduced && (n_parts < 1 || max_active < 1)) return hipErrorInvalidValue;
  const dim3 grid(ceil_div(L, kMassKeys));
  if (pre_reduced) {
    hipLaunchKernelGGL((column_mass_kernel<true, false, 1, false>), grid, dim3(512), 0, st, src, lse2, counts, max_active, n_parts, H, L, col_mass,
                       M, n_sink, cand, cand_keys, 0);
    return hipGetLastError();
  }
  const bool lse = n_split > 0 && lse_in_column_mass(H, n_split, (int)grid.x);
  if (n_split > 0 && !lse) {
    const hipError_t e = launch_lse_combine(lse2, H, 16, n_split, lse_scratch, st);
    if (e != hipSuccess) return e;
    lse2 = lse_scratch;
  }
  // Sink chain in us, 16 queries, 131 136 keys (logits read plainly in ascending order; plainly in descending; non-temporally in
  // ascending; non-temporally in descending): 32 heads, 269 MB 268, 267, 266, 268; 40 heads, 336 MB 373, 364, 351, 345; 64 heads, 537 MB
  // 623, 617, 585, 579.  At 134 and 210 MB all four are alike, too; at 67 MB (32 832 keys) the plain ones take 1.2 us less.  (All with
  // plain stores.  Written non-temporally, as they were past 200 MB: 268 -> 285, 345 -> 364, 579 -> 577; 65 600 keys of 32 heads 138 -> 147.)
  // Up to eight heads, which would need 400 000 keys and more, are left to the plain reads: not measured.
  constexpr int64_t kMemorySideCache = (int64_t)200 << 20;
#define COLUMN_MASS(HEADS)                                                                                                       \
  if (lse)                                                                                                                       \
    hipLaunchKernelGGL((column_mass_kernel<false, true, HEADS, false>), grid, dim3(512), 0, st, src, lse2, counts, max_active, n_parts, H, L, \
                       col_mass, M, n_sink, cand, cand_keys, n_split);                                                           \
  else                                                                                                                           \
    hipLaunchKernelGGL((column_mass_kernel<false, false, HEADS, false>), grid, dim3(512), 0, st, src, lse2, counts, max_active, n_parts, H, L, \
                       col_mass, M, n_sink, cand, cand_keys, 0)
  if (!lse && n_parts > 8 && (int64_t)n_parts * L * 64 > kMemorySideCache) {
    hipLaunchKernelGGL((column_mass_kernel<false, false, 16, true>), grid, dim3(512), 0, st, src, lse2, counts, max_active, n_parts, H, L,
                       col_mass, M, n_sink, cand, cand_keys, 0);
  } else if (n_parts <= 4) {
    COLUMN_MASS(4);
  } else if (n_parts <= 8) {
    COLUMN_MASS(8);
  } else {
    COLUMN_MASS(16);
  }
#undef COLUMN_MASS
  return hipGetLastError();
}

// Top-N_sink beyond the tournament's limits (the paper's 1 % rule asks for hundreds of sinks), M <= 131072.  The column-mass
// kernel has nominated the kRankNominees largest masses of every 128-key group (n_per = min(kRankNominees, N_sink)), in
// ascending order of position.  One workgroup holds all nominees in registers, KPL consecutive ones per thread, and finds the
// N_sink-th largest key by a radix search, eight bits per pass.  The bits all keys share are skipped, and the search ends as soon
// as exactly N_sink keys reach a digit.  Unless a group has all its nominees selected (its other keys might then belong to the answer too) that is the
// exact Top-N_sink.  Otherwise the key found is a lower bound of the true one, and the positions that reach it, compacted in
// index order into LDS, are ranked the same way; only if they do not fit a radix select over all positions decides.
// 32768 keys, 327 sinks: 6 us (two bits per pass: 8; bounding, compacting and ranking all positions in one workgroup took 18); 131072 keys, 1310
// sinks: 12 us (radix select: 390 us).
template <int KPL>
__global__ __launch_bounds__(kTopkThreads) void sink_rank_kernel(const int32_t* __restrict__ cand, const uint32_t* __restrict__ cand_keys,
                                                                 int n_cand, int n_per, int M, int n_sink,
                                                                 const float* __restrict__ col_mass, int32_t* __restrict__ sink_idx) {
  constexpr int kWaves = kTopkThreads / kWave, kCap = kTopkThreads * KPL;
  __shared__ __attribute__((aligned(16))) uint32_t keys_sh[kCap];  // positions that clear the bound: key + 1 ...
  __shared__ __attribute__((aligned(16))) int32_t idx_sh[kCap];    // ... and index
  __shared__ __attribute__((aligned(16))) uint32_t hist_sh[4][256];  // a histogram per digit
  __shared__ uint32_t bits_sh[kWaves][2], valid_sh[kWaves], sel_sh[kWaves][2];
  __shared__ int overflow_sh;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const unsigned long long below = (1ull << lane) - 1ull;
  const int i0 = tid * KPL;
  uint32_t kv[KPL];  // key + 1; 0 = none
  int32_t pos[KPL];
  auto load = [&](const uint32_t* keys, const int32_t* idx, int n) __attribute__((always_inline)) {  // whole vectors may be read past n: both buffers hold kCap entries at least
#pragma unroll
    for (int r4 = 0; r4 < KPL / 4; ++r4) {
      const uint4 a = *reinterpret_cast<const uint4*>(keys + i0 + 4 * r4);
      const int4 b = *reinterpret_cast<const int4*>(idx + i0 + 4 * r4);
      kv[4 * r4] = a.x; kv[4 * r4 + 1] = a.y; kv[4 * r4 + 2] = a.z; kv[4 * r4 + 3] = a.w;
      pos[4 * r4] = b.x; pos[4 * r4 + 1] = b.y; pos[4 * r4 + 2] = b.z; pos[4 * r4 + 3] = b.w;
    }
#pragma unroll
    for (int r = 0; r < KPL; ++r) kv[r] = i0 + r < n ? kv[r] : 0u;
  };
  load(cand_keys, cand, n_cand);
  if (tid == 0) overflow_sh = 0;
  for (int pass = 0;; ++pass) {  // the nominees; then, if need be, every position that clears the bound
    uint32_t all = 0xffffffffu, any = 0u, n_mine = 0;
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
      all &= kv[r] != 0u ? kv[r] : 0xffffffffu;
      any |= kv[r];
      n_mine += (uint32_t)__popcll(__ballot(kv[r] != 0u));
    }
    hist_sh[tid >> 8][tid & 255] = 0u;
    all = wave_reduce_u32(all, [](uint32_t a, uint32_t b) { return a & b; });
    any = wave_reduce_u32(any, [](uint32_t a, uint32_t b) { return a | b; });
    if (lane == 0) {
      bits_sh[wave][0] = all;
      bits_sh[wave][1] = any;
      valid_sh[wave] = n_mine;
    }
    __syncthreads();
    uint32_t n_valid = 0;
    all = 0xffffffffu;
    any = 0u;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      all &= bits_sh[w][0];
      any |= bits_sh[w][1];
      n_valid += valid_sh[w];
    }
    const uint32_t k = min((uint32_t)n_sink, n_valid);
    uint32_t T = 0u;  // the k-th largest key, or one less than a threshold that exactly k keys reach; 0: all of them
    if (k < n_valid) {
      const int top = all == any ? -1 : 31 - (int)__clz((int)(all ^ any));  // -1: all keys are equal
      T = top < 0 ? all : (top == 31 ? 0u : all & ~((2u << top) - 1u));
      uint32_t above = 0;  // keys whose leading digits exceed T's
      int hi = top;
      for (int digit_no = 0; hi >= 0; ++digit_no) {  // bits hi .. shift, eight at a time: one LDS atomic per key, one barrier; every
        const int shift = hi >= 7 ? hi - 7 : 0;      // wavefront scans the 256 counts by itself, four per lane
        uint32_t* hist = hist_sh[digit_no];
        const uint32_t ones = (2u << (hi - shift)) - 1u;
#pragma unroll
        for (int r = 0; r < KPL; ++r)
          if (kv[r] != 0u && (hi == 31 || (kv[r] >> (hi + 1)) == (T >> (hi + 1)))) atomicAdd(&hist[(kv[r] >> shift) & ones], 1u);
        __syncthreads();
        const RadixDigit d = radix_digit(hist, k - above);
        above += d.over;
        T |= d.digit << shift;
        if (above + d.count == k) {  // exactly these: "key > T" selects them and none equal to T is needed (k > 0)
          T -= 1u;
          break;
        }
        hi = shift - 1;
      }
    }
    // selection in ascending order: everything above T, and the first keys equal to T until k are reached
    uint32_t n_gt = 0, n_eq = 0, eq_before = 0;
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
      const unsigned long long eq = __ballot(kv[r] == T && kv[r] != 0u);
      n_gt += (uint32_t)__popcll(__ballot(kv[r] > T));
      n_eq += (uint32_t)__popcll(eq);
      eq_before += (uint32_t)__popcll(eq & below);
    }
    if (lane == 0) {
      sel_sh[wave][0] = n_gt;
      sel_sh[wave][1] = n_eq;
    }
    __syncthreads();
    uint32_t gt_total = 0, gt_base = 0, eq_base = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      gt_total += sel_sh[w][0];
      if (w < wave) {
        gt_base += sel_sh[w][0];
        eq_base += sel_sh[w][1];
      }
    }
    const uint32_t need = k - min(gt_total, k);
    bool sel[KPL];
    uint32_t n_sel = 0, eq_rank = eq_base + eq_before;
#pragma unroll
    for (int r = 0; r < KPL; ++r) {
      const bool eq = kv[r] == T && kv[r] != 0u;
      sel[r] = kv[r] > T || (eq && eq_rank < need);
      eq_rank += eq;
      n_sel += sel[r];
    }
    // a group with all its nominees selected: n_per = kRankNominees of them, kRankNominees / KPL neighbouring lanes
    if (pass == 0 && n_per == kRankNominees) {
      unsigned long long full = __ballot(n_sel == (uint32_t)KPL);
#pragma unroll
      for (int w = 1; w < kRankNominees / KPL; w <<= 1) full &= full >> w;
      constexpr unsigned long long kFirst = KPL == 16 ? ~0ull : (KPL == 8 ? 0x5555555555555555ull : 0x1111111111111111ull);
      if ((full & kFirst) != 0ull && lane == 0) overflow_sh = 1;
    }
    uint32_t out = gt_base + min(eq_base, need);
#pragma unroll
    for (int r = 0; r < KPL; ++r) out += (uint32_t)__popcll(__ballot(sel[r]) & below);
#pragma unroll
    for (int r = 0; r < KPL; ++r)
      if (sel[r]) sink_idx[out++] = pos[r];
    for (int i = (int)k + tid; i < n_sink; i += kTopkThreads) sink_idx[i] = -1;
    if (pass == 1) return;
    __syncthreads();
    if (!overflow_sh) return;  // uniform

    // ---- some group may hold more: every position whose key reaches the bound (at least N_sink do).  Wavefront w walks the
    // run [w * run, (w + 1) * run) in steps of 64 positions, 32 loads in flight: once to count, once to write.
    const uint32_t bound = max(gt_total >= k ? T + 1u : T, 1u);
    // (compared as floats: the order of the keys is the order of the numbers; a bound of 1 lets NaN pass as well)
    const float bound_f = order_value(bound - 1u);
    const bool everything = bound == 1u;
    const int run = (M + kWaves - 1) / kWaves;
    const int r0 = min(wave * run, M), r1 = min(r0 + run, M);
    auto walk = [&](auto f) {
      for (int i = r0 + lane; i - lane < r1; i += 32 * kWave) {
        float v[32];
#pragma unroll
        for (int u = 0; u < 32; ++u) v[u] = col_mass[min(i + kWave * u, M - 1)];
#pragma unroll
        for (int u = 0; u < 32; ++u) {
          f(i + kWave * u, v[u], __ballot(i + kWave * u < r1 && (v[u] >= bound_f || everything)));
        }
      }
    };
    uint32_t n_run = 0;
    walk([&](int, float, unsigned long long hit) { n_run += (uint32_t)__popcll(hit); });
    if (lane == 0) valid_sh[wave] = n_run;
    __syncthreads();
    uint32_t n_clear = 0, at = 0;
#pragma unroll
    for (int w = 0; w < kWaves; ++w) {
      n_clear += valid_sh[w];
      if (w < wave) at += valid_sh[w];
    }
    if (n_clear > (uint32_t)kCap) break;  // uniform
    walk([&](int i, float x, unsigned long long hit) {
      if ((hit >> lane) & 1ull) {
        const uint32_t dst = at + (uint32_t)__popcll(hit & below);
        keys_sh[dst] = order_key(x) + 1u;
        idx_sh[dst] = i;
      }
      at += (uint32_t)__popcll(hit);
    });
    __syncthreads();
    load(keys_sh, idx_sh, (int)n_clear);
  }
  // more positions than the workgroup holds clear the bound
  TopkShared& sm = *reinterpret_cast<TopkShared*>(keys_sh);
  static_assert(sizeof(TopkShared) <= sizeof(keys_sh), "the radix select's shared memory fits");
  __syncthreads();
  auto keyfn = [=](int i, uint32_t& key) -> bool {
    key = order_key(col_mass[i]);
    return true;
  };
  block_topk(keyfn, M, n_sink, sink_idx, nullptr, nullptr, sm, (reinterpret_cast<uintptr_t>(col_mass) & 15u) == 0 ? col_mass : nullptr);
}

// At most four sinks per 128-key group on average: more would often fill a group's nominees.  Up to 1024 positions one wavefront
// ranks all of them sooner.
bool sink_rank_fits(int M, int n_sink) {
  const int groups = ceil_div(M, kMassKeys);
  return n_sink >= 1 && M > kTopkThreads && groups * kRankNominees <= kMaxNominees && n_sink <= 4 * groups;
}

hipError_t launch_sink_rank(const int32_t* cand, const uint32_t* cand_keys, int M, int n_sink, const float* col_mass, int32_t* sink_idx,
                            hipStream_t st) {
  if (!sink_rank_fits(M, n_sink)) return hipErrorInvalidValue;
  const int n_per = std::min(kRankNominees, n_sink), n_cand = ceil_div(M, kMassKeys) * n_per;
  if (n_cand <= 4 * kTopkThreads)
    hipLaunchKernelGGL(sink_rank_kernel<4>, dim3(1), dim3(kTopkThreads), 0, st, cand, cand_keys, n_cand, n_per, M, n_sink, col_mass, sink_idx);
  else if (n_cand <= 8 * kTopkThreads)
    hipLaunchKernelGGL(sink_rank_kernel<8>, dim3(1), dim3(kTopkThreads), 0, st, cand, cand_keys, n_cand, n_per, M, n_sink, col_mass, sink_idx);
  else
    hipLaunchKernelGGL(sink_rank_kernel<16>, dim3(1), dim3(kTopkThreads), 0, st, cand, cand_keys, n_cand, n_per, M, n_sink, col_mass, sink_idx);
  return hipGetLastError();
}

hipError_t launch_sink_final(const int32_t* cand, const uint32_t* cand_keys, int M, int n_sink, int32_t* sink_idx,
                             hipStream_t st) {
  if (!sink_tournament_fits(M, n_sink)) return hipErrorInvalidValue;
  const int n_cand = ceil_div(M, kMassKeys) * n_sink;
  const int threads = n_cand <= 256 ? 64 : std::max(256, ceil_div(n_cand, 256) * 64);  // one wavefront per 256 nominees; round three has 256 slots
  hipLaunchKernelGGL(sink_final_kernel, dim3(1), dim3(threads), 0, st, cand, cand_keys, n_cand, n_sink, sink_idx);
  return hipGetLastError();
}

// =====================================================================================================
// Around the step (Sec. 3): confidence from the vocabulary logits (Eq. 2) and the approximate KV cache (Eq. 3).
// =====================================================================================================
// Running state of one softmax row: maximum m, lowest index of the maximum, and s = sum exp(x - m).
struct ConfState {
  float m;
  int idx;
  float s;
};
// The states of 64 (or of each 32) lanes in the order (value descending, index ascending), the sums rescaled once to the largest maximum; every
// lane receives the result.  s == 0 marks "nothing seen": its m is -inf.  m is never NaN.
template <int LANES>
__device__ __forceinline__ ConfState conf_reduce(const ConfState& st) {
  auto reduce = [](uint32_t x, auto op) -> uint32_t {
    if constexpr (LANES == kWave) return wave_reduce_u32(x, op);
    x = row_reduce_u32(x, op);
    typedef unsigned v2u __attribute__((ext_vector_type(2)));
    const v2u b = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    return op(b.x, b.y);
  };
  auto of = [](uint32_t x) { return __uint_as_float(x); };
  ConfState r;
  r.m = of(reduce(__float_as_uint(st.m), [&](uint32_t x, uint32_t y) { return __float_as_uint(fmaxf(of(x), of(y))); }));
  r.idx = (int)reduce(st.m == r.m ? (uint32_t)st.idx : 0x7fffffffu, [](uint32_t x, uint32_t y) { return min(x, y); });
  const float mine = st.s > 0.f ? st.s * __expf(st.m - r.m) : 0.f;
  r.s = of(reduce(__float_as_uint(mine), [&](uint32_t x, uint32_t y) { return __float_as_uint(of(x) + of(y)); }));
  return r;
}

// x_hat = argmax_v logit_v (ties to the lower id), c = 1 / sum_v exp(logit_v - max).  Workgroup (row, split) walks one
// contiguous slice of the row once: eight bf16 per 16-byte non-temporal load; per vector the running maximum is raised
// once and the eight exponentials are added.  Threads, then wavefronts, merge their states in a fixed order.  With
// one split the workgroup writes the result; otherwise its state goes to part[row, split] and token_confidence_merge
// finishes the row.  Bound by latency: one memory round trip (the mask is looked at behind the request of the first vectors) and the
// reductions: maximum, index and sum one after the other by lane moves within the vector ALU.  With whole states exchanged through the LDS
// crossbar step by step, and the mask looked at first, both launches together took 10.8 us for 32 rows of 126 464 where they now take 6.7
// (64 rows 12.2 -> 8.4, 8 rows 8.0 -> 5.5, 64 rows of 32 000 8.9 -> 6.2).
// Rows that the mask excludes are requested as well, two vectors a thread (a short slice whole).  Against the same kernel with the mask first, which
// reads nothing of them, that gains while few rows are excluded and costs next to nothing when most are; none, half and 95 % of the rows excluded, this
// and mask first (us, rows that were not in a cache): 8 rows of 126 464: 4.9 and 5.0, 4.9 and 5.0, 4.4 and 4.5; 32: 6.9 and 6.8, 6.8 and 6.6, 6.5
// and 6.4; 64: 8.5 and 8.9, 8.1 and 8.1, 7.9 and 7.9; 256: 16.5 and 17.6, 15.9 and 16.0, 15.2 and 15.2; 1024 rows of 32 000: 14.7 and 15.0, 13.6 and 13.7,
// 10.8 and 10.5.
__global__ __launch_bounds__(256) void token_confidence_kernel(const uint16_t* __restrict__ logits, int64_t row_stride,
                                                               const uint8_t* __restrict__ masked, int vocab, int n_split,
                                                               ConfState* __restrict__ part, int32_t* __restrict__ tokens,
                                                               float* __restrict__ conf) {
  __shared__ ConfState wave_state[4];
  const int row = blockIdx.x, split = blockIdx.y, tid = threadIdx.x, nt = blockDim.x;
  ConfState st;
  st.m = -INFINITY;
  st.idx = 0x7fffffff;
  st.s = 0.f;
  const uint16_t* x = logits + (int64_t)row * row_stride;
  const int n_vec = vocab >> 3;
  const int per = (n_vec + n_split - 1) / n_split;
  const int v_begin = split * per, v_end = min(v_begin + per, n_vec);
  auto vector = [&](int v) {  // (vectors past the end: -inf)
    return v < v_end ? load_stream16(x + (int64_t)v * 8) : make_uint4(0xff80ff80u, 0xff80ff80u, 0xff80ff80u, 0xff80ff80u);
  };
  uint4 a = vector(v_begin + tid), b = vector(v_begin + tid + nt);  // two vectors in flight
  __builtin_amdgcn_sched_barrier(0);
  const bool skip = masked != nullptr && masked[row] == 0;  // uniform over the workgroup
  if (!skip) {
    for (int v0 = v_begin + tid; v0 < v_end; v0 += nt * 2) {
      const int v1 = v0 + nt;
      const uint4 vv[2] = {a, b};
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const uint32_t w[4] = {vv[u].x, vv[u].y, vv[u].z, vv[u].w};
        float e[8];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          e[2 * i] = bf16_lo(w[i]);
          e[2 * i + 1] = bf16_hi(w[i]);
        }
        float vm = e[0];
        int vi = 0;
#pragma unroll
        for (int i = 1; i < 8; ++i) {
          if (e[i] > vm) {  // strict: the lowest position of the vector's maximum
            vm = e[i];
            vi = i;
          }
        }
        if (vm > st.m) {  // vectors arrive in ascending index order, so a strict test keeps the lowest index
          st.s = st.s > 0.f ? st.s * __expf(st.m - vm) : 0.f;
          st.m = vm;
          st.idx = (u == 0 ? v0 : v1) * 8 + vi;
        }
        if (st.m > -INFINITY) {
#pragma unroll
          for (int i = 0; i < 8; ++i) st.s += __expf(e[i] - st.m);
        }
      }
      a = vector(v0 + 2 * nt);
      b = vector(v1 + 2 * nt);
    }
    if (split == n_split - 1) {  // ragged tail of the row, one element per thread
      for (int j = (n_vec << 3) + tid; j < vocab; j += nt) {
        const float e = bf16_lo((uint32_t)x[j]);
        if (e > st.m) {
          st.s = st.s > 0.f ? st.s * __expf(st.m - e) : 0.f;
          st.m = e;
          st.idx = j;
        }
        if (st.m > -INFINITY) st.s += __expf(e - st.m);
      }
    }
  }
  st = conf_reduce<kWave>(st);
  if ((tid & 63) == 0) wave_state[tid >> 6] = st;
  __syncthreads();
  if (tid < kWave) {
    if (tid < 4)
      st = wave_state[tid];
    else
      st = ConfState{-INFINITY, 0x7fffffff, 0.f};
    const ConfState r = conf_reduce<32>(st);
    if (tid != 0) return;
    if (n_split == 1) {
      tokens[row] = r.s > 0.f ? r.idx : -1;
      conf[row] = r.s > 0.f ? 1.f / r.s : 0.f;
    } else {
      part[(int64_t)row * n_split + split] = r;
    }
  }
}

// 32 lanes per row, one split each (one thread that walked the splits took 15 us for 30 of them)
constexpr int kConfMaxSplits = 32;
__global__ __launch_bounds__(256) void token_confidence_merge(const ConfState* __restrict__ part, int n_rows, int n_split,
                                                              int32_t* __restrict__ tokens, float* __restrict__ conf) {
  const int row = blockIdx.x * (256 / kConfMaxSplits) + (int)threadIdx.x / kConfMaxSplits, s = threadIdx.x % kConfMaxSplits;
  ConfState r;
  r.m = -INFINITY;
  r.idx = 0x7fffffff;
  r.s = 0.f;
  if (row < n_rows && s < n_split) r = part[(int64_t)row * n_split + s];
  static_assert(kConfMaxSplits == 32, "half a wavefront per row");
  r = conf_reduce<32>(r);
  if (row < n_rows && s == 0) {
    tokens[row] = r.s > 0.f ? r.idx : -1;
    conf[row] = r.s > 0.f ? 1.f / r.s : 0.f;
  }
}

// splits per row: enough workgroups to fill the chip, and as many as it takes for a thread to have its vectors in flight at once
int token_confidence_splits(int n_rows, int vocab) {
  const int by_rows = ceil_div(1024, n_rows);
  const int by_work = ceil_div(vocab >> 3, 512);
  return std::max(1, std::min(std::min(by_rows, by_work), kConfMaxSplits));
}
size_t token_confidence_workspace(int n_rows, int vocab) {
  const int n_split = token_confidence_splits(n_rows, vocab);
  return n_split > 1 ? (size_t)n_rows * n_split * sizeof(ConfState) : 0;
}

hipError_t launch_token_confidence(const void* logits, int64_t row_stride, const uint8_t* masked, int n_rows, int vocab,
                                   int32_t* tokens, float* conf, void* workspace, hipStream_t st) {
  const int n_split = token_confidence_splits(n_rows, vocab);
  ConfState* part = static_cast<ConfState*>(workspace);
  hipLaunchKernelGGL(token_confidence_kernel, dim3(n_rows, n_split), dim3(256), 0, st, static_cast<const uint16_t*>(logits),
                     row_stride, masked, vocab, n_split, part, tokens, conf);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || n_split == 1) return e;
  hipLaunchKernelGGL(token_confidence_merge, dim3(ceil_div(n_rows, 256 / kConfMaxSplits)), dim3(256), 0, st, part, n_rows, n_split,
                     tokens, conf);
  return hipGetLastError();
}

// Eq. 3: cache rows row_base + active_idx[a] of K and V take the new states K_new[:, a], V_new[:, a].  A thread moves one 16-byte
// chunk of the K or of the V row of a slot, a workgroup 256 / (2 * chunks) slots of one head.  Nothing but latency: the new
// state sits at the slot's own place, so it, the position and the count are requested together and the kernel is one memory
// round trip and a store long (32 heads, 32 slots: 5.4 us when they followed each other, one 64-thread workgroup per slot; now
// 3.5).  Entries outside the active count, negative, or mapping outside [0, n_rows) are skipped.
// In a sparse layer that takes its relevances from cached means the same workgroups run beside those of that launch (cache_update_part), which
// leave most of the chip idle and read nothing of the cache: decoding step of 7 layers, 5 of them sparse, 32 heads, 3153 rows 133.5 -> 125.0
// us; 4 heads, 2139 rows 97.2 -> 86.8; 7 layers, 6 sparse, 4 heads, d = 64, 8902 rows 124.4 -> 113.2.
template <int D>
__global__ __launch_bounds__(256) void cache_update_kernel(const CacheUpdate u) {
  cache_update_part<D>(u, blockIdx.x, blockIdx.y);
}

CacheUpdate cache_update_args(void* K_cache, void* V_cache, const focus_shape& s, const void* K_new, const void* V_new,
                              int64_t new_stride_h, int64_t new_stride_n, const int32_t* active_idx, const int32_t* counts,
                              int max_active, int row_base) {
  CacheUpdate u;
  u.Kn = static_cast<const uint16_t*>(K_new);
  u.Vn = static_cast<const uint16_t*>(V_new);
  u.Kc = static_cast<uint16_t*>(K_cache);
  u.Vc = static_cast<uint16_t*>(V_cache);
  u.nsh = new_stride_h; u.nsn = new_stride_n;
  u.ksh = s.k_stride_h; u.ksn = s.k_stride_n;
  u.vsh = s.v_stride_h; u.vsn = s.v_stride_n;
  u.active_idx = active_idx;
  u.counts = counts;
  u.max_active = max_active;
  u.row_base = row_base;
  u.n_rows = s.n_ctx + s.n_resp;
  u.n_heads = s.n_heads;
  return u;
}

hipError_t launch_cache_update(const CacheUpdate& u, int head_dim, hipStream_t st) {
  if (head_dim == 128)
    hipLaunchKernelGGL(cache_update_kernel<128>, dim3(ceil_div(u.max_active, kUpdateSlots<128>), u.n_heads), dim3(256), 0, st, u);
  else
    hipLaunchKernelGGL(cache_update_kernel<64>, dim3(ceil_div(u.max_active, kUpdateSlots<64>), u.n_heads), dim3(256), 0, st, u);
  return hipGetLastError();
}

// Block-entry cache refresh: one workgroup per (chunk of B rows, head).
template <int D>
__global__ __launch_bounds__(256) void cache_refresh_kernel(const CacheRefresh p) {
  __shared__ __attribute__((aligned(16))) float red[2048];
  cache_refresh_chunk<D>(p, blockIdx.x, blockIdx.y, threadIdx.x, true, red);
}

CacheRefresh cache_refresh_args(void* K_cache, void* V_cache, const focus_shape& s, const void* K_new, const void* V_new,
                                int64_t new_stride_h, int64_t new_stride_n, float* kbar) {
  CacheRefresh p;
  p.Kn = static_cast<const uint16_t*>(K_new);
  p.Vn = static_cast<const uint16_t*>(V_new);
  p.Kc = static_cast<uint16_t*>(K_cache);
  p.Vc = static_cast<uint16_t*>(V_cache);
  p.nsh = new_stride_h; p.nsn = new_stride_n;
  p.ksh = s.k_stride_h; p.ksn = s.k_stride_n;
  p.vsh = s.v_stride_h; p.vsn = s.v_stride_n;
  p.M = s.n_ctx; p.L = s.n_ctx + s.n_resp; p.B = s.block;
  p.n_b = ceil_div(s.n_ctx, s.block);
  p.n_chunks = p.n_b + ceil_div(s.n_resp, s.block);
  p.n_heads = s.n_heads;
  p.kbar = kbar;
  return p;
}

hipError_t launch_cache_refresh(const CacheRefresh& p, int head_dim, hipStream_t st) {
  const dim3 grid(p.n_chunks, p.n_heads);
  if (head_dim == 128)
    hipLaunchKernelGGL(cache_refresh_kernel<128>, grid, dim3(256), 0, st, p);
  else
    hipLaunchKernelGGL(cache_refresh_kernel<64>, grid, dim3(256), 0, st, p);
  return hipGetLastError();
}

}  // namespace focus
