// Host-side launch functions of the kernels (one per kernel family) and the launch-shape helpers the
// API layer and the workspace-size query share.  Internal to the library.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "../../include/focus.h"

namespace focus {

constexpr int kSubTile = 32;        // keys one wavefront stages and multiplies at a time
constexpr int kWavesPerGroup = 4;   // wavefronts per workgroup of the MFMA kernels
constexpr int kQTile = 16;          // queries per MFMA tile
constexpr int kMaxQTilesPerGroup = 4;

static inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
// A grid of n_x workgroups in x by n workgroups in y, continued in z: n may exceed the 65535 of one axis.
constexpr int kGridSlice = 32768;
static inline dim3 grid_x_yz(int n_x, int n) { return dim3(n_x, n < kGridSlice ? n : kGridSlice, ceil_div(n, kGridSlice)); }
__device__ __forceinline__ int grid_yz() { return (int)(blockIdx.z * kGridSlice + blockIdx.y); }
static inline int64_t ceil_div64(int64_t a, int64_t b) { return (a + b - 1) / b; }
// A list of n workgroups, in slices along y: one axis of a launch has fewer than 2^32 threads, 2^23 workgroups of 512.  Slices are a
// multiple of eight long, so that list_index() mod 8 = blockIdx.x mod 8 stays the round-robin place among the XCDs.  The last slice is
// whole: indices of n and more occur.
constexpr int kListSlice = 1 << 22;
constexpr int64_t kMaxList = (int64_t(1) << 31) - kListSlice;  // list_index() is an int
static inline dim3 grid_list(int64_t n) {
  return dim3((uint32_t)(n < kListSlice ? n : kListSlice), (uint32_t)ceil_div64(n, kListSlice));
}
__device__ __forceinline__ int list_index() { return (int)(blockIdx.y * kListSlice + blockIdx.x); }

// How the key axis of an MFMA kernel is cut: n_sub sub-tiles per head, n_split workgroups per (head, query group).  The
// splits take turns: split s works on the rounds of four sub-tiles (one per wavefront) s, s + n_split, s + 2 n_split, ...
// All of them are equally long up to one round, and together they sweep one window of K and V.  (Contiguous ranges per split
// start at multiples of a length that is often close to a power of two, which puts all workgroups on the same memory
// channels: the 32K dense layer with 30 queries takes 96 us that way, 89 us this way.)
struct SplitPlan {
  int n_sub, n_split;
  bool pipelined = false;  // attention only: wavefronts walk several sub-tiles, use the key loop
  int q_tiles, q_tiles_per_group, q_groups, q_pad;  // q_pad = 16 * q_tiles
};

// workgroups of a launch whose list has the query groups of eight (head, key split) pairs next to each other
static inline int64_t query_group_list(const SplitPlan& p, int n_heads) {
  return ceil_div64((int64_t)p.n_split * n_heads, 8) * 8 * p.q_groups;
}

// lean: the plan with fewer key splits that a workspace too small for the other's partial results is given (focus_workspace_bytes
// speaks of the other; it must never refuse what it took before the splits of some shapes grew)
SplitPlan plan_attention(const focus_shape& s, int max_active, int n_keep, int n_sink, bool lean = false);
SplitPlan plan_attention_dense(const focus_shape& s, int max_active);  // all M + N rows, no block structure
SplitPlan plan_logits(const focus_shape& s, int max_active, bool lean = false);

// ---- small kernels (focus_small.hip)
hipError_t launch_select_queries(const float* conf, const uint8_t* masked, int n_gen, int k, int window, int lo,
                                 int hi, int32_t* focus_idx, int32_t* active_idx, int max_active, int32_t* counts,
                                 hipStream_t st);
// grouped-query attention: index lists of the selection -> lists of rows g * n_gen + i of the [H_kv, group * n_gen, d] view of Q
hipError_t launch_expand_groups(const int32_t* focus_idx, int max_focus, const int32_t* active_idx, int max_active,
                                const int32_t* counts, int n_gen, int group, int32_t* focus_out, int32_t* active_out,
                                int32_t* counts_out, hipStream_t st);
hipError_t launch_block_means(const void* K, const focus_shape& s, float* kbar, hipStream_t st);
// one scan of K that yields the per-head partial relevances (and, if kbar is not null, the block means)
hipError_t launch_block_means_relevance(const void* K, const void* Q, const int32_t* focus_idx, const int32_t* counts,
                                        int n_focus_max, const focus_shape& s, float* kbar, float* part, hipStream_t st);
constexpr int kRelGroup = 4;  // heads whose partial relevances are added before they leave a workgroup
// Eq. 3: new K/V states of the active positions, to be scattered into the cache
struct CacheUpdate {
  const uint16_t* Kn;
  const uint16_t* Vn;
  uint16_t* Kc;
  uint16_t* Vc;
  int64_t nsh, nsn, ksh, ksn, vsh, vsn;
  const int32_t* active_idx;
  const int32_t* counts;
  int max_active, row_base, n_rows, n_heads;
};
CacheUpdate cache_update_args(void* K_cache, void* V_cache, const focus_shape& s, const void* K_new, const void* V_new,
                              int64_t new_stride_h, int64_t new_stride_n, const int32_t* active_idx, const int32_t* counts,
                              int max_active, int row_base);
// update: made by workgroups of the same launch
// partial relevances (sum over the focus queries, not yet scaled): per_head part[H, n_b], else part[ceil(H / 4), n_b], sums over
// groups of four heads
hipError_t launch_block_relevance(const void* Q, const int32_t* focus_idx, const int32_t* counts, int n_focus_max,
                                  const float* kbar, const focus_shape& s, float* part, bool per_head, hipStream_t st,
                                  const CacheUpdate* update = nullptr);
// part [n_heads, n_b] -> [ceil(n_heads / 4), n_b] in place, sums over groups of four heads
hipError_t launch_group_heads(float* part, int n_heads, int n_b, hipStream_t st);
// values[j] = sum_i part[i, j] / (|I_focus| n_heads) when part != nullptr (else values are read), then top-k over values[0..n):
// out[k] ascending indices.  n_parts = n_heads, or ceil(n_heads / 4) groups
hipError_t launch_reduce_topk(const float* part, int n_parts, int n_heads, const int32_t* counts, int n_focus_max, float* values, int n,
                              int k, int32_t* out, hipStream_t st);
// part_ml [H, n_split, q_pad, 2] -> lse2 [H, q_pad]
hipError_t launch_lse_combine(const float* part_ml, int H, int q_pad, int n_split, float* lse2, hipStream_t st);
// Sink selection as a tournament (small N_sink): every 128-key group of the column-mass kernel nominates its own
// Top-N_sink, one more workgroup ranks the nominees.  Limits of that path:
constexpr int kTournamentMaxSinks = 16;
constexpr int kTournamentMaxCand = 4096;  // ceil(M / 128) * n_sink
// Of any path: what the workspaces hold, and the sixteen nominees a thread of sink_rank_kernel keeps in registers.  Prompts past 131072
// rows, whose groups nominate more, are left to the radix select over all masses (16 queries, 32 heads: sink chain 292 us at 131072
// rows, 669 at 131200); longer runs per thread have not been tried.
constexpr int kMaxNominees = 16384;
bool sink_tournament_fits(int M, int n_sink);
// cand: nullptr, or int32[ceil(M / 128) * n_sink] that receives the nominees (n_sink: nominees per group);
// cand_keys: uint32 of the same size that receives their order keys + 1 (0 where cand holds -1); required with cand.
// pre_reduced = false: src = scaled logits [H, ceil(L / 4), 16, 4] of at most 16 queries (written by the MFMA kernels), n_parts = H;
// pre_reduced = true:  src = column sums [n_parts, L] from the second pass over K.
// n_split > 0 (pre_reduced = false): lse2 = the statistics [H, n_split, 16, 2] of the key splits instead of the log-sum-exps
// [H, 16], which are then formed by the same launch or by one more, into lse_scratch.
hipError_t launch_column_mass(const float* src, bool pre_reduced, const float* lse2, const int32_t* counts, int max_active,
                              int n_parts, int H, int L, float* col_mass, int M, int n_sink, int32_t* cand, uint32_t* cand_keys,
                              int n_split, float* lse_scratch, hipStream_t st);
// Many sinks, or few in a long prompt (n_ctx <= 131072): the groups nominate min(kRankNominees, N_sink) each, one workgroup ranks
// them and falls back to all positions if a group may hold more.  No requirement on the alignment of col_mass.
constexpr int kRankNominees = 16;
bool sink_rank_fits(int M, int n_sink);
hipError_t launch_sink_rank(const int32_t* cand, const uint32_t* cand_keys, int M, int n_sink, const float* col_mass, int32_t* sink_idx,
                            hipStream_t st);
hipError_t launch_sink_final(const int32_t* cand, const uint32_t* cand_keys, int M, int n_sink, int32_t* sink_idx,
                             hipStream_t st);

// Eq. 2: tokens[i] = argmax over the vocabulary of row i of the bf16 logits, conf[i] = its softmax probability
// (workspace of token_confidence_workspace() bytes: per-split states when a row is cut into several workgroups)
size_t token_confidence_workspace(int n_rows, int vocab);
hipError_t launch_token_confidence(const void* logits, int64_t row_stride, const uint8_t* masked, int n_rows, int vocab,
                                   int32_t* tokens, float* conf, void* workspace, hipStream_t st);
hipError_t launch_cache_update(const CacheUpdate& u, int head_dim, hipStream_t st);
// block entry: every cache row takes its new state; block means of the prompt keys from the same pass (kbar may be null)
struct CacheRefresh {
  const uint16_t* Kn;
  const uint16_t* Vn;
  uint16_t* Kc;
  uint16_t* Vc;
  int64_t nsh, nsn, ksh, ksn, vsh, vsn;
  int M, L, B, n_b;
  int n_chunks, n_heads;  // chunks of B rows per head: n_b prompt blocks, then the response rows
  float* kbar;
};
CacheRefresh cache_refresh_args(void* K_cache, void* V_cache, const focus_shape& s, const void* K_new, const void* V_new,
                                int64_t new_stride_h, int64_t new_stride_n, float* kbar);
hipError_t launch_cache_refresh(const CacheRefresh& p, int head_dim, hipStream_t st);

// ---- MFMA kernels (focus_mfma.hip)
// mode 0: logits [H, ceil(L / 4), 16, 4] + part_ml out (at most 16 queries); mode 1: part_ml out only; mode 2: lse2 in, or part_ml of
// mode 1 (not null; lse_in_logits), colpart [q_groups * H, L] out
// select (modes 0 and 1): the query selection (Eq. 4, Eq. 5) is made by the same launch; active_idx and counts are not read
bool lse_in_logits(const SplitPlan& p);  // mode 2 may form the log-sum-exps itself
constexpr int kSelectInLogitsGen = 64;  // n_gen at most: a wavefront holds one position per lane
struct SelectArgs {
  const float* conf;
  const uint8_t* masked;
  int k, half, lo, hi;
  int32_t* focus_idx;
  int32_t* active_idx;
  int32_t* counts;
};
hipError_t launch_qk_logits(const void* Q, const int32_t* active_idx, const int32_t* counts, int max_active,
                            const void* K, const focus_shape& s, const SplitPlan& p, int mode, float* logits,
                            float* part_ml, const float* lse2, float* colpart, hipStream_t st, const SelectArgs* select = nullptr);
// Extra arguments of the fused layer path: the attention kernel ranks the blocks itself from the partial relevances
// (n_b <= kFusedMaxBlocks).  The limit is what the prologues are built for: one, four or eight keys a thread of four wavefronts, for each up to
// eight parts requested at once.  The parts of a K scan come per head: up to kFusedMaxBlocksPerHead blocks, one key a thread, 32 of them are
// requested, past that up to eight as of the groups, and of more heads launch_group_heads adds them up first.  Past the limit a launch
// of one workgroup ranks the blocks and costs more than the blocks themselves (16 queries, 30 blocks of 64 kept, launch and prologue: 32 heads, 1025 blocks 36.2 and 22.0 us a layer, 2048 blocks 39.8 and 25.1; 4 heads, 2048 blocks
// 28.8 and 15.5; 1024 blocks with four keys a thread 19.9).
constexpr int kFusedManyBlocks = 1024, kFusedMaxBlocks = 2048, kFusedMaxBlocksPerHead = 256;
struct FusedTopC {
  const float* rel_part;  // [ceil(H / 4), n_b] from launch_block_relevance, or with per_head [H, n_b]
  bool per_head;
  float* scores_out;      // [n_b] or null
  int32_t* kept_out;      // [n_keep]
  int n_focus_max;
  const float* kbar = nullptr;  // relevance_in_attention: there are no partial relevances, the kernel works them out
  const int32_t* focus_idx = nullptr;
};
bool relevance_in_attention(const focus_shape& s, const SplitPlan& p);  // unless outputs and inputs share memory (sparse_layer_impl)

// Memory that a call reads or writes: nothing (lo = hi), or the bytes [lo, hi) from the first to the last row of a tensor, those between
// its rows included.
struct Extent {
  uintptr_t lo = 0, hi = 0;
  bool meets(const Extent& o) const { return lo < o.hi && o.lo < hi; }
};
static inline Extent extent(const void* p, int64_t bytes) {
  Extent e;
  if (p != nullptr && bytes > 0) {
    e.lo = reinterpret_cast<uintptr_t>(p);
    e.hi = e.lo + (uintptr_t)bytes;
  }
  return e;
}
// bf16 [heads, rows, d]; the heads may lie in descending order
static inline Extent extent(const void* p, int64_t stride_h, int64_t stride_n, int heads, int64_t rows, int d) {
  const int64_t last = 2 * (heads - 1) * stride_h;
  const void* first = p == nullptr ? nullptr : static_cast<const char*>(p) + (last < 0 ? last : 0);
  return extent(first, (last < 0 ? -last : last) + 2 * ((rows - 1) * stride_n + d));
}
// True where the outputs of an attention call lie clear of what its attention kernel reads
bool attention_outputs_apart(const void* Q, const int32_t* active_idx, int max_active, const void* K, const void* V, const focus_shape& s,
                             const int32_t* kept_blocks, int n_keep, const int32_t* sink_idx, int n_sink, const void* out, const float* lse);
// Dense (probe) layer: every one of the M + N key rows is attended (kept_blocks / sink_idx unused, plan from
// plan_attention_dense); optionally the scaled logits (at most 16 active queries) and the base-2 row log-sum-exps are
// written for the sink scoring that follows.
struct DenseProbe {
  float* logits_out;  // [H, ceil((M + N) / 4), 16 queries, 4 keys] or null
  float* lse2_out;    // [H, q_pad] or null
};
hipError_t launch_sparse_attn(const void* Q, const int32_t* active_idx, const int32_t* counts, int max_active,
                              const void* K, const void* V, const focus_shape& s, const int32_t* kept_blocks,
                              int n_keep, const int32_t* sink_idx, int n_sink, const SplitPlan& p, void* out,
                              float* lse, float* part_o, float* part_ml, const FusedTopC* fused, hipStream_t st,
                              const DenseProbe* probe = nullptr);

// Block-entry refresh: dense attention of all n_gen rows of Q over all M + N keys (out [H, n_gen, d], lse [H, n_gen])
// copy: the cache refresh of the same layer, on the side of the attention's last launch; K and V are then its new states
hipError_t launch_refresh_attn(const void* Q, const void* K, const void* V, const focus_shape& s, void* out, float* lse,
                               hipStream_t st, const CacheRefresh* copy = nullptr);

}  // namespace focus
