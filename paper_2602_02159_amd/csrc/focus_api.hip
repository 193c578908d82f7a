// extern "C" boundary: argument validation on the host, workspace carving, launch sequencing.
// Nothing here touches the GPU before every argument has been checked.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>

#include "focus_kernels.h"

namespace focus {

static thread_local char g_err[512] = "";

static int fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}

static int launch_fail(const char* what, hipError_t e) {
  return fail(FOCUS_ELAUNCH, "%s: %s", what, hipGetErrorString(e));
}

static inline size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

// Launch shapes (workgroups per launch the key axis is cut for).  Fixed constants: split counts decide workspace
// sizes and the order in which partial results are merged, so they must not vary between calls.
constexpr int kAttnGroups = 512;      // one sub-tile per slot: every workgroup resident at once, two per compute unit
// d = 64, up to 16 queries: half the LDS and few registers, twice as many are resident (four per compute unit without a key loop, whatever
// number of blocks they rank: at most 40 548 bytes, which the kernel asserts; two with one).  One sub-tile per wavefront up to 128 a head
// (32 heads, whole layer against 512 workgroups, 256 blocks to rank: 67 sub-tiles 15.5 -> 13.9 us, 123 17.1 -> 15.4; 512 blocks: 65
// sub-tiles 16.8 -> 15.1, 97 18.2 -> 16.5, 127 19.4 -> 18.1; 2048 blocks: 65 21.6 -> 20.7, 97 23.1 -> 22.6, 127 23.6 and 23.6), then two
// workgroups per compute unit (131 17.9 -> 16.7, 259 23.2 -> 21.8, 1026 51.7 -> 46.5), as long as no more than 64 partial results per row
// come of it: merging them costs a memory round trip for every 64 (4 heads, 1004 sub-tiles: 18.4 us in 64 splits, 23.6 in 251).  32-query tiles (24 queries) gain at 67 sub-tiles
// only (16.6 -> 15.4) and lose from 91 on; nor does the probe layer gain, whose kernel also writes its logits (1026 sub-tiles 80.0 ->
// 80.7).
constexpr int kAttnGroupsSmall = 1024, kAttnGroupsSmallPipe = 512, kAttnSplitsSmall = 64;
// Many sub-tiles per slot: one workgroup per compute unit.  With up to 32 queries, whose slots have one stage, two would be resident, but
// one keeps enough under way, and two leave twice the partial results (256 workgroups and 512, a call: 32 heads, 8256 keys 26.7 and 28.9
// us, 32 832 keys 84.0 and 86.8; 28 queries 28.3 and 31.3, 86.2 and 90.6; half of 512 blocks, 25 queries 51.0 and 53.3; 8 heads, 16 448
// keys 18.6 and 19.8; 4 heads, d = 64, 28 queries, 32 832 keys 13.7 and 15.3; probe layer of 32 832 keys 128.2 and 129.7).  33 to 64
// queries have two stages, and LDS for one.
constexpr int kAttnGroupsPipe = 256;
constexpr int kAttnGroupsWide = 512;  // the same where query groups share the rows: one stage per slot, two workgroups per compute unit
// Sink scoring, one query tile.  About four rounds of sub-tiles per workgroup where all workgroups are resident at once (1024), so that a
// workgroup's start passes beside the others' rows and there are few statistics to merge, and the same number of workgroups for every
// compute unit: with 17 instead of 16 splits of 32 heads some have a third more to do.  Past that, or where one split would have a
// fifth round that nothing runs beside, two rounds in up to kLogitGroups workgroups: short ones even out the tail of the scan.
// Sink chain in us (splits): 32 heads, 8256 keys 32.5 (65), 31.2 (13), 29.2 (16), 33.0 (17), 29.2 (32); 10 100 keys 34.3 (12), 32.2 (16),
// 36.8 (19), 32.5 (24); 15 986 keys 43.8 (31), 42.0 (32); 16 448 keys 46.5 (32), 48.7 (33), 44.9 (65); 32 832 keys 75.4 (128), 73.5
// (129), 78.6 (257); 1056 keys 16.0 (9), 14.9 (8); 16 heads, 32 832 keys 47.1 (256), 42.7 (128), 42.7 (64), 45.6 (65); 8 heads 34.5
// (256), 26.9 (128), 27.2 (64).
constexpr int kLogitGroups = 4096, kLogitGroupsResident = 1024, kLogitGroupsCu = 256, kLogitRounds = 4;
// Two passes over K (more than 16 queries): every workgroup first fetches its query rows.  33 to 64 queries per group: as many
// workgroups as are resident at once, three per compute unit.  Up to 32: four are; more of them even out the tail of a long scan,
// as long as each has four rounds of sub-tiles.
constexpr int kLogitGroupsMany = 768;
constexpr int kLogitGroupsTwo = 2048, kLogitGroupsTwoMin = 512, kLogitRoundsTwo = 4;

// `most`: 16-query tiles per query group at most.  q_pad is the same for every `most`: the rows of per-query results.
static void plan_queries(SplitPlan& p, int max_active, int most) {
  p.q_tiles = ceil_div(max_active, kQTile);
  p.q_tiles_per_group = p.q_tiles <= 2 ? p.q_tiles : most;
  p.q_groups = ceil_div(p.q_tiles, p.q_tiles_per_group);
  p.q_pad = p.q_tiles <= 2 ? p.q_tiles * kQTile : ceil_div(p.q_tiles, kMaxQTilesPerGroup) * kMaxQTilesPerGroup * kQTile;
}

// As many splits as the target allows, at least one round of four sub-tiles each
static void plan_splits(SplitPlan& p, int n_heads, int q_groups, int target_groups) {
  const int per_head = (int)std::max<int64_t>(1, target_groups / ((int64_t)n_heads * q_groups));
  p.n_split = std::max(1, std::min(per_head, ceil_div(p.n_sub, kWavesPerGroup)));
}

static void plan_attention_splits(SplitPlan& p, const focus_shape& s, bool logits_out, bool lean) {
  const bool d64 = s.head_dim == 64 && p.q_tiles == 1 && !logits_out && !lean;
  auto small = [&](int groups) { return d64 && groups / s.n_heads <= kAttnSplitsSmall; };
  plan_splits(p, s.n_heads, p.q_groups, small(kAttnGroupsSmall) ? kAttnGroupsSmall : kAttnGroups);
  // Many sub-tiles per wavefront (dense layers, alpha = 0.5): fewer, longer workgroups with key loops.
  // One sub-tile per wavefront (the 3 % keep configurations): nothing to overlap.
  if (p.n_split * kWavesPerGroup < p.n_sub) {
    plan_splits(p, s.n_heads, p.q_groups, small(kAttnGroupsSmallPipe) ? kAttnGroupsSmallPipe : (p.q_groups > 1 ? kAttnGroupsWide : kAttnGroupsPipe));
    p.pipelined = p.n_split * kWavesPerGroup < p.n_sub;
  }
}

SplitPlan plan_attention(const focus_shape& s, int max_active, int n_keep, int n_sink, bool lean) {
  SplitPlan p;
  plan_queries(p, max_active, max_active <= 64 ? 4 : 2);
  p.n_sub = n_keep * ceil_div(s.block, kSubTile) + ceil_div(s.n_resp, kSubTile) + ceil_div(n_sink, kSubTile);
  plan_attention_splits(p, s, false, lean);
  return p;
}

SplitPlan plan_attention_dense(const focus_shape& s, int max_active) {
  SplitPlan p;
  plan_queries(p, max_active, max_active <= 64 ? 4 : 2);
  p.n_sub = ceil_div(s.n_ctx + s.n_resp, kSubTile);
  plan_attention_splits(p, s, p.q_tiles == 1, false);
  return p;
}

SplitPlan plan_logits(const focus_shape& s, int max_active, bool lean) {
  SplitPlan p;
  plan_queries(p, max_active, kMaxQTilesPerGroup);
  p.n_sub = ceil_div(s.n_ctx + s.n_resp, kSubTile);
  if (p.q_tiles_per_group == 1) {
    const int rounds = ceil_div(p.n_sub, kWavesPerGroup), step = std::max(1, kLogitGroupsCu / s.n_heads);
    const int n = step * std::max(1, (rounds + step * kLogitRounds / 2) / (step * kLogitRounds));  // the nearest multiple of step
    const int64_t groups = (int64_t)n * s.n_heads;
    const bool lone_round = rounds > n * kLogitRounds && groups + (int64_t)step * s.n_heads > kLogitGroupsResident;
    const int most = std::max(1, kLogitGroups / s.n_heads);
    if (groups <= kLogitGroupsResident && !lone_round)
      p.n_split = std::min(rounds, n);
    else  // (one split more than the limit where that saves a lone round)
      p.n_split = ceil_div(rounds, 2) <= most + (lean ? 0 : 1) ? ceil_div(rounds, 2) : most;
    return p;
  }
  plan_splits(p, s.n_heads, p.q_groups, p.q_tiles_per_group == 2 ? kLogitGroupsTwo : kLogitGroupsMany);
  if (p.q_tiles_per_group == 2) {
    const int rounds = p.n_sub / kWavesPerGroup;
    p.n_split = std::min(p.n_split, std::max(std::max(1, kLogitGroupsTwoMin / s.n_heads), rounds / kLogitRoundsTwo));
  }
  return p;
}

// ---- validation helpers -------------------------------------------------------------------------------
static bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

static int check_shape(const focus_shape* s, bool need_q, bool need_k, bool need_v, bool need_o) {
  if (!s) return fail(FOCUS_EINVAL, "shape is NULL");
  if (s->n_heads < 1 || s->n_ctx < 1 || s->n_resp < 0 || s->block < 1 || s->n_gen < 1)
    return fail(FOCUS_EINVAL, "shape: n_heads=%d n_ctx=%d n_resp=%d block=%d n_gen=%d out of range", s->n_heads,
                s->n_ctx, s->n_resp, s->block, s->n_gen);
  if (s->head_dim != 64 && s->head_dim != 128)
    return fail(FOCUS_EUNSUPPORTED, "head_dim=%d: only 64 and 128 are built", s->head_dim);
  if ((int64_t)s->n_ctx + s->n_resp > (1 << 30)) return fail(FOCUS_EUNSUPPORTED, "more than 2^30 key rows");
  const int64_t d = s->head_dim, L = (int64_t)s->n_ctx + s->n_resp;
  auto bad = [&](int64_t sh, int64_t sn, int64_t) { return sn < d || (sn & 7) || sh < 0 || (sh & 7); };
  if (need_q && bad(s->q_stride_h, s->q_stride_n, s->n_gen)) return fail(FOCUS_EINVAL, "Q strides invalid or not multiples of 8");
  if (need_k && bad(s->k_stride_h, s->k_stride_n, L)) return fail(FOCUS_EINVAL, "K strides invalid or not multiples of 8");
  if (need_v && bad(s->v_stride_h, s->v_stride_n, L)) return fail(FOCUS_EINVAL, "V strides invalid or not multiples of 8");
  if (need_o && (s->o_stride_n < d || (s->o_stride_n & 7) || (s->o_stride_h & 7)))
    return fail(FOCUS_EINVAL, "output strides invalid or not multiples of 8");
  return FOCUS_OK;
}

struct ScoreWs {
  size_t part, scores, total;
};
static ScoreWs ws_block_scores(const focus_shape& s) {
  const size_t n_b = ceil_div(s.n_ctx, s.block);
  ScoreWs w;
  w.part = 0;
  w.scores = w.part + align_up((size_t)s.n_heads * n_b * sizeof(float));  // per head: the K scan's layout
  w.total = w.scores + align_up(n_b * sizeof(float));
  return w;
}

struct SinkWs {
  size_t logits, part_ml, lse2, col_mass, cand, total;
};
// At most 16 active queries: one pass over K that spills the scaled logits (64 bytes per key and head), which the
// column-mass kernel re-reads.  More: the spill would outweigh K itself, so K is scanned twice — statistics first,
// then probabilities summed over the queries on the fly — and only [q_groups * H, L] column sums are stored.
static bool sinks_two_pass(const SplitPlan& p) { return p.q_pad > 16; }
// the spilled logits of at most 16 queries: [H, ceil(L / 4), 16 queries, 4 keys] fp32
static size_t spilled_logits_bytes(const focus_shape& s) {
  const size_t L = (size_t)s.n_ctx + s.n_resp;
  return (size_t)s.n_heads * ((L + 3) / 4) * 16 * 4 * sizeof(float);
}

static SinkWs ws_find_sinks(const focus_shape& s, const SplitPlan& p) {
  SinkWs w;
  const size_t L = (size_t)s.n_ctx + s.n_resp;
  w.logits = 0;  // logits [H, ceil(L / 4), 16, 4], or column sums [q_groups * H, L]
  size_t off = align_up(sinks_two_pass(p) ? (size_t)p.q_groups * s.n_heads * L * sizeof(float) : spilled_logits_bytes(s));
  w.part_ml = off;
  off += align_up((size_t)s.n_heads * p.q_pad * p.n_split * 2 * sizeof(float));
  w.lse2 = off;
  off += align_up((size_t)s.n_heads * p.q_pad * sizeof(float));
  w.col_mass = off;
  off += align_up(L * sizeof(float));
  w.cand = off;  // nominees of the 128-key groups: positions, then their keys
  off += align_up((size_t)2 * kMaxNominees * sizeof(int32_t));
  w.total = off;
  return w;
}

struct ProbeWs {
  size_t part_o, part_ml, lse2, scratch, col_mass, cand, total;  // scratch: logits [H, ceil(L / 4), 16, 4] or column sums [q_groups H, L]
};
struct AttnWs {
  size_t part_o, part_ml, total;
};
static AttnWs ws_attn(const focus_shape& s, const SplitPlan& p) {
  AttnWs w;
  w.part_o = 0;
  if (p.n_split <= 1) {  // a single key split writes the output itself: no partial results
    w.part_ml = 0;
    w.total = 256;
    return w;
  }
  size_t off = align_up((size_t)s.n_heads * p.q_pad * p.n_split * s.head_dim * sizeof(float));
  w.part_ml = off;
  off += align_up((size_t)s.n_heads * p.q_pad * p.n_split * 2 * sizeof(float));
  w.total = off;
  return w;
}

static ProbeWs ws_probe_layer(const focus_shape& s, const SplitPlan& pa, const SplitPlan& pl) {
  ProbeWs w;
  const size_t L = (size_t)s.n_ctx + s.n_resp;
  const AttnWs a = ws_attn(s, pa);
  w.part_o = a.part_o;
  w.part_ml = a.part_ml;
  size_t off = a.total;
  w.lse2 = off;
  off += align_up((size_t)s.n_heads * pa.q_pad * sizeof(float));
  w.scratch = off;
  off += align_up(sinks_two_pass(pl) ? (size_t)pl.q_groups * s.n_heads * L * sizeof(float) : spilled_logits_bytes(s));
  w.col_mass = off;
  off += align_up(L * sizeof(float));
  w.cand = off;  // as above
  off += align_up((size_t)2 * kMaxNominees * sizeof(int32_t));
  w.total = off;
  return w;
}

// Second half of the sink identification: column masses S from the kept logits or per-part column sums, then Top-N_sink.  Few
// sinks, or not too many: the 128-key groups of the column-mass kernel nominate and one workgroup decides (a tournament of up to 16
// sinks, or a ranking of all nominees); else a radix select.
// lse2: row log-sum-exps, or with n_split > 0 the statistics of the key splits (then lse_scratch takes the log-sum-exps).
static int column_mass_and_sinks(const char* who, const float* src, bool two_pass, const float* lse2, int n_split, float* lse_scratch,
                                 const int32_t* counts, int max_active, int q_groups, const focus_shape& s, int n_sink, float* S,
                                 char* cand_ws, int32_t* sink_idx, hipStream_t st) {
  const bool tournament = sink_tournament_fits(s.n_ctx, n_sink), rank = !tournament && sink_rank_fits(s.n_ctx, n_sink);
  int32_t* cand = (tournament || rank) ? reinterpret_cast<int32_t*>(cand_ws) : nullptr;
  uint32_t* cand_keys = cand ? reinterpret_cast<uint32_t*>(cand_ws) + kMaxNominees : nullptr;
  hipError_t e = launch_column_mass(src, two_pass, lse2, counts, max_active, two_pass ? q_groups * s.n_heads : s.n_heads, s.n_heads,
                                    s.n_ctx + s.n_resp, S, s.n_ctx, rank ? std::min(n_sink, kRankNominees) : n_sink, cand, cand_keys, n_split,
                                    lse_scratch, st);
  if (e != hipSuccess) return fail(FOCUS_ELAUNCH, "%s(column mass): %s", who, hipGetErrorString(e));
  if (tournament)
    e = launch_sink_final(cand, cand_keys, s.n_ctx, n_sink, sink_idx, st);
  else if (rank)
    e = launch_sink_rank(cand, cand_keys, s.n_ctx, n_sink, S, sink_idx, st);
  else if (n_sink > 0)
    e = launch_reduce_topk(nullptr, 0, 0, nullptr, 0, S, s.n_ctx, n_sink, sink_idx, st);
  if (e != hipSuccess) return fail(FOCUS_ELAUNCH, "%s(top-N): %s", who, hipGetErrorString(e));
  return FOCUS_OK;
}

static int check_select(const char* who, const float* conf, int32_t n_gen, int32_t k, int32_t window, int32_t lo, int32_t hi,
                        const int32_t* focus_idx, const int32_t* active_idx, int32_t max_active, const int32_t* counts) {
  if (!conf || !focus_idx || !active_idx || !counts) return fail(FOCUS_EINVAL, "%s: NULL pointer", who);
  if (n_gen < 1 || n_gen > 16384) return fail(FOCUS_EINVAL, "%s: n_gen=%d not in [1, 16384]", who, n_gen);
  if (k < 1 || k > n_gen) return fail(FOCUS_EINVAL, "%s: k=%d not in [1, n_gen=%d]", who, k, n_gen);
  if (window < 0) return fail(FOCUS_EINVAL, "%s: window=%d negative", who, window);
  if (lo < 0 || hi > n_gen || lo >= hi) return fail(FOCUS_EINVAL, "%s: [lo=%d, hi=%d) not inside [0, %d)", who, lo, hi, n_gen);
  const int64_t span = 2 * (int64_t)(window / 2) + 1;
  const int64_t need = std::min<int64_t>(hi - lo, (int64_t)k * span);
  if (max_active < need) return fail(FOCUS_EINVAL, "%s: max_active=%d < %lld", who, max_active, (long long)need);
  return FOCUS_OK;
}

// select != nullptr: the query selection comes first, in the logits launch where the block is small enough for that.
static int find_sinks_impl(const char* who, const SelectArgs* select, const void* Q, const int32_t* active_idx, const int32_t* counts,
                           int32_t max_active, const void* K, const focus_shape* shape, int32_t n_sink, float* col_mass,
                           int32_t* sink_idx, void* workspace, size_t ws_bytes, void* stream) {
  if (int rc = check_shape(shape, true, true, false, false)) return rc;
  if (!Q || !active_idx || !K) return fail(FOCUS_EINVAL, "%s: NULL pointer", who);
  if (max_active < 1 || max_active > shape->n_gen) return fail(FOCUS_EINVAL, "%s: max_active=%d not in [1, n_gen]", who, max_active);
  if (n_sink < 0 || n_sink > shape->n_ctx) return fail(FOCUS_EINVAL, "%s: n_sink=%d not in [0, n_ctx]", who, n_sink);
  if (n_sink > 0 && !sink_idx) return fail(FOCUS_EINVAL, "%s: sink_idx is NULL", who);
  if (!aligned16(Q) || !aligned16(K)) return fail(FOCUS_EINVAL, "%s: pointers must be 16-byte aligned", who);
  SplitPlan p = plan_logits(*shape, max_active);
  SinkWs w = ws_find_sinks(*shape, p);
  if (ws_bytes < w.total) w = ws_find_sinks(*shape, p = plan_logits(*shape, max_active, true));
  if (!workspace || ws_bytes < w.total || !aligned16(workspace))
    return fail(FOCUS_EWORKSPACE, "%s: workspace needs %zu bytes, 16-byte aligned", who, w.total);
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  float* logits = reinterpret_cast<float*>(ws + w.logits);
  float* part_ml = reinterpret_cast<float*>(ws + w.part_ml);
  float* lse2 = reinterpret_cast<float*>(ws + w.lse2);
  float* S = col_mass ? col_mass : reinterpret_cast<float*>(ws + w.col_mass);
  const bool two_pass = sinks_two_pass(p);
  hipError_t e = hipSuccess;
  if (select != nullptr && shape->n_gen > kSelectInLogitsGen) {
    e = launch_select_queries(select->conf, select->masked, shape->n_gen, select->k, 2 * select->half, select->lo, select->hi,
                              select->focus_idx, select->active_idx, max_active, select->counts, st);
    if (e != hipSuccess) return fail(FOCUS_ELAUNCH, "%s(selection): %s", who, hipGetErrorString(e));
    select = nullptr;
  }
  e = launch_qk_logits(Q, active_idx, counts, max_active, K, *shape, p, two_pass ? 1 : 0, logits, part_ml, nullptr, nullptr, st, select);
  if (e != hipSuccess) return fail(FOCUS_ELAUNCH, "%s(logits): %s", who, hipGetErrorString(e));
  if (two_pass) {
    const bool in_logits = lse_in_logits(p);
    if (!in_logits) {
      e = launch_lse_combine(part_ml, shape->n_heads, p.q_pad, p.n_split, lse2, st);
      if (e != hipSuccess) return fail(FOCUS_ELAUNCH, "%s(lse): %s", who, hipGetErrorString(e));
    }
    e = launch_qk_logits(Q, active_idx, counts, max_active, K, *shape, p, 2, nullptr, in_logits ? part_ml : nullptr, lse2, logits, st);
    if (e != hipSuccess) return fail(FOCUS_ELAUNCH, "%s(column sums): %s", who, hipGetErrorString(e));
  }
  return column_mass_and_sinks(who, logits, two_pass, two_pass ? lse2 : part_ml, two_pass ? 0 : p.n_split, lse2, counts, max_active,
                               p.q_groups, *shape, n_sink, S, ws + w.cand, sink_idx, st);
}

constexpr size_t kStaticScratchBytes = (size_t)8 << 20;  // the array of focus_sparse_layer_static

struct LayerWs {
  size_t attn, need, total;  // need <= total: with less than total, more than kFusedManyBlocks blocks are ranked by a launch of their own
  ScoreWs sc;
  AttnWs at;
};
// A launch that ranks the blocks is the last to read the relevances, and the attention's partial results may take their place; inside
// the attention kernel both are in use.  Up to kFusedManyBlocks blocks the two always have places of their own.  (Were that so for any
// number, 50 000 blocks and more of 32 heads could exceed the scratch array of focus_sparse_layer_static by the few per cent that the
// splits of the attention had grown.)
static LayerWs ws_layer(const focus_shape& s, const SplitPlan& p) {
  const int n_b = ceil_div(s.n_ctx, s.block);
  LayerWs w;
  w.sc = ws_block_scores(s);
  w.at = ws_attn(s, p);
  w.attn = w.sc.total;
  const size_t apart = w.attn + w.at.total, shared = std::max(w.sc.total, w.at.total);
  w.need = n_b > kFusedManyBlocks ? shared : apart;
  w.total = n_b > kFusedMaxBlocks ? shared : apart;
  if (w.need <= kStaticScratchBytes && w.total > kStaticScratchBytes) w.total = w.need;  // (what the static call takes shows in the size)
  return w;
}

// ---- scratch memory for callers that cannot allocate (focus_sparse_layer_static) --------------------------------
// One array per GPU, resident from the moment the library's code object is loaded on that GPU until the process ends.
// In host code the array's name is only a stand-in: its device address is looked up once per device with
// hipGetSymbolAddress and that pointer is what the kernels receive.
static __device__ __align__(256) unsigned char g_static_scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
static void* g_scratch_addr[kMaxDevices];  // by device ordinal; nullptr = not looked up yet
static std::mutex g_scratch_mutex;

static int static_scratch_ptr(void** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return launch_fail("focus_sparse_layer_static(hipGetDevice)", e);
  if (dev < 0 || dev >= kMaxDevices) return fail(FOCUS_EUNSUPPORTED, "focus_sparse_layer_static: device ordinal %d not below %d", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_addr[dev] == nullptr) {  // first call on this device, which is the current one
    void* ptr = nullptr;
    e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(g_static_scratch));
    if (e != hipSuccess || ptr == nullptr) return launch_fail("focus_sparse_layer_static(hipGetSymbolAddress)", e);
    g_scratch_addr[dev] = ptr;
  }
  *out = g_scratch_addr[dev];
  return FOCUS_OK;
}

static int check_cache_update(const char* who, const void* K_cache, const void* V_cache, const focus_shape* shape, const void* K_new,
                              const void* V_new, int64_t new_stride_h, int64_t new_stride_n, const int32_t* active_idx, int32_t max_active) {
  if (int rc = check_shape(shape, false, true, true, false)) return rc;
  if (!K_cache || !V_cache || !K_new || !V_new || !active_idx) return fail(FOCUS_EINVAL, "%s: NULL pointer", who);
  if (max_active < 1 || max_active > 65535) return fail(FOCUS_EINVAL, "%s: max_active=%d not in [1, 65535]", who, max_active);
  if (new_stride_n < shape->head_dim || (new_stride_n & 7) || new_stride_h < 0 || (new_stride_h & 7))
    return fail(FOCUS_EINVAL, "%s: strides of the new states invalid or not multiples of 8", who);
  if (!aligned16(K_cache) || !aligned16(V_cache) || !aligned16(K_new) || !aligned16(V_new))
    return fail(FOCUS_EINVAL, "%s: pointers must be 16-byte aligned", who);
  return FOCUS_OK;
}

static int sparse_layer_impl(const char* who, const void* Q, const int32_t* focus_idx, const int32_t* active_idx,
                             const int32_t* counts, int32_t n_focus_max, int32_t max_active, const void* K, const void* V,
                             const float* kbar, const focus_shape* shape, int32_t n_keep, const int32_t* sink_idx,
                             int32_t n_sink, float* scores, int32_t* kept_blocks, void* out, float* lse, void* workspace,
                             size_t ws_bytes, bool static_scratch, void* stream, const CacheUpdate* update = nullptr) {
  if (int rc = check_shape(shape, true, true, true, true)) return rc;
  if (!Q || !focus_idx || !active_idx || !K || !V || !out) return fail(FOCUS_EINVAL, "%s: NULL pointer", who);
  const int n_b = ceil_div(shape->n_ctx, shape->block);
  if (n_focus_max < 1 || n_focus_max > shape->n_gen) return fail(FOCUS_EINVAL, "%s: n_focus_max=%d not in [1, n_gen]", who, n_focus_max);
  if (max_active < 1 || max_active > shape->n_gen) return fail(FOCUS_EINVAL, "%s: max_active=%d not in [1, n_gen]", who, max_active);
  if (n_keep < 0 || n_keep > n_b) return fail(FOCUS_EINVAL, "%s: n_keep=%d not in [0, n_b=%d]", who, n_keep, n_b);
  if (n_sink < 0 || n_sink > shape->n_ctx) return fail(FOCUS_EINVAL, "%s: n_sink=%d not in [0, n_ctx]", who, n_sink);
  if ((n_keep > 0 && !kept_blocks) || (n_sink > 0 && !sink_idx)) return fail(FOCUS_EINVAL, "%s: index array is NULL", who);
  if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(out) || (kbar && !aligned16(kbar)))
    return fail(FOCUS_EINVAL, "%s: pointers must be 16-byte aligned", who);
  SplitPlan p = plan_attention(*shape, max_active, n_keep, n_sink);
  LayerWs w = ws_layer(*shape, p);
  if (!static_scratch && ws_bytes < w.need) w = ws_layer(*shape, p = plan_attention(*shape, max_active, n_keep, n_sink, true));
  if (static_scratch) {  // every argument has been checked by now: look the built-in array up (first call on a device) and use it
    if (kStaticScratchBytes < w.need)
      return fail(FOCUS_EWORKSPACE, "%s: this shape needs %zu bytes of scratch, the built-in array holds %zu; use focus_sparse_layer with a caller workspace",
                  who, w.need, kStaticScratchBytes);
    if (int rc = static_scratch_ptr(&workspace)) return rc;
    ws_bytes = kStaticScratchBytes;
  }
  if (!workspace || ws_bytes < w.need || !aligned16(workspace))
    return fail(FOCUS_EWORKSPACE, "%s: workspace needs %zu bytes, 16-byte aligned", who, w.need);
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  const bool apart = ws_bytes >= w.attn + w.at.total;  // (else n_b > kFusedManyBlocks)
  const bool fused = n_b <= kFusedMaxBlocks && n_keep > 0 && apart;
  // The parts of a K scan are per head.  More than the attention kernel requests at once are added up by a launch in between.
  const bool grouped = fused && !kbar && n_b > kFusedMaxBlocksPerHead && shape->n_heads > 8;
  const size_t attn = apart ? w.attn : 0;
  float* part = reinterpret_cast<float*>(ws + w.sc.part);
  float* R = scores ? scores : reinterpret_cast<float*>(ws + w.sc.scores);
  float* part_o = reinterpret_cast<float*>(ws + attn + w.at.part_o);
  float* part_ml = reinterpret_cast<float*>(ws + attn + w.at.part_ml);
  hipError_t e = hipSuccess;
  // (one launch then reads what a launch of its own had read before any output was written: as in attention_outputs_apart)
  auto relevance_inputs_apart = [&]() {
    const Extent read[] = {extent(Q, shape->q_stride_h, shape->q_stride_n, shape->n_heads, shape->n_gen, shape->head_dim),
                           extent(kbar, (int64_t)shape->n_heads * n_b * shape->head_dim * 4), extent(focus_idx, (int64_t)n_focus_max * 4)};
    const Extent written[] = {extent(out, shape->o_stride_h, shape->o_stride_n, shape->n_heads, max_active, shape->head_dim),
                              extent(lse, (int64_t)shape->n_heads * max_active * 4), extent(R, (int64_t)n_b * 4), extent(kept_blocks, (int64_t)n_keep * 4)};
    for (const Extent& r : read)
      for (const Extent& o : written)
        if (r.meets(o)) return false;
    return true;
  };
  const bool inner = fused && kbar && relevance_in_attention(*shape, p) && relevance_inputs_apart() &&
                     attention_outputs_apart(Q, active_idx, max_active, K, V, *shape, nullptr, 0, sink_idx, n_sink, out, lse);
  if (update != nullptr && (!kbar || inner)) {  // no launch that reads nothing of the cache
    e = launch_cache_update(*update, shape->head_dim, st);
    if (e != hipSuccess) return launch_fail("focus_sparse_layer(cache update)", e);
    update = nullptr;
  }
  if (!kbar)
    e = launch_block_means_relevance(K, Q, focus_idx, counts, n_focus_max, *shape, nullptr, part, st);
  else if (!inner)
    e = launch_block_relevance(Q, focus_idx, counts, n_focus_max, kbar, *shape, part, false, st, update);
  if (e == hipSuccess && grouped) e = launch_group_heads(part, shape->n_heads, n_b, st);
  if (e != hipSuccess) return launch_fail("focus_sparse_layer(relevance)", e);
  if (fused) {
    FusedTopC f;
    f.rel_part = part;
    f.per_head = kbar == nullptr && !grouped;
    f.scores_out = R;
    f.kept_out = kept_blocks;
    f.n_focus_max = n_focus_max;
    if (inner) {
      f.kbar = kbar;
      f.focus_idx = focus_idx;
    }
    e = launch_sparse_attn(Q, active_idx, counts, max_active, K, V, *shape, nullptr, n_keep, sink_idx, n_sink, p, out, lse,
                           part_o, part_ml, &f, st);
    if (e != hipSuccess) return launch_fail("focus_sparse_layer(attention)", e);
    return FOCUS_OK;
  }
  e = launch_reduce_topk(part, kbar ? ceil_div(shape->n_heads, kRelGroup) : shape->n_heads, shape->n_heads, counts, n_focus_max, R, n_b, n_keep, kept_blocks, st);
  if (e != hipSuccess) return launch_fail("focus_sparse_layer(top-C)", e);
  e = launch_sparse_attn(Q, active_idx, counts, max_active, K, V, *shape, kept_blocks, n_keep, sink_idx, n_sink, p, out, lse,
                         part_o, part_ml, nullptr, st);
  if (e != hipSuccess) return launch_fail("focus_sparse_layer(attention)", e);
  return FOCUS_OK;
}

}  // namespace focus

using namespace focus;

extern "C" {

const char* focus_last_error(void) { return g_err; }
const char* focus_version(void) { return "focus-gfx950 0.1"; }

int32_t focus_helper_k(double rho, int32_t n_unmask) { return (int32_t)std::floor(rho * (double)n_unmask + 0.5); }
int32_t focus_helper_n_keep(double alpha, int32_t n_blocks) { return (int32_t)std::floor(alpha * (double)n_blocks); }
int32_t focus_helper_n_sink(double frac, int32_t n_ctx) { return (int32_t)std::floor(frac * (double)n_ctx); }

size_t focus_workspace_bytes(int32_t fn, const focus_shape* shape, int32_t max_active, int32_t n_keep, int32_t n_sink) {
  if (check_shape(shape, false, false, false, false) != FOCUS_OK) return 0;
  const int n_b = ceil_div(shape->n_ctx, shape->block);
  switch (fn) {
    case FOCUS_FN_BLOCK_SCORES:
      return ws_block_scores(*shape).total;
    case FOCUS_FN_FIND_SINKS:
      if (max_active < 1 || max_active > shape->n_gen) return 0;
      return ws_find_sinks(*shape, plan_logits(*shape, max_active)).total;
    case FOCUS_FN_SPARSE_ATTN:
      if (max_active < 1 || max_active > shape->n_gen || n_keep < 0 || n_keep > n_b || n_sink < 0 ||
          n_sink > shape->n_ctx)
        return 0;
      return ws_attn(*shape, plan_attention(*shape, max_active, n_keep, n_sink)).total;
    case FOCUS_FN_PROBE_LAYER:
      if (max_active < 1 || max_active > shape->n_gen) return 0;
      return ws_probe_layer(*shape, plan_attention_dense(*shape, max_active), plan_logits(*shape, max_active)).total;
    case FOCUS_FN_SPARSE_LAYER:
      if (max_active < 1 || max_active > shape->n_gen || n_keep < 0 || n_keep > n_b || n_sink < 0 ||
          n_sink > shape->n_ctx)
        return 0;
      return ws_layer(*shape, plan_attention(*shape, max_active, n_keep, n_sink)).total;
    default:
      fail(FOCUS_EINVAL, "focus_workspace_bytes: unknown function id %d", fn);
      return 0;
  }
}

int focus_select_queries(const float* conf, const uint8_t* masked, int32_t n_gen, int32_t k, int32_t window, int32_t lo,
                         int32_t hi, int32_t* focus_idx, int32_t* active_idx, int32_t max_active, int32_t* counts,
                         void* stream) {
  if (int rc = check_select("focus_select_queries", conf, n_gen, k, window, lo, hi, focus_idx, active_idx, max_active, counts)) return rc;
  hipError_t e = launch_select_queries(conf, masked, n_gen, k, window, lo, hi, focus_idx, active_idx, max_active, counts,
                                       static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return launch_fail("focus_select_queries", e);
  return FOCUS_OK;
}

int focus_expand_groups(const int32_t* focus_idx, int32_t max_focus, const int32_t* active_idx, int32_t max_active,
                        const int32_t* counts, int32_t n_gen, int32_t group, int32_t* focus_out, int32_t* active_out,
                        int32_t* counts_out, void* stream) {
  if (!focus_idx || !active_idx || !focus_out || !active_out || !counts_out)
    return fail(FOCUS_EINVAL, "focus_expand_groups: NULL pointer");
  if (n_gen < 1 || group < 1 || max_focus < 1 || max_active < 1)
    return fail(FOCUS_EINVAL, "focus_expand_groups: n_gen=%d group=%d max_focus=%d max_active=%d must be positive", n_gen, group,
                max_focus, max_active);
  if ((int64_t)group * n_gen > (1 << 30) || (int64_t)group * std::max(max_focus, max_active) > (1 << 30))
    return fail(FOCUS_EUNSUPPORTED, "focus_expand_groups: more than 2^30 rows");
  hipError_t e = launch_expand_groups(focus_idx, max_focus, active_idx, max_active, counts, n_gen, group, focus_out, active_out,
                                      counts_out, static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return launch_fail("focus_expand_groups", e);
  return FOCUS_OK;
}

int focus_block_means(const void* K, const focus_shape* shape, float* kbar, void* stream) {
  if (int rc = check_shape(shape, false, true, false, false)) return rc;
  if (!K || !kbar) return fail(FOCUS_EINVAL, "focus_block_means: NULL pointer");
  if (!aligned16(K) || !aligned16(kbar)) return fail(FOCUS_EINVAL, "focus_block_means: pointers must be 16-byte aligned");
  hipError_t e = launch_block_means(K, *shape, kbar, static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return launch_fail("focus_block_means", e);
  return FOCUS_OK;
}

int focus_block_scores(const void* Q, const int32_t* focus_idx, const int32_t* counts, int32_t n_focus_max, const void* K,
                       const float* kbar, const focus_shape* shape, int32_t n_keep, float* scores, int32_t* kept_blocks,
                       void* workspace, size_t ws_bytes, void* stream) {
  if (int rc = check_shape(shape, true, kbar == nullptr, false, false)) return rc;
  if (!Q || !focus_idx) return fail(FOCUS_EINVAL, "focus_block_scores: NULL pointer");
  if (!kbar && !K) return fail(FOCUS_EINVAL, "focus_block_scores: both kbar and K are NULL");
  const int n_b = ceil_div(shape->n_ctx, shape->block);
  if (n_focus_max < 1 || n_focus_max > shape->n_gen) return fail(FOCUS_EINVAL, "focus_block_scores: n_focus_max=%d not in [1, n_gen]", n_focus_max);
  if (n_keep < 0 || n_keep > n_b) return fail(FOCUS_EINVAL, "focus_block_scores: n_keep=%d not in [0, n_b=%d]", n_keep, n_b);
  if (n_keep > 0 && !kept_blocks) return fail(FOCUS_EINVAL, "focus_block_scores: kept_blocks is NULL");
  if (!aligned16(Q) || (kbar && !aligned16(kbar)) || (!kbar && !aligned16(K)))
    return fail(FOCUS_EINVAL, "focus_block_scores: pointers must be 16-byte aligned");
  const ScoreWs w = ws_block_scores(*shape);
  if (!workspace || ws_bytes < w.total || !aligned16(workspace))
    return fail(FOCUS_EWORKSPACE, "focus_block_scores: workspace needs %zu bytes, 16-byte aligned", w.total);
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  float* part = reinterpret_cast<float*>(ws + w.part);
  float* R = scores ? scores : reinterpret_cast<float*>(ws + w.scores);
  hipError_t e;
  if (!kbar)  // one scan of K gives the partial relevances directly; the means are not materialised
    e = launch_block_means_relevance(K, Q, focus_idx, counts, n_focus_max, *shape, nullptr, part, st);
  else
    e = launch_block_relevance(Q, focus_idx, counts, n_focus_max, kbar, *shape, part, false, st);
  if (e != hipSuccess) return launch_fail("focus_block_scores(relevance)", e);
  e = launch_reduce_topk(part, kbar ? ceil_div(shape->n_heads, kRelGroup) : shape->n_heads, shape->n_heads, counts, n_focus_max, R, n_b, n_keep, kept_blocks, st);
  if (e != hipSuccess) return launch_fail("focus_block_scores(top-C)", e);
  return FOCUS_OK;
}

int focus_block_partials(const void* Q, const int32_t* focus_idx, const int32_t* counts, int32_t n_focus_max, const void* K,
                         const float* kbar, const focus_shape* shape, float* partials, void* stream) {
  if (int rc = check_shape(shape, true, kbar == nullptr, false, false)) return rc;
  if (!Q || !focus_idx || !partials) return fail(FOCUS_EINVAL, "focus_block_partials: NULL pointer");
  if (!kbar && !K) return fail(FOCUS_EINVAL, "focus_block_partials: both kbar and K are NULL");
  if (n_focus_max < 1 || n_focus_max > shape->n_gen) return fail(FOCUS_EINVAL, "focus_block_partials: n_focus_max=%d not in [1, n_gen]", n_focus_max);
  if (!aligned16(Q) || (kbar && !aligned16(kbar)) || (!kbar && !aligned16(K)))
    return fail(FOCUS_EINVAL, "focus_block_partials: pointers must be 16-byte aligned");
  hipStream_t st = static_cast<hipStream_t>(stream);
  hipError_t e = kbar ? launch_block_relevance(Q, focus_idx, counts, n_focus_max, kbar, *shape, partials, true, st)
                      : launch_block_means_relevance(K, Q, focus_idx, counts, n_focus_max, *shape, nullptr, partials, st);
  if (e != hipSuccess) return launch_fail("focus_block_partials", e);
  return FOCUS_OK;
}

int focus_top_blocks(const float* partials, int32_t n_parts, const int32_t* counts, int32_t n_focus_max, int32_t n_blocks,
                     int32_t n_keep, float* scores, int32_t* kept_blocks, void* stream) {
  if (!partials || !scores) return fail(FOCUS_EINVAL, "focus_top_blocks: NULL pointer");
  if (n_parts < 1 || n_parts > 1024) return fail(FOCUS_EINVAL, "focus_top_blocks: n_parts=%d not in [1, 1024]", n_parts);
  if (n_blocks < 1) return fail(FOCUS_EINVAL, "focus_top_blocks: n_blocks=%d", n_blocks);
  if (n_focus_max < 1) return fail(FOCUS_EINVAL, "focus_top_blocks: n_focus_max=%d", n_focus_max);
  if (n_keep < 0 || n_keep > n_blocks) return fail(FOCUS_EINVAL, "focus_top_blocks: n_keep=%d not in [0, n_blocks=%d]", n_keep, n_blocks);
  if (n_keep > 0 && !kept_blocks) return fail(FOCUS_EINVAL, "focus_top_blocks: kept_blocks is NULL");
  hipError_t e = launch_reduce_topk(partials, n_parts, n_parts, counts, n_focus_max, scores, n_blocks, n_keep, kept_blocks,
                                    static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return launch_fail("focus_top_blocks", e);
  return FOCUS_OK;
}

int focus_find_sinks(const void* Q, const int32_t* active_idx, const int32_t* counts, int32_t max_active, const void* K,
                     const focus_shape* shape, int32_t n_sink, float* col_mass, int32_t* sink_idx, void* workspace,
                     size_t ws_bytes, void* stream) {
  return find_sinks_impl("focus_find_sinks", nullptr, Q, active_idx, counts, max_active, K, shape, n_sink, col_mass, sink_idx, workspace,
                         ws_bytes, stream);
}

int focus_select_and_find_sinks(const float* conf, const uint8_t* masked, int32_t k, int32_t window, int32_t lo, int32_t hi,
                                int32_t* focus_idx, int32_t* active_idx, int32_t max_active, int32_t* counts, const void* Q,
                                const void* K, const focus_shape* shape, int32_t n_sink, float* col_mass, int32_t* sink_idx,
                                void* workspace, size_t ws_bytes, void* stream) {
  if (int rc = check_shape(shape, true, true, false, false)) return rc;
  if (int rc = check_select("focus_select_and_find_sinks", conf, shape->n_gen, k, window, lo, hi, focus_idx, active_idx, max_active, counts))
    return rc;
  SelectArgs sel;
  sel.conf = conf;
  sel.masked = masked;
  sel.k = k;
  sel.half = window / 2;
  sel.lo = lo;
  sel.hi = hi;
  sel.focus_idx = focus_idx;
  sel.active_idx = active_idx;
  sel.counts = counts;
  return find_sinks_impl("focus_select_and_find_sinks", &sel, Q, active_idx, counts, max_active, K, shape, n_sink, col_mass, sink_idx,
                         workspace, ws_bytes, stream);
}

size_t focus_token_confidence_workspace(int32_t n_rows, int32_t vocab) {
  if (n_rows < 1 || n_rows > 65535 || vocab < 1) return 0;
  return std::max<size_t>(token_confidence_workspace(n_rows, vocab), 16);
}

static int check_refresh_attn(const char* who, const void* Q, const void* K, const void* V, const focus_shape* shape, const void* out,
                              int64_t k_row, int64_t v_row) {
  if (!Q || !K || !V || !out) return fail(FOCUS_EINVAL, "%s: NULL pointer", who);
  if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(out))
    return fail(FOCUS_EINVAL, "%s: pointers must be 16-byte aligned", who);
  if ((int64_t)ceil_div(shape->n_gen, 128) * shape->n_heads > 0x3fffffff) return fail(FOCUS_EUNSUPPORTED, "%s: grid too large", who);
  if (k_row >= (1 << 25) || v_row >= (1 << 25))  // 32-row byte offsets are kept in 32 bits
    return fail(FOCUS_EUNSUPPORTED, "%s: K/V row stride must be below 2^25 elements", who);
  return FOCUS_OK;
}

static int check_cache_refresh(const char* who, const void* K_cache, const void* V_cache, const focus_shape* shape, const void* K_new,
                               const void* V_new, int64_t new_stride_h, int64_t new_stride_n, const float* kbar) {
  if (!K_cache || !V_cache || !K_new || !V_new) return fail(FOCUS_EINVAL, "%s: NULL pointer", who);
  if (new_stride_n < shape->head_dim || (new_stride_n & 7) || new_stride_h < 0 || (new_stride_h & 7))
    return fail(FOCUS_EINVAL, "%s: strides of the new states invalid or not multiples of 8", who);
  if (!aligned16(K_cache) || !aligned16(V_cache) || !aligned16(K_new) || !aligned16(V_new) || !aligned16(kbar))
    return fail(FOCUS_EINVAL, "%s: pointers must be 16-byte aligned", who);
  if (K_cache == K_new || V_cache == V_new) return fail(FOCUS_EINVAL, "%s: the new states must not alias the cache", who);
  if (shape->n_heads > 65535) return fail(FOCUS_EUNSUPPORTED, "%s: more than 65535 heads", who);
  return FOCUS_OK;
}

int focus_refresh_attn(const void* Q, const void* K, const void* V, const focus_shape* shape, void* out, float* lse,
                       void* stream) {
  if (int rc = check_shape(shape, true, true, true, true)) return rc;
  if (int rc = check_refresh_attn("focus_refresh_attn", Q, K, V, shape, out, shape->k_stride_n, shape->v_stride_n)) return rc;
  hipError_t e = launch_refresh_attn(Q, K, V, *shape, out, lse, static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return launch_fail("focus_refresh_attn", e);
  return FOCUS_OK;
}

int focus_block_entry(void* K_cache, void* V_cache, const focus_shape* shape, const void* Q, const void* K_new, const void* V_new,
                      int64_t new_stride_h, int64_t new_stride_n, float* kbar, void* out, float* lse, void* stream) {
  if (int rc = check_shape(shape, true, true, true, true)) return rc;
  if (int rc = check_cache_refresh("focus_block_entry", K_cache, V_cache, shape, K_new, V_new, new_stride_h, new_stride_n, kbar)) return rc;
  if (int rc = check_refresh_attn("focus_block_entry", Q, K_new, V_new, shape, out, new_stride_n, new_stride_n)) return rc;
  const CacheRefresh copy = cache_refresh_args(K_cache, V_cache, *shape, K_new, V_new, new_stride_h, new_stride_n, kbar);
  hipError_t e = launch_refresh_attn(Q, K_new, V_new, *shape, out, lse, static_cast<hipStream_t>(stream), &copy);
  if (e != hipSuccess) return launch_fail("focus_block_entry", e);
  return FOCUS_OK;
}

int focus_token_confidence(const void* logits, int64_t row_stride, const uint8_t* masked, int32_t n_rows, int32_t vocab,
                           int32_t* tokens, float* conf, void* workspace, size_t ws_bytes, void* stream) {
  if (!logits || !tokens || !conf) return fail(FOCUS_EINVAL, "focus_token_confidence: NULL pointer");
  if (n_rows < 1 || n_rows > 65535) return fail(FOCUS_EINVAL, "focus_token_confidence: n_rows=%d not in [1, 65535]", n_rows);
  if (vocab < 1) return fail(FOCUS_EINVAL, "focus_token_confidence: vocab=%d", vocab);
  if (row_stride < vocab || (row_stride & 7) || !aligned16(logits))
    return fail(FOCUS_EINVAL, "focus_token_confidence: rows must be 16-byte aligned (row_stride a multiple of 8, >= vocab)");
  const size_t need = token_confidence_workspace(n_rows, vocab);
  if (need > 0 && (!workspace || ws_bytes < need || !aligned16(workspace)))
    return fail(FOCUS_EWORKSPACE, "focus_token_confidence: workspace needs %zu bytes, 16-byte aligned", need);
  hipError_t e = launch_token_confidence(logits, row_stride, masked, n_rows, vocab, tokens, conf, workspace,
                                         static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return launch_fail("focus_token_confidence", e);
  return FOCUS_OK;
}

int focus_cache_update(void* K_cache, void* V_cache, const focus_shape* shape, const void* K_new, const void* V_new,
                       int64_t new_stride_h, int64_t new_stride_n, const int32_t* active_idx, const int32_t* counts,
                       int32_t max_active, int32_t row_base, void* stream) {
  if (int rc = check_cache_update("focus_cache_update", K_cache, V_cache, shape, K_new, V_new, new_stride_h, new_stride_n, active_idx, max_active)) return rc;
  const CacheUpdate u = cache_update_args(K_cache, V_cache, *shape, K_new, V_new, new_stride_h, new_stride_n, active_idx, counts, max_active, row_base);
  hipError_t e = launch_cache_update(u, shape->head_dim, static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return launch_fail("focus_cache_update", e);
  return FOCUS_OK;
}

int focus_update_sparse_layer(void* K_cache, void* V_cache, const void* K_new, const void* V_new, int64_t new_stride_h, int64_t new_stride_n,
                              int32_t row_base, const void* Q, const int32_t* focus_idx, const int32_t* active_idx, const int32_t* counts,
                              int32_t n_focus_max, int32_t max_active, const float* kbar, const focus_shape* shape, int32_t n_keep,
                              const int32_t* sink_idx, int32_t n_sink, float* scores, int32_t* kept_blocks, void* out, float* lse,
                              void* workspace, size_t ws_bytes, void* stream) {
  if (int rc = check_cache_update("focus_update_sparse_layer", K_cache, V_cache, shape, K_new, V_new, new_stride_h, new_stride_n, active_idx, max_active)) return rc;
  const CacheUpdate u = cache_update_args(K_cache, V_cache, *shape, K_new, V_new, new_stride_h, new_stride_n, active_idx, counts, max_active, row_base);
  return sparse_layer_impl("focus_update_sparse_layer", Q, focus_idx, active_idx, counts, n_focus_max, max_active, K_cache, V_cache, kbar, shape,
                           n_keep, sink_idx, n_sink, scores, kept_blocks, out, lse, workspace, ws_bytes, false, stream, &u);
}

int focus_cache_refresh(void* K_cache, void* V_cache, const focus_shape* shape, const void* K_new, const void* V_new,
                        int64_t new_stride_h, int64_t new_stride_n, float* kbar, void* stream) {
  if (int rc = check_shape(shape, false, true, true, false)) return rc;
  if (int rc = check_cache_refresh("focus_cache_refresh", K_cache, V_cache, shape, K_new, V_new, new_stride_h, new_stride_n, kbar)) return rc;
  const CacheRefresh p = cache_refresh_args(K_cache, V_cache, *shape, K_new, V_new, new_stride_h, new_stride_n, kbar);
  hipError_t e = launch_cache_refresh(p, shape->head_dim, static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return launch_fail("focus_cache_refresh", e);
  return FOCUS_OK;
}

int focus_probe_layer(const void* Q, const int32_t* active_idx, const int32_t* counts, int32_t max_active, const void* K,
                      const void* V, const focus_shape* shape, int32_t n_sink, void* out, float* lse, float* col_mass,
                      int32_t* sink_idx, void* workspace, size_t ws_bytes, void* stream) {
  if (int rc = check_shape(shape, true, true, true, true)) return rc;
  if (!Q || !active_idx || !K || !V || !out) return fail(FOCUS_EINVAL, "focus_probe_layer: NULL pointer");
  if (max_active < 1 || max_active > shape->n_gen) return fail(FOCUS_EINVAL, "focus_probe_layer: max_active=%d not in [1, n_gen]", max_active);
  if (n_sink < 0 || n_sink > shape->n_ctx) return fail(FOCUS_EINVAL, "focus_probe_layer: n_sink=%d not in [0, n_ctx]", n_sink);
  if (n_sink > 0 && !sink_idx) return fail(FOCUS_EINVAL, "focus_probe_layer: sink_idx is NULL");
  if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(out))
    return fail(FOCUS_EINVAL, "focus_probe_layer: pointers must be 16-byte aligned");
  const SplitPlan pa = plan_attention_dense(*shape, max_active);
  const SplitPlan pl = plan_logits(*shape, max_active);
  const ProbeWs w = ws_probe_layer(*shape, pa, pl);
  if (!workspace || ws_bytes < w.total || !aligned16(workspace))
    return fail(FOCUS_EWORKSPACE, "focus_probe_layer: workspace needs %zu bytes, 16-byte aligned", w.total);
  hipStream_t st = static_cast<hipStream_t>(stream);
  char* ws = static_cast<char*>(workspace);
  float* lse2 = reinterpret_cast<float*>(ws + w.lse2);
  float* scratch = reinterpret_cast<float*>(ws + w.scratch);
  float* S = col_mass ? col_mass : reinterpret_cast<float*>(ws + w.col_mass);
  const bool two_pass = sinks_two_pass(pa);
  // dense attention of the active queries over all keys; with at most 16 queries its QK^T products are kept
  DenseProbe probe;
  probe.logits_out = two_pass ? nullptr : scratch;
  probe.lse2_out = lse2;
  hipError_t e = launch_sparse_attn(Q, active_idx, counts, max_active, K, V, *shape, nullptr, 0, nullptr, 0, pa, out, lse,
                                    reinterpret_cast<float*>(ws + w.part_o), reinterpret_cast<float*>(ws + w.part_ml), nullptr,
                                    st, &probe);
  if (e != hipSuccess) return launch_fail("focus_probe_layer(attention)", e);
  if (two_pass) {  // more queries: one more pass over K turns the known row log-sum-exps into column sums
    e = launch_qk_logits(Q, active_idx, counts, max_active, K, *shape, pl, 2, nullptr, nullptr, lse2, scratch, st);
    if (e != hipSuccess) return launch_fail("focus_probe_layer(column sums)", e);
  }
  if (int rc = column_mass_and_sinks("focus_probe_layer", scratch, two_pass, lse2, 0, nullptr, counts, max_active, pl.q_groups, *shape, n_sink, S,
                                     ws + w.cand, sink_idx, st))
    return rc;
  return FOCUS_OK;
}

int focus_sparse_attn(const void* Q, const int32_t* active_idx, const int32_t* counts, int32_t max_active, const void* K,
                      const void* V, const focus_shape* shape, const int32_t* kept_blocks, int32_t n_keep,
                      const int32_t* sink_idx, int32_t n_sink, void* out, float* lse, void* workspace, size_t ws_bytes,
                      void* stream) {
  if (int rc = check_shape(shape, true, true, true, true)) return rc;
  if (!Q || !active_idx || !K || !V || !out) return fail(FOCUS_EINVAL, "focus_sparse_attn: NULL pointer");
  const int n_b = ceil_div(shape->n_ctx, shape->block);
  if (max_active < 1 || max_active > shape->n_gen) return fail(FOCUS_EINVAL, "focus_sparse_attn: max_active=%d not in [1, n_gen]", max_active);
  if (n_keep < 0 || n_keep > n_b) return fail(FOCUS_EINVAL, "focus_sparse_attn: n_keep=%d not in [0, n_b=%d]", n_keep, n_b);
  if (n_sink < 0 || n_sink > shape->n_ctx) return fail(FOCUS_EINVAL, "focus_sparse_attn: n_sink=%d not in [0, n_ctx]", n_sink);
  if ((n_keep > 0 && !kept_blocks) || (n_sink > 0 && !sink_idx)) return fail(FOCUS_EINVAL, "focus_sparse_attn: index array is NULL");
  if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(out))
    return fail(FOCUS_EINVAL, "focus_sparse_attn: pointers must be 16-byte aligned");
  SplitPlan p = plan_attention(*shape, max_active, n_keep, n_sink);
  AttnWs w = ws_attn(*shape, p);
  if (!workspace || ws_bytes < w.total) w = ws_attn(*shape, p = plan_attention(*shape, max_active, n_keep, n_sink, true));
  if (p.n_split > 1 && (!workspace || ws_bytes < w.total || !aligned16(workspace)))
    return fail(FOCUS_EWORKSPACE, "focus_sparse_attn: workspace needs %zu bytes, 16-byte aligned", w.total);
  char* ws = static_cast<char*>(workspace);
  hipError_t e = launch_sparse_attn(Q, active_idx, counts, max_active, K, V, *shape, kept_blocks, n_keep, sink_idx, n_sink, p,
                                    out, lse, ws ? reinterpret_cast<float*>(ws + w.part_o) : nullptr,
                                    ws ? reinterpret_cast<float*>(ws + w.part_ml) : nullptr, nullptr,
                                    static_cast<hipStream_t>(stream));
  if (e != hipSuccess) return launch_fail("focus_sparse_attn", e);
  return FOCUS_OK;
}

int focus_sparse_layer(const void* Q, const int32_t* focus_idx, const int32_t* active_idx, const int32_t* counts,
                       int32_t n_focus_max, int32_t max_active, const void* K, const void* V, const float* kbar,
                       const focus_shape* shape, int32_t n_keep, const int32_t* sink_idx, int32_t n_sink, float* scores,
                       int32_t* kept_blocks, void* out, float* lse, void* workspace, size_t ws_bytes, void* stream) {
  return sparse_layer_impl("focus_sparse_layer", Q, focus_idx, active_idx, counts, n_focus_max, max_active, K, V, kbar, shape,
                           n_keep, sink_idx, n_sink, scores, kept_blocks, out, lse, workspace, ws_bytes, false, stream);
}

int focus_sparse_layer_static(const void* Q, const int32_t* focus_idx, const int32_t* active_idx, const int32_t* counts,
                              int32_t n_focus_max, int32_t max_active, const void* K, const void* V, const float* kbar,
                              const focus_shape* shape, int32_t n_keep, const int32_t* sink_idx, int32_t n_sink,
                              float* scores, int32_t* kept_blocks, void* out, float* lse, void* stream) {
  return sparse_layer_impl("focus_sparse_layer_static", Q, focus_idx, active_idx, counts, n_focus_max, max_active, K, V, kbar,
                           shape, n_keep, sink_idx, n_sink, scores, kept_blocks, out, lse, nullptr, 0, true, stream);
}

}  // extern "C"
