// The MFMA kernels (64-lane wavefronts):
//
//   sparse_attn_kernel   Eq. 8 + Eq. 9: gathers the kept blocks, the sinks and the response rows of K / V and
//                        runs a split-KV online-softmax attention of up to 16 active queries over them
//                        (v_mfma_f32_16x16x32_bf16).  The same kernel with every row kept is the dense layer (probe
//                        layer, dense comparison).
//   wide_attn_kernel     the same for more than 16 queries (v_mfma_f32_32x32x16_bf16; described where it is defined).
//   attn_combine_kernel, attn_combine_few_kernel   merge the key splits of the two kernels above.
//   refresh_attn_kernel  block entry (Alg. 1): dense attention of EVERY position over every key, the one MFMA-bound
//                        launch of the method (v_mfma_f32_32x32x16_bf16; described where it is defined).
//   refresh_tail_kernel  the query tiles the former leaves over, with the layer's cache refresh beside them.
//   qk_logits_kernel     Eq. 6, up to 16 active queries: their scaled logits against every key of the probe layer, written
//                        out, with the per-split row maxima / sums of the softmax normaliser (v_mfma_f32_16x16x32_bf16).
//   wide_logits_kernel   the same for more than 16 queries, in two passes over K (v_mfma_f32_32x32x16_bf16): the normalisers,
//                        then the probabilities summed over the queries.
//
// Work decomposition.  The key axis of one head is cut into sub-tiles of 32 rows, staged in LDS with an XOR
// swizzle (applied on the global side of the load) so that the operand reads are conflict free.  The rows go from HBM
// straight into a slot of LDS (global_load_lds_dwordx4: no staging registers, no ds_write; refresh_attn_kernel alone goes
// through registers).  With up to 32 queries in a group a wavefront owns a sub-tile from the memory request to the MFMAs,
// wavefronts never wait for each other inside the key loop and meet once, at the end, to merge their softmax states.
//
// MFMA layout used (16x16x32, D[i][j] += sum_k A[i][k] B[k][j]; lane = 16*g + c):
//   A operand: lane holds A[i = c][k = 8g .. 8g+7];  B operand: lane holds B[k = 8g .. 8g+7][j = c];
//   D: lane holds D[i = 4g + r][j = c], r = 0..3.
// Logits are produced transposed, S^T[key][query] = K_tile . Q^T, so that every lane keeps the values of ONE
// query (j = c): row maxima, sums and rescale factors are lane-local up to two lane swaps, and the
// exponentiated values already sit in B-operand layout for the second product O^T[dcol][query] = V^T . P^T,
// where the contraction slot (g, e) stands for key 16*(e/4) + 4g + (e%4) of the sub-tile on both operands.
// The V^T operand is read from the row-major staged tile with the transposing LDS read ds_read_b64_tr_b16.
#include <algorithm>
#include <cfloat>
#include <cstdlib>
#include <type_traits>
#include <utility>

#include "focus_cache.h"
#include "focus_common.h"
#include "focus_kernels.h"
#include "focus_topk.h"

namespace focus {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

template <int D>
struct Geo {
  static constexpr int kChunks = D / 8;               // 16-byte chunks per row
  static constexpr int kRowsPerLoad = 64 / kChunks;   // rows covered by one wave-wide 16-byte load
  static constexpr int kLoads = kSubTile / kRowsPerLoad;
  static constexpr int kKSteps = D / 32;              // MFMA k-steps of the QK^T product
  static constexpr int kColTiles = D / 16;            // 16-wide d tiles of the PV product
  static constexpr int kRowBytes = D * 2;
  static constexpr int kStageBytes = kSubTile * kRowBytes;  // one staged K (or V) sub-tile
};

// byte offset of 16-byte chunk `chunk` of staged row `row`: position chunk ^ (row mod chunks-per-row)
template <int D>
__device__ __forceinline__ int stage_off(int row, int chunk) {
  return row * Geo<D>::kRowBytes + ((chunk ^ (row & (Geo<D>::kChunks - 1))) << 4);
}

// swizzle of a V stage that is read in transposed 32x32x16 operands (see read_v_operand32)
template <int D>
__device__ __forceinline__ int vstage_swz(int row) {
  return D == 128 ? (row & 3) << 2 : ((row >> 1) & 1) << 2;
}

// cache policy of the K/V row loads: non-temporal (every row is read once per launch)
constexpr int kStreamPolicy = 2;

// s_waitcnt vmcnt(0): every outstanding global load, LDS-direct ones included, has landed
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }
// s_waitcnt vmcnt(N): every global load and store but the N issued last has completed
template <int N>
__device__ __forceinline__ void wait_loads_but() {
  static_assert(N < 64, "six bits");
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
  __builtin_amdgcn_sched_barrier(0);
}
// s_waitcnt lgkmcnt(0): every LDS read of this wavefront has returned.  Placed before an LDS-direct load that
// overwrites a stage the wavefront has just read: that write-after-read order is not covered by vmcnt, and the fence
// keeps the compiler from moving the load above the wait.
__device__ __forceinline__ void wait_lds_reads() {
  __builtin_amdgcn_s_waitcnt(0xC07F);
  __builtin_amdgcn_sched_barrier(0);
}

// ---------------------------------------------------------------------------------------- sub-tiles
// Which rows of K/V a sub-tile covers.  Wave-uniform.
struct SubTile {
  int row0;        // first row when contiguous (kind 0), first sink entry when kind 1
  int kind;        // 0: contiguous rows row0 .. ; 1: scattered rows sink_idx[row0 + slot]
  uint32_t vmask;  // bit s set: slot s holds a key that takes part
  int sink_row;    // kind 1, per lane: the row that slot `lane` stages (lanes 0..31; see subtile_row)
};

__device__ __forceinline__ uint32_t low_mask(int n) { return n >= 32 ? 0xffffffffu : (n > 0 ? ((1u << n) - 1u) : 0u); }

// Locate sub-tile `st` of the attention key list: kept blocks first (n_keep * sub_per_block sub-tiles), then
// the response rows, then the sinks.  Block ids outside [0, n_b) are skipped.  The union of Eq. 8 is a set:
// a sink is dropped when it is outside the prompt, inside a kept block or listed earlier in sink_idx (the block
// list itself must not repeat a block).  For sink sub-tiles lane r < 32 owns slot r.  dense_rows > 0 replaces all of
// that by "all of the first dense_rows rows".
//   "inside a kept block": one look-up in `kept_bits` (bit b set <=> block b is kept; LDS, built by the workgroup)
//   when that is given, else the block list is scanned 64 entries per load.
//   "listed earlier": a strictly ascending list (what focus_find_sinks writes) cannot repeat an entry; `ascending`
//   says so (1 / 0, established once by the workgroup), or -1: not known, then a scan of 64 entries per step
//   establishes it here.  Only lists that are not ascending pay for the all-pairs comparison.
// A list of at most one sub-tile (n_sink <= 32) costs no memory access here: lane r < n_sink holds its entry r in `few_sinks`
// (-1 in the other lanes), requested at the start of the kernel.
constexpr int kBitmapBlocks = 8192;  // largest n_b for which workgroups keep a bitmap of the kept blocks
// A wave-uniform 4-byte read of global memory that no kernel writes while this one runs, issued as a scalar load: it
// returns through the scalar cache instead of queueing behind the wavefront's vector loads (which return in order), and
// a hit there is much quicker than a vector load's trip through L2.
__device__ __forceinline__ int32_t uniform_load(const int32_t* ptr) {
  typedef const __attribute__((address_space(4))) int32_t* cptr_t;
  return *(cptr_t)(uintptr_t)ptr;
}
__device__ __forceinline__ int32_t uniform_load(const uint16_t* ptr) { return *ptr; }  // (lists of 16 bits lie in LDS: KeptList)
// Sub-tile `st` of the sink list
template <class Id>
__device__ __forceinline__ SubTile locate_sinks(int st, int lane, int M, int B, const Id* __restrict__ kept_blocks, int n_keep,
                                                const int32_t* __restrict__ sink_idx, int n_sink, const uint32_t* kept_bits, int ascending,
                                                int few_sinks) {
  SubTile t;
  t.kind = 1;
  t.row0 = st * kSubTile;
  const int e = t.row0 + lane;
  const bool few = n_sink <= kSubTile;  // the list is one sub-tile, which the caller holds in registers
  const int mine = few ? few_sinks : ((lane < kSubTile && e < n_sink) ? sink_idx[e] : -1);
  const int n_slots = min(n_sink - t.row0, kSubTile);
  const bool in_prompt = mine >= 0 && mine < M;
  const int my_block = in_prompt ? mine / B : -1;
  uint32_t bad = 0u;
  if (kept_bits != nullptr) {
    const bool kept = my_block >= 0 && ((kept_bits[my_block >> 5] >> (my_block & 31)) & 1u);
    bad = (uint32_t)(__ballot(kept) & 0xffffffffull);
  } else {
    for (int j0 = 0; j0 < n_keep; j0 += kWave) {
      const int v = j0 + lane < n_keep ? kept_blocks[j0 + lane] : -2;
      for (int r = 0; r < n_slots; ++r) {
        const int sb = __builtin_amdgcn_readlane(my_block, r);
        if (__ballot(v == sb) != 0ull) bad |= 1u << r;
      }
    }
  }
  const int e_end = min(t.row0 + kSubTile, n_sink);
  if (few) {
    const int before = __shfl_up(mine, 1, kWave);
    ascending = 1;
    if (__ballot(lane > 0 && lane < n_sink && mine <= before) != 0ull) {
      for (int r = 1; r < n_slots; ++r)
        if (__ballot(mine == __builtin_amdgcn_readlane(mine, r) && lane < r) != 0ull) bad |= 1u << r;
    }
  }
  if (ascending < 0) {  // sink_idx[0 .. e_end) strictly ascending?
    ascending = 1;
    for (int j0 = 0; j0 + 1 < e_end; j0 += kWave) {
      const int idx = j0 + lane;
      const bool pair = idx + 1 < e_end;
      const int a = pair ? sink_idx[idx] : 0, b = pair ? sink_idx[idx + 1] : 1;
      if (__ballot(b <= a) != 0ull) ascending = 0;
    }
  }
  if (ascending == 0) {
    for (int j0 = 0; j0 < e_end; j0 += kWave) {
      const int idx = j0 + lane;
      const int v = idx < e_end ? sink_idx[idx] : -2;
      for (int r = 0; r < n_slots; ++r) {
        const int s = __builtin_amdgcn_readlane(mine, r);
        if (__ballot(v == s && idx < t.row0 + r) != 0ull) bad |= 1u << r;
      }
    }
  }
  t.vmask = (uint32_t)(__ballot(in_prompt) & 0xffffffffull) & ~bad;
  // a slot whose sink was dropped stages the sub-tile's first valid sink instead
  const int fallback = __shfl(mine, t.vmask != 0u ? __builtin_ctz(t.vmask) : 0, kWave);
  t.sink_row = ((t.vmask >> (lane & 31)) & 1u) ? mine : fallback;
  return t;
}

template <class Id>
__device__ __forceinline__ SubTile locate_subtile(int st, int lane, int M, int N, int B, int n_b, int sub_per_block,
                                                  const Id* __restrict__ kept_blocks, int n_keep,
                                                  const int32_t* __restrict__ sink_idx, int n_sink,
                                                  const uint32_t* kept_bits = nullptr, int ascending = -1,
                                                  int dense_rows = 0, bool blocks_in_lds = false, int few_sinks = -1) {
  SubTile t;
  t.kind = 0;
  t.row0 = 0;
  t.vmask = 0u;
  t.sink_row = 0;
  if (dense_rows > 0) {  // every key row takes part (dense layers): sub-tile st is rows [32 st, 32 st + 32)
    t.row0 = st * kSubTile;
    t.vmask = low_mask(min(dense_rows - t.row0, kSubTile));
    return t;
  }
  const int n_blk_sub = n_keep * sub_per_block;
  const int n_resp_sub = (N + kSubTile - 1) / kSubTile;
  if (st < n_blk_sub) {
    const int slot = st / sub_per_block, sub = st % sub_per_block;
    const int b = blocks_in_lds ? kept_blocks[slot] : uniform_load(kept_blocks + slot);
    if (b < 0 || b >= n_b) return t;
    const int first = b * B + sub * kSubTile;
    const int end = min(min((b + 1) * B, M), first + kSubTile);
    t.row0 = first;
    t.vmask = low_mask(end - first);
    return t;
  }
  st -= n_blk_sub;
  if (st < n_resp_sub) {
    const int first = M + st * kSubTile;
    t.row0 = first;
    t.vmask = low_mask(min(M + N - first, kSubTile));
    return t;
  }
  return locate_sinks(st - n_resp_sub, lane, M, B, kept_blocks, n_keep, sink_idx, n_sink, kept_bits, ascending, few_sinks);
}

// Row of K/V that staged slot `slot` of sub-tile t reads.  Every slot reads a row of the key set, also the slots that
// hold no key (they are masked out of the softmax, but their V row still meets a zero probability in the PV product,
// and 0 x inf would poison the output): past the end of a contiguous tile the tile's last valid row, for a dropped
// sink the sub-tile's first valid sink.  `last` = highest valid slot.  Requires t.vmask != 0.
__device__ __forceinline__ int subtile_row(const SubTile& t, int slot, int last) {
  if (t.kind == 0) return t.row0 + min(slot, last);
  return __shfl(t.sink_row, slot, kWave);  // wave-uniform branch; the list was read once, when the sub-tile was located
}

// HBM -> LDS for one 32-row sub-tile of a [rows, D] bf16 matrix.  Lane l of load i supplies the 16 bytes that
// land at stage + 1024 i + 16 l, i.e. position (l mod chunks) of staged row i * rows_per_load + l / chunks; with
// the swizzle that position holds logical chunk (l mod chunks) ^ (row mod chunks).  No load is predicated: a
// slot that holds no key reads another row of the key set instead (subtile_row) and is masked out of the softmax.
// Requires t.vmask != 0.
// The loads [first, first + NL) of a sub-tile, straight into LDS (all of them, or a wavefront's share when several
// wavefronts stage one sub-tile).  A whole contiguous sub-tile — the common case — takes the short way: one scalar base
// address per sub-tile plus per-lane byte offsets that depend on the lane and the load only (the compiler keeps them
// across a key loop), so a request costs no per-lane address arithmetic; ragged and scattered sub-tiles work out a row
// per lane and load.
// VSWZ: the rows are swizzled for the transposed reads of the 32x32 tiles (vstage_swz) instead of for row reads.
template <int D, int NL, bool VSWZ = false, int POLICY = kStreamPolicy>
__device__ __forceinline__ void issue_subtile_part(const uint16_t* __restrict__ base, int64_t sn, const SubTile& t, char* stage,
                                                   int lane, int first) {
  using G = Geo<D>;
  typedef const __attribute__((address_space(1))) void* gptr_t;
  typedef __attribute__((address_space(3))) void* lptr_t;
  const int sub = lane / G::kChunks, pos = lane % G::kChunks;
  if (t.kind == 0 && t.vmask == 0xffffffffu && sn < (int64_t(1) << 26)) {  // wave-uniform; 31 rows of the stride fit 32 bits
    // load i starts rows_per_load * i rows further down (scalar), so the per-lane offset depends on i only through the
    // swizzle: at most four different ones per matrix
    const char* tile = reinterpret_cast<const char*>(base + (int64_t)__builtin_amdgcn_readfirstlane(t.row0) * sn);
    const uint32_t lane_row = (uint32_t)sub * (uint32_t)(sn * 2);  // a sub-tile spans < 4 GB
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int slot = (first + i) * G::kRowsPerLoad + sub;
      const int chunk = pos ^ (VSWZ ? vstage_swz<D>(slot) : (slot & (G::kChunks - 1)));
      const char* rows = tile + (int64_t)((first + i) * G::kRowsPerLoad) * (sn * 2);
      __builtin_amdgcn_global_load_lds((gptr_t)(rows + (lane_row + (uint32_t)(chunk * 16))), (lptr_t)(stage + (first + i) * 1024), 16, 0,
                                       POLICY);
    }
    return;
  }
  const int last = 31 - __builtin_clz(t.vmask);
  int lane_now = lane;  // ragged and scattered sub-tiles are rare: nothing of theirs is kept in registers across a key loop
  asm volatile("" : "+v"(lane_now));
  const int sub_now = lane_now / G::kChunks, pos_now = lane_now % G::kChunks;
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int slot = (first + i) * G::kRowsPerLoad + sub_now;
    const int row = subtile_row(t, slot, last);
    const int chunk = pos_now ^ (VSWZ ? vstage_swz<D>(slot) : (slot & (G::kChunks - 1)));
    const uint16_t* src = base + (int64_t)row * sn + chunk * 8;
    __builtin_amdgcn_global_load_lds((gptr_t)src, (lptr_t)(stage + (first + i) * 1024), 16, 0, POLICY);
  }
}
template <int D, bool VSWZ = false, int POLICY = kStreamPolicy>
__device__ __forceinline__ void issue_subtile(const uint16_t* __restrict__ base, int64_t sn, const SubTile& t, char* stage,
                                              int lane) {
  issue_subtile_part<D, Geo<D>::kLoads, VSWZ, POLICY>(base, sn, t, stage, lane, 0);
}

typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------------------- queries
// Row of Q for query slot q0 + (lane % 16), or -1.  The index is fetched for every slot below max_active
// without waiting for the device-side count; slots at or past the count are zeroed afterwards (mask_q_tile),
// which keeps the count out of the load chain.
__device__ __forceinline__ int fetch_q_row(const int32_t* __restrict__ active_idx, int q0, int max_active, int n_gen,
                                           int lane) {
  const int a = q0 + (lane & 15);
  int row = -1;
  if (a < max_active) row = active_idx[a];
  return (row >= 0 && row < n_gen) ? row : -1;
}
// Q rows of one 16-query tile in B-operand layout: lane (c, g) holds Q[query c][32*kk + 8g .. +7].
template <int D>
__device__ __forceinline__ void load_q_tile(bf16x8 (&q)[Geo<D>::kKSteps], const uint16_t* __restrict__ Qh, int64_t qsn,
                                            int row, int lane) {
  const int g = lane >> 4;
  const uint16_t* src = Qh + (int64_t)max(row, 0) * qsn + g * 8;
#pragma unroll
  for (int kk = 0; kk < Geo<D>::kKSteps; ++kk) {
    const uint4 v = *reinterpret_cast<const uint4*>(src + kk * 32);
    q[kk] = as_bf16x8(row >= 0 ? v : make_uint4(0u, 0u, 0u, 0u));
  }
}
template <int D>
__device__ __forceinline__ void mask_q_tile(bf16x8 (&q)[Geo<D>::kKSteps], int q0, int n_act, int lane) {
  if (q0 + (lane & 15) >= n_act) {
#pragma unroll
    for (int kk = 0; kk < Geo<D>::kKSteps; ++kk) q[kk] = as_bf16x8(make_uint4(0u, 0u, 0u, 0u));
  }
}

// ---------------------------------------------------------------------------------------- tile math
// S^T tiles of one staged K sub-tile: acc[kt][r] = logit of key 16kt + 4g + r.
template <int D>
__device__ __forceinline__ void qk_subtile(floatx4 (&acc)[2], const char* stageK, const bf16x8 (&q)[Geo<D>::kKSteps], int lane) {
  const int c = lane & 15, g = lane >> 4;
#pragma unroll
  for (int kt = 0; kt < 2; ++kt) {
    acc[kt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int kk = 0; kk < Geo<D>::kKSteps; ++kk) {
      const bf16x8 a = as_bf16x8(*reinterpret_cast<const uint4*>(stageK + stage_off<D>(kt * 16 + c, kk * 4 + g)));
      acc[kt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, q[kk], acc[kt], 0, 0, 0);
    }
  }
}

// eight fp32 -> eight bf16 (round to nearest even) with v_cvt_pk_bf16_f32
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t cvt_pk_bf16(float lo, float hi) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((floatx2){lo, hi}, bf16x2));
}
// sum + lo + hi of a packed pair, in fp32
__device__ __forceinline__ float add_bf16_pair(float sum, uint32_t pair) {
  const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pair), ones, sum, false);
}
__device__ __forceinline__ bf16x8 pack_bf16x8(const float (&v)[8]) {
  return as_bf16x8(make_uint4(cvt_pk_bf16(v[0], v[1]), cvt_pk_bf16(v[2], v[3]), cvt_pk_bf16(v[4], v[5]), cvt_pk_bf16(v[6], v[7])));
}

// A operand of the PV product for d-column tile `ct`: lane (c, g) needs V[key slot (g, e)][16 ct + c], e = 0..7,
// i.e. eight different rows at one column of the row-major staged tile.  ds_read_b64_tr_b16 does that
// transposition in the LDS unit: within a block of 16 lanes, lane i receives element (i % 4) of the 8-byte
// groups addressed by lanes i/4, i/4 + 4, i/4 + 8, i/4 + 12.  Lane s therefore points at row 4g + s/4 (first
// read) or 16 + 4g + s/4 (second read), columns 16 ct + 4 (s % 4) .. + 3.
typedef short shortx4 __attribute__((ext_vector_type(4)));
template <int D>
__device__ __forceinline__ bf16x8 read_v_operand(const char* stageV, int ct, int lane) {
  const int s = lane & 15, g = lane >> 4;
  const int row = 4 * g + (s >> 2);
  const int col = 16 * ct + 4 * (s & 3);
  const int off0 = stage_off<D>(row, col >> 3) + (col & 7) * 2;
  const int off1 = stage_off<D>(row + 16, col >> 3) + (col & 7) * 2;
  typedef shortx4 __attribute__((address_space(3))) * lds_ptr;
  const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(stageV + off0));
  const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(stageV + off1));
  struct { shortx4 a, b; } both = {lo, hi};
  return __builtin_bit_cast(bf16x8, both);
}

// All K (V) operands of a staged sub-tile into registers, complete on return.  Key loops that request the next K rows while the V
// rows of this sub-tile are still under way need the reads outside the compiler's sight: it would wait for every outstanding
// LDS-direct load in front of them.  The callers wait for the rows (wait_loads_but).  Stages are aligned to 256 bytes, so that the
// swizzle of a chunk is an exclusive or of the address.
__device__ __forceinline__ uint32_t lds_address(const char* p) {
  typedef const __attribute__((address_space(3))) char* lds_ptr;
  return (uint32_t)(uintptr_t)(lds_ptr)p;
}
template <int D>
__device__ __forceinline__ void read_k_operands16(bf16x8 (&k)[2][D / 32], const char* stageK, int lane) {
  const uint32_t a = lds_address(stageK) + stage_off<D>(lane & 15, lane >> 4);  // chunk 4 kk + g, row 16 kt + c
  if constexpr (D == 128) {
    asm volatile(
        "ds_read_b128 %0, %8\n\tds_read_b128 %1, %9\n\tds_read_b128 %2, %10\n\tds_read_b128 %3, %11\n\t"
        "ds_read_b128 %4, %8 offset:4096\n\tds_read_b128 %5, %9 offset:4096\n\tds_read_b128 %6, %10 offset:4096\n\t"
        "ds_read_b128 %7, %11 offset:4096\n\ts_waitcnt lgkmcnt(0)"
        : "=&v"(k[0][0]), "=&v"(k[0][1]), "=&v"(k[0][2]), "=&v"(k[0][3]), "=&v"(k[1][0]), "=&v"(k[1][1]), "=&v"(k[1][2]), "=&v"(k[1][3])
        : "v"(a), "v"(a ^ 64u), "v"(a ^ 128u), "v"(a ^ 192u)
        : "memory");
  } else {
    asm volatile(
        "ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %4 offset:2048\n\tds_read_b128 %3, %5 offset:2048\n\t"
        "s_waitcnt lgkmcnt(0)"
        : "=&v"(k[0][0]), "=&v"(k[0][1]), "=&v"(k[1][0]), "=&v"(k[1][1])
        : "v"(a), "v"(a ^ 64u)
        : "memory");
  }
}
template <int D>
__device__ __forceinline__ void read_v_operands16(bf16x8 (&v)[D / 16], const char* stageV, int lane) {
  const int s = lane & 15, g = lane >> 4, col = 4 * (s & 3);
  const uint32_t a = lds_address(stageV) + stage_off<D>(4 * g + (s >> 2), col >> 3) + (col & 7) * 2;  // column tile ct: chunk 2 ct further
  shortx4 r[D / 16][2];
  if constexpr (D == 128) {
    asm volatile(
        "ds_read_b64_tr_b16 %0, %16\n\tds_read_b64_tr_b16 %1, %16 offset:4096\n\t"
        "ds_read_b64_tr_b16 %2, %17\n\tds_read_b64_tr_b16 %3, %17 offset:4096\n\t"
        "ds_read_b64_tr_b16 %4, %18\n\tds_read_b64_tr_b16 %5, %18 offset:4096\n\t"
        "ds_read_b64_tr_b16 %6, %19\n\tds_read_b64_tr_b16 %7, %19 offset:4096\n\t"
        "ds_read_b64_tr_b16 %8, %20\n\tds_read_b64_tr_b16 %9, %20 offset:4096\n\t"
        "ds_read_b64_tr_b16 %10, %21\n\tds_read_b64_tr_b16 %11, %21 offset:4096\n\t"
        "ds_read_b64_tr_b16 %12, %22\n\tds_read_b64_tr_b16 %13, %22 offset:4096\n\t"
        "ds_read_b64_tr_b16 %14, %23\n\tds_read_b64_tr_b16 %15, %23 offset:4096\n\ts_waitcnt lgkmcnt(0)"
        : "=&v"(r[0][0]), "=&v"(r[0][1]), "=&v"(r[1][0]), "=&v"(r[1][1]), "=&v"(r[2][0]), "=&v"(r[2][1]), "=&v"(r[3][0]), "=&v"(r[3][1]),
          "=&v"(r[4][0]), "=&v"(r[4][1]), "=&v"(r[5][0]), "=&v"(r[5][1]), "=&v"(r[6][0]), "=&v"(r[6][1]), "=&v"(r[7][0]), "=&v"(r[7][1])
        : "v"(a), "v"(a ^ 32u), "v"(a ^ 64u), "v"(a ^ 96u), "v"(a ^ 128u), "v"(a ^ 160u), "v"(a ^ 192u), "v"(a ^ 224u)
        : "memory");
  } else {
    asm volatile(
        "ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %8 offset:2048\n\t"
        "ds_read_b64_tr_b16 %2, %9\n\tds_read_b64_tr_b16 %3, %9 offset:2048\n\t"
        "ds_read_b64_tr_b16 %4, %10\n\tds_read_b64_tr_b16 %5, %10 offset:2048\n\t"
        "ds_read_b64_tr_b16 %6, %11\n\tds_read_b64_tr_b16 %7, %11 offset:2048\n\ts_waitcnt lgkmcnt(0)"
        : "=&v"(r[0][0]), "=&v"(r[0][1]), "=&v"(r[1][0]), "=&v"(r[1][1]), "=&v"(r[2][0]), "=&v"(r[2][1]), "=&v"(r[3][0]), "=&v"(r[3][1])
        : "v"(a), "v"(a ^ 32u), "v"(a ^ 64u), "v"(a ^ 96u)
        : "memory");
  }
#pragma unroll
  for (int ct = 0; ct < D / 16; ++ct) {
    struct { shortx4 a, b; } both = {r[ct][0], r[ct][1]};
    v[ct] = __builtin_bit_cast(bf16x8, both);
  }
}

typedef float floatx16 __attribute__((ext_vector_type(16)));
// A operand of O^T += V^T P^T (32x32x16) for d tile `dt` and k-step `ks`: lane (dcol = lane % 32, hh) needs
// V[16 ks + 8 (e / 4) + 4 hh + e % 4][32 dt + dcol], e = 0..7 — two transposed reads of four consecutive rows each.
// A V staged for the 32x32 tiles is only ever read this way — one instruction touches eight rows (four per half of the
// wavefront) and 64 bytes of each — so its rows are swizzled for that: rows that would fall on the same banks
// (consecutive rows at d = 128, every other row at d = 64) get different 64-byte segments.
template <int D>
__device__ __forceinline__ int vstage_off(int row, int chunk) {
  return row * Geo<D>::kRowBytes + ((chunk ^ vstage_swz<D>(row)) << 4);
}
template <int D>
__device__ __forceinline__ bf16x8 read_v_operand32(const char* stageV, int dt, int ks, int lane) {
  const int s = lane & 15, b = lane >> 4;
  const int row = 16 * ks + 4 * (b >> 1) + (s >> 2);
  const int col = 32 * dt + 16 * (b & 1) + 4 * (s & 3);
  const int off0 = vstage_off<D>(row, col >> 3) + (col & 7) * 2;
  const int off1 = vstage_off<D>(row + 8, col >> 3) + (col & 7) * 2;
  typedef shortx4 __attribute__((address_space(3))) * lds_ptr;
  const shortx4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(stageV + off0));
  const shortx4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(stageV + off1));
  struct { shortx4 a, b; } both = {lo, hi};
  return __builtin_bit_cast(bf16x8, both);
}

// Scaled logits of one 32-key sub-tile (contiguous rows row0 .., row0 a multiple of 32) against up to 16 queries, kept
// for the column-mass kernel in the layout [head][key quad][query][key within the quad] (fp32): a lane holds, per
// 16-key tile, the logits of ONE query for four consecutive keys — one 16-byte store — and the 64 lanes of a store
// instruction cover 1 KB of consecutive bytes (query fastest, then the four quads of the tile).  Quads that start at or
// past key L are not written; the padding keys of the last quad hold finite values nobody reads.  Neither are the slots of queries past
// the capacity n_q of the list, and the column-mass kernel does not fetch them: at eight queries half of the traffic beside K (32 heads, sink
// chain of 8192 keys 28.8 -> 26.7 us, 32 832 73.5 -> 67.1, 131 136 255 -> 232; probe layer of 32 832 128 -> 118; four queries take as
// long as eight, a line of 128 bytes; sixteen as before).  The device-side count would come too late for the second kernel's first loads.
// n_q >= 1, which the launchers check: a whole sub-tile is then kSpillStores store instructions, whatever the list, and the key loops count
// them among the requests under way.
constexpr int kSpillStores = 2;
__device__ __forceinline__ void spill_logits(float* __restrict__ logits, int h, int L, int n_q, int row0, const floatx4 (&acc)[2],
                                             float scale_log2, int lane) {
  const int c = lane & 15, g = lane >> 4;
  const int64_t n_quads = (L + 3) >> 2;
#pragma unroll
  for (int kt = 0; kt < kSpillStores; ++kt) {
    const int key0 = row0 + 16 * kt + 4 * g;
    if (key0 < L && c < n_q) {
      floatx4* dst = reinterpret_cast<floatx4*>(logits + (((int64_t)h * n_quads + (key0 >> 2)) * 16 + c) * 4);
      *dst = acc[kt] * scale_log2;
    }
  }
}

// One step of the base-2 online softmax for the 8 logits a lane holds of one query; returns the rescale factor
// of the running state and leaves exp2(scale * s - m) in ps.  The running maximum m is kept in the scaled domain;
// the scale (> 0) is applied to the raw maximum once and folded into the exponent's multiply-add for the rest.
// A sub-tile whose 32 slots all hold keys (the common case) skips the per-slot masking.
__device__ __forceinline__ float softmax_step(const floatx4 (&acc)[2], uint32_t vmask, int g, float scale_log2, float& m_run,
                                              float& l_run, float (&ps)[8]) {
  float s[8];
  float mx = -INFINITY;
  if (vmask == 0xffffffffu) {  // wave-uniform
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      s[e] = acc[e >> 2][e & 3];
      mx = fmaxf(mx, s[e]);
    }
  } else {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int slot = 16 * (e >> 2) + 4 * g + (e & 3);
      s[e] = ((vmask >> slot) & 1u) ? acc[e >> 2][e & 3] : -INFINITY;
      mx = fmaxf(mx, s[e]);
    }
  }
  mx = group_max(mx) * scale_log2;  // -inf stays -inf
  const float m_new = fmaxf(m_run, mx);
  const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
  const float alpha = __builtin_amdgcn_exp2f(m_run - m_use);
  float lsum = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    ps[e] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[e], scale_log2, -m_use));
    lsum += ps[e];
  }
  lsum = group_sum(lsum);
  l_run = l_run * alpha + lsum;
  m_run = m_new;
  return alpha;
}

// =====================================================================================================
// Sparse attention
// =====================================================================================================
struct AttnArgs {
  const uint16_t* Q;
  const uint16_t* K;
  const uint16_t* V;
  const int32_t* active_idx;
  const int32_t* counts;
  const int32_t* kept_blocks;
  const int32_t* sink_idx;
  uint16_t* out;
  float* lse;
  float* part_o;   // [H, q_pad, n_split, D]
  float* part_ml;  // [H, q_pad, n_split, 2]
  int64_t qsh, qsn, ksh, ksn, vsh, vsn, osh, osn;
  int H, M, N, B, n_b, n_gen, n_keep, n_sink, max_active;
  int sub_per_block, n_sub, n_split, q_pad, q_groups;
  float scale_log2;
  uint32_t head_turn;                // (2^32 - 1) / H      see SplitRounds
  int split_rounds, split_rounds_more;  // every split has so many rounds, the first so many splits one more
  // fused layer path only: partial relevances in, scores / kept blocks out
  // (where the kernel works the relevances out itself rel_part is the representative keys [H, n_b, D] and kept_blocks the focus rows' ids)
  const float* rel_part;  // [ceil(H / 4), n_b], or with rel_per_head [H, n_b]
  bool rel_per_head;
  float* scores_out;      // [n_b] or null
  int32_t* kept_out;      // [n_keep]
  int n_focus_max;
  // dense (probe) layer only
  int dense_rows;     // > 0: attend to all of the first dense_rows = M + N key rows, block and sink lists unused
  float* logits_out;  // [H, ceil(L / 4), 16, 4] scaled base-2 logits of the (at most 16) active queries (spill_logits), or null
  float* lse2_out;    // [H, q_pad] base-2 log-sum-exp per row (+inf for an empty row), or null
};

// |I_focus| and |I_active| as they lie in memory (or the capacities of the lists): scalar loads that a kernel requests at its start and
// waits for once its first vector loads are out (one that first looked whether its query group is past the count, and read the other
// count when the relevances had come, spent two memory round trips on it: layers of more than 16 queries 0.3 to 0.7 us).
struct Counts {
  int focus, active;
  __device__ __forceinline__ explicit Counts(const AttnArgs& p) : focus(p.n_focus_max), active(p.max_active) {
    if (p.counts) {
      focus = p.counts[0];
      active = p.counts[1];
    }
  }
  __device__ __forceinline__ int n_active(const AttnArgs& p) const { return min(max(active, 0), p.max_active); }
};

// The arguments that the first memory requests of an attention kernel need, once more as leading scalar parameters: those (14
// dwords) are in scalar registers when a wavefront starts (-amdgpu-kernarg-preload-count), while a member of AttnArgs is a load
// of its own in front of everything that depends on it.  H arrives negative where the partial relevances are per head.
#define ATTN_FIRST_PARAMS                                                                                                  \
  const float *rel_part, const int32_t *active_idx, const uint16_t *Q, const int32_t *counts, int n_b, int H, int max_active, \
      int n_gen, int n_split, int n_sub
#define ATTN_FIRST_NAMES rel_part, active_idx, Q, counts, n_b, H, max_active, n_gen, n_split, n_sub
// wide_attn_kernel: n_gen is needed later, the number of query groups at once
#define WIDE_FIRST_PARAMS                                                                                                     \
  const float *rel_part, const int32_t *active_idx, const uint16_t *Q, const int32_t *counts, int n_b, int H, int max_active, \
      int q_groups, int n_split, int n_sub
__device__ __forceinline__ AttnArgs with_first(AttnArgs p, ATTN_FIRST_PARAMS) {
  p.rel_part = rel_part;
  p.active_idx = active_idx;
  p.Q = Q;
  p.counts = counts;
  p.n_b = n_b;
  p.H = abs(H);
  p.rel_per_head = H < 0;
  p.max_active = max_active;
  p.n_gen = n_gen;
  p.n_split = n_split;
  p.n_sub = n_sub;
  return p;
}
#define WIDE_LAUNCH(kernel, grid, block, st, a)                                                                            \
  hipLaunchKernelGGL(kernel, grid, block, 0, st, (a).rel_part, (a).active_idx, (a).Q, (a).counts, (a).n_b, (a).rel_per_head ? -(a).H : (a).H, (a).max_active, \
                     (a).q_groups, (a).n_split, (a).n_sub, a)
#define ATTN_LAUNCH(kernel, grid, block, st, a)                                                                            \
  hipLaunchKernelGGL(kernel, grid, block, 0, st, (a).rel_part, (a).active_idx, (a).Q, (a).counts, (a).n_b, (a).rel_per_head ? -(a).H : (a).H, (a).max_active, \
                     (a).n_gen, (a).n_split, (a).n_sub, a)

// Where a workgroup that ranks the blocks itself keeps the list.  Up to 256 blocks: beside the ranking's scratch memory.  More: in 16 bits
// per block, in the place of the histograms, which everyone has read by then; beside them and in 32 bits a workgroup of
// sparse_attn_kernel<64, .> without a key loop took 43 620 bytes (up to 1024 blocks) and 47 716 (2048), and of the four that the plan
// of the key splits counts on per compute unit (kAttnGroupsSmall) three fitted (32 heads, d = 64, whole layer: 512 blocks, 97 sub-tiles
// 20.4 -> 16.5 us, 127 21.7 -> 18.1; 2048 blocks 27.9 -> 22.6, 29.3 -> 23.6).
template <bool FUSED, int BLOCKS>
struct KeptList {
  static constexpr bool kInScratch = FUSED && BLOCKS > 256;
  using Id = std::conditional_t<kInScratch, uint16_t, int32_t>;
  static constexpr int kEntriesBeside = FUSED && !kInScratch ? BLOCKS : 1;
  static_assert(!kInScratch || BLOCKS * sizeof(Id) <= sizeof(TopkShared::keys), "fits the histograms");
  static __device__ __forceinline__ Id* place(char* scratch, int32_t* beside) {
    if constexpr (kInScratch)
      return reinterpret_cast<Id*>(reinterpret_cast<TopkShared*>(scratch)->keys);
    else
      return beside;
  }
};

// What the attention kernels prepare before their first K/V request.
// R_b = (1 / (|I_focus| H)) sum_h qsum^h . kbar^h_b, then Top-C into kept_sh; the workgroup with `writer` set also writes scores
// and kept blocks out.  First use of `sm`.  Thread t of THREADS ranks the blocks t, t + THREADS, ...; n_b <= kFusedMaxBlocks.
// FirstParts holds the loads of the first NP parts (32 heads in groups of four are 8 parts), which the caller requests before it
// waits for anything.  BLOCKS: the most blocks of the variant, 256, kFusedManyBlocks or kFusedMaxBlocks.  Few blocks to keep of up to 256: the tournament of block_topk_small; else
// block_topk_planes.  Repeating it in every workgroup takes less time than the launch of a kernel that ranks the blocks once
// (sparse layer at 128K, 30 of 1024 blocks, 34.7 -> 29.0 us; half of 512 64-row blocks 63.2 -> 60.1).
template <int NP, int THREADS, int BLOCKS>
struct FirstParts {
  static constexpr int kPlanes = BLOCKS > 256 ? BLOCKS / THREADS : 1;
  float part[kPlanes][NP];
};
template <int NP, int THREADS, int BLOCKS>
__device__ __forceinline__ void first_partials(FirstParts<NP, THREADS, BLOCKS>& f, const AttnArgs& p, bool per_head) {
  const int last = (per_head ? p.H : (p.H + kRelGroup - 1) / kRelGroup) - 1;
#pragma unroll
  for (int l = 0; l < f.kPlanes; ++l) {
    const uint32_t b = min((int)threadIdx.x + l * THREADS, p.n_b - 1);  // n_b <= kFusedMaxBlocks: small offsets
#pragma unroll
    for (int i = 0; i < NP; ++i) f.part[l][i] = p.rel_part[(uint32_t)(min(i, last) * p.n_b) + b];
  }
  __builtin_amdgcn_sched_barrier(0);  // (the scheduler would move the wait for the row ids in front of these loads)
}
// The whole relevance in the attention kernel (relevance_in_attention): a wavefront takes one head and kInnerBlocks consecutive blocks, all
// of its representative keys requested before the focus rows, and the sums of the groups of four heads go to the thread that ranks the
// block, in the order of relevance_partial_kernel.
constexpr int kInnerBlocks = 16, kInnerGroups = 4;  // WAVES <= 16 heads
template <int D, int WAVES, int NP, int BLOCKS>
__device__ __forceinline__ void relevance_parts(FirstParts<NP, 64 * WAVES, BLOCKS>& f, const AttnArgs& p, int entry, int n_focus, float* dots,
                                                int wave, int lane) {
  constexpr int CPR = D / 8, R = kWave / CPR, P = kInnerBlocks / R;
  static_assert(WAVES <= kInnerGroups * kRelGroup && kInnerGroups <= NP && FirstParts<NP, 64 * WAVES, BLOCKS>::kPlanes == 1,
                "a thread ranks one block and holds the sums of all groups");
  const int c = lane % CPR, r = lane / CPR;
  const int per_head = (p.n_b + kInnerBlocks - 1) / kInnerBlocks;
  const int h = wave / per_head, b0 = (wave - h * per_head) * kInnerBlocks;
  if (h < p.H) {
    float4 k0[P], k1[P];
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const float4* kp = reinterpret_cast<const float4*>(p.rel_part + ((int64_t)h * p.n_b + min(b0 + i * R + r, p.n_b - 1)) * D + c * 8);
      k0[i] = kp[0];
      k1[i] = kp[1];
    }
    __builtin_amdgcn_sched_barrier(0);
    float qs[8];
    focus_row_sum<D, true>(qs, p.Q + (int64_t)h * p.qsh, p.qsn, p.kept_blocks, entry, min(max(n_focus, 0), p.n_focus_max), p.n_gen);
#pragma unroll
    for (int i = 0; i < P; ++i) {
      const float dot = chunk_dot_reduce<CPR>(qs, k0[i], k1[i]);
      if (c == 0) dots[wave * kInnerBlocks + i * R + r] = dot;
    }
  }
  __syncthreads();
  const int b = min((int)threadIdx.x, p.n_b - 1);
#pragma unroll
  for (int g = 0; g < kInnerGroups; ++g) {
    const int h0 = g * kRelGroup;
    float acc = h0 < p.H ? dots[h0 * per_head * kInnerBlocks + b] : 0.f;
#pragma unroll
    for (int w = 1; w < kRelGroup; ++w) acc = h0 + w < p.H ? acc + dots[(h0 + w) * per_head * kInnerBlocks + b] : acc;
    f.part[0][g] = acc;
  }
}
template <int NP, int THREADS, int BLOCKS>
__device__ __forceinline__ void rank_blocks(const AttnArgs& p, const FirstParts<NP, THREADS, BLOCKS>& f, bool per_head, int n_focus,
                                            typename KeptList<true, BLOCKS>::Id* kept_sh, TopkShared& sm, bool writer) {
  constexpr int kPlanes = FirstParts<NP, THREADS, BLOCKS>::kPlanes;
  const int tid = threadIdx.x;
  // more than eight wavefronts (one_split_waves: at most 256 blocks, at most 16 to keep): the first four rank
  constexpr int kRankWaves = THREADS > 512 ? 4 : THREADS / kWave;
  const bool tournament = BLOCKS <= 256 && (THREADS > 512 || p.n_keep * kRankWaves <= kWave);  // uniform
  if (!tournament) {
    block_topk_clear<THREADS>(sm);
    __syncthreads();
  }
  const int n_f = min(max(n_focus, 0), p.n_focus_max);
  const float scale = n_f > 0 ? 1.f / ((float)n_f * (float)p.H) : 0.f;
  const int n_groups = (p.H + kRelGroup - 1) / kRelGroup;
  float rel[kPlanes];
#pragma unroll
  for (int l = 0; l < kPlanes; ++l) {
    const float(&part)[NP] = f.part[l];
    const int b = tid + l * THREADS;
    float r = 0.f;  // in the order of sum_partials
    if (per_head) {
#pragma unroll
      for (int h = 0; h < NP; h += kRelGroup) {
        float g = part[h];
#pragma unroll
        for (int i = 1; i < kRelGroup; ++i) g = h + i < p.H ? g + part[h + i] : g;
        r = h < p.H ? r + g : r;
      }
      if (p.H > NP && b < p.n_b) r = sum_partials(p.rel_part, p.H, false, p.n_b, b, NP, r);
    } else {
#pragma unroll
      for (int g = 0; g < NP; ++g) r = g < n_groups ? r + part[g] : r;
      if (n_groups > NP && b < p.n_b) r = sum_partials(p.rel_part, n_groups, true, p.n_b, b, NP, r);
    }
    rel[l] = r * scale;
    if (writer && p.scores_out && b < p.n_b) p.scores_out[b] = rel[l];
  }
  if (tournament) {
    auto keyfn = [&](int, uint32_t& key) -> bool {
      key = order_key(rel[0]);
      return true;
    };
    if constexpr (BLOCKS <= 256)
      block_topk_small<256, true, (THREADS > 512 ? kRankWaves : 0)>(keyfn, p.n_b, p.n_keep, kept_sh, nullptr, sm);
  } else if constexpr (THREADS <= 512) {
    uint32_t key1[kPlanes];
#pragma unroll
    for (int l = 0; l < kPlanes; ++l) key1[l] = tid + l * THREADS < p.n_b ? order_key(rel[l]) + 1u : 0u;
    block_topk_planes<kPlanes, THREADS>(key1, p.n_b, p.n_keep, kept_sh, sm);
  }
  if (writer)
    for (int i = tid; i < p.n_keep; i += THREADS) p.kept_out[i] = kept_sh[i];
}

// Workgroups whose key range reaches the sink sub-tiles prepare the union of Eq. 8 once: a bitmap of the kept blocks, and
// whether the sink list is strictly ascending (then it cannot name a position twice).  A list of one sub-tile needs neither: its
// wavefront holds it in registers (few_sinks; three memory round trips behind the Top-C became none, 1 us of the 32K layer).
__device__ __forceinline__ int request_few_sinks(const AttnArgs& p, int lane) {
  return p.n_sink <= kSubTile && lane < p.n_sink && p.dense_rows == 0 ? p.sink_idx[lane] : -1;
}
struct SinkUnion {
  const uint32_t* kept_bits;  // see locate_subtile; null when there is none
  int ascending;
};
template <class Id>
__device__ __forceinline__ SinkUnion prepare_union(const AttnArgs& p, int split, const Id* kept_blocks, uint32_t* bits_sh,
                                                   int* unsorted_sh) {
  SinkUnion u;
  u.kept_bits = nullptr;
  u.ascending = -1;
  const int first_sink_sub = p.n_keep * p.sub_per_block + (p.N + kSubTile - 1) / kSubTile;
  const int n_round = (p.n_sub + kWavesPerGroup - 1) / kWavesPerGroup;                      // rounds of four sub-tiles ...
  const int last = n_round - 1 - (n_round - 1 - split) % p.n_split;                         // ... the last one of this split
  if (p.dense_rows == 0 && p.n_sink > kSubTile && (last + 1) * kWavesPerGroup > first_sink_sub) {  // uniform over the workgroup
    const bool bitmap = p.n_keep > 0 && p.n_b <= kBitmapBlocks;
    const int words = bitmap ? (p.n_b + 31) >> 5 : 0;
    for (int i = threadIdx.x; i < words; i += blockDim.x) bits_sh[i] = 0u;
    if (threadIdx.x == 0) *unsorted_sh = 0;
    __syncthreads();
    if (bitmap) {
      for (int i = threadIdx.x; i < p.n_keep; i += blockDim.x) {
        const int b = kept_blocks[i];
        if (b >= 0 && b < p.n_b) atomicOr(&bits_sh[b >> 5], 1u << (b & 31));
      }
    }
    for (int i = threadIdx.x; i + 1 < p.n_sink; i += blockDim.x)
      if (p.sink_idx[i + 1] <= p.sink_idx[i]) *unsorted_sh = 1;
    __syncthreads();
    if (bitmap) u.kept_bits = bits_sh;
    u.ascending = *unsorted_sh ? 0 : 1;
  }
  return u;
}

// The rounds of four sub-tiles of one key split (see SplitPlan) in the order in which a key loop takes them: head h begins h / H of the
// way down the list and wraps around.  All heads sweep their keys at the same time, and with the same place in the sweep the rows
// being fetched are the head stride apart, which for some lengths keeps meeting the same memory channels (32 heads, 16 queries:
// 33 024 rows 92 us from the top for every head, 87.5 this way; 32 832 rows 86.5 either way; 256 of 512 blocks, 256 response
// rows, 25 queries, whole layer 66 and 60).
struct SplitRounds {
  int first, step, n_rounds, turn, n_sub;
  __device__ __forceinline__ SplitRounds(const AttnArgs& p, int split, int h) {
    first = split * kWavesPerGroup;
    step = p.n_split * kWavesPerGroup;
    n_sub = p.n_sub;
    n_rounds = p.split_rounds + (split < p.split_rounds_more);
    turn = (int)__umulhi((uint32_t)h * p.head_turn, (uint32_t)n_rounds);  // < n_rounds
  }
  // sub-tile of slot `slot` in the i-th round; n_sub or more: none
  __device__ __forceinline__ int sub(int i, int slot) const {
    if (i >= n_rounds) return n_sub;
    const int r = i + turn;
    return first + slot + (r >= n_rounds ? r - n_rounds : r) * step;
  }
};

// The sub-tiles of 64 rounds at a time, lane i those of round i0 + i: a key loop takes them by lane reads, where working one out per round
// put a division and the wait for a block id in front of the products (a call of 32 heads, 8256 keys, 16 queries 27.4 -> 26.9 us, 28
// queries 28.8 -> 28.0; half of 512 blocks, 25 queries 50.5 -> 49.0; 8 heads, 16 448 keys 19.3 -> 18.6).  n: rows, -1: sub-tile row0 of
// the sink list.
struct RoundTable {
  int row0, n;
};
template <class Id>
__device__ __forceinline__ RoundTable tabulate_rounds(const AttnArgs& p, const SplitRounds& rounds, int slot, int i0, int lane, const Id* kept_blocks) {
  RoundTable r{0, 0};
  int sub = rounds.sub(i0 + lane, slot);
  if (sub >= p.n_sub) return r;
  if (p.dense_rows > 0) {
    r.row0 = sub * kSubTile;
    r.n = min(p.dense_rows - r.row0, kSubTile);
    return r;
  }
  const int n_blk_sub = p.n_keep * p.sub_per_block, n_resp_sub = (p.N + kSubTile - 1) / kSubTile;
  if (sub < n_blk_sub) {
    const int i = sub / p.sub_per_block, b = kept_blocks[i];
    if (b >= 0 && b < p.n_b) {
      r.row0 = b * p.B + (sub - i * p.sub_per_block) * kSubTile;
      r.n = max(min(min((b + 1) * p.B, p.M) - r.row0, kSubTile), 0);
    }
    return r;
  }
  sub -= n_blk_sub;
  if (sub < n_resp_sub) {
    r.row0 = p.M + sub * kSubTile;
    r.n = min(p.M + p.N - r.row0, kSubTile);
  } else {
    r.row0 = sub - n_resp_sub;
    r.n = -1;
  }
  return r;
}
// rounds 0, 1, 2, ... of a slot, one call each
template <class Id>
struct RoundList {
  const AttnArgs& p;
  const SplitRounds& rounds;
  const SinkUnion& uni;
  const Id* kept_blocks;
  int slot, lane, few_sinks, next = 0;
  RoundTable table{0, 0};
  __device__ __forceinline__ SubTile take() {
    const int i = next & (kWave - 1);
    if (i == 0) table = tabulate_rounds(p, rounds, slot, next, lane, kept_blocks);
    ++next;
    const int n = __builtin_amdgcn_readlane(table.n, i), row0 = __builtin_amdgcn_readlane(table.row0, i);
    if (n < 0) return locate_sinks(row0, lane, p.M, p.B, kept_blocks, p.n_keep, p.sink_idx, p.n_sink, uni.kept_bits, uni.ascending, few_sinks);
    SubTile t;
    t.kind = 0;
    t.row0 = row0;
    t.vmask = low_mask(n);
    t.sink_row = 0;
    return t;
  }
};

// Up to 16 active queries.  One workgroup works on one (head, key split); the key axis is walked in rounds of four 32-row
// sub-tiles ("slots"), and every one of its four wavefronts owns its slot end to end — it stages the sub-tile, multiplies it
// against the one query tile and keeps its own running softmax; the four states are merged at the end.
//
// FUSE bit 0 clear: kept_blocks comes from memory.
// FUSE bit 0 set (fused layer path): the workgroup first assembles R_b from the partial relevances and ranks
// them itself — every workgroup repeats this small computation instead of waiting for a separate Top-C kernel.
// FUSE bit 6 set (with bit 0): and works the partial relevances out, too (relevance_parts).
// FUSE bit 3 set (with bit 0): the partial relevances come per head, from a K scan, and not per group of four heads (more than 256 blocks: of
// up to eight heads; a variant of its own, because the choice at run time cost 0.9 us a layer of 32 heads and 323 blocks).
// FUSE bit 4 set (with bit 0): more than 256 blocks to rank.
// FUSE bit 2 set (dense probe layer): the scaled logits of every (query, key) are also written out, so that
// the column attention mass of Eq. 6 needs no QK^T pass of its own.
// FUSE bit 1 set: key loop, for launches in which a wavefront walks several sub-tiles (the dense comparison, the probe layer).  As in
// wide_attn_kernel with NT = 1 the K and V rows of the one stage travel separately.  Against two stages and a request for the pair: 32
// heads, 8256 keys 30.3 -> 28.3 us a call, 32 832 keys 86.3 -> 85.1; 8 heads, 16 448 keys 20.6 -> 18.9; 30 of 1024 blocks, whole layer
// 27.0 -> 26.1; probe layer of 32 832 keys 130.4 -> 128.7.
// WAVES: four, and a second, small kernel merges the key splits.  (Letting the last workgroup of a head merge them
// behind device-scope fences was measured on earlier forms: the fences cost several times what the launch does.)  Eight, twelve or sixteen
// for the one workgroup of a head with a short key list, which writes the output itself (one_split_waves); the first 256 threads store.
template <int D, int FUSE, int WAVES>
__global__ __launch_bounds__(64 * WAVES, WAVES == 4 ? 2 : WAVES / 4) void sparse_attn_kernel(ATTN_FIRST_PARAMS, const AttnArgs args) {
  const AttnArgs p = with_first(args, ATTN_FIRST_NAMES);
  using G = Geo<D>;
  constexpr bool FUSED = (FUSE & 1) != 0;                // Top-C in the prologue
  constexpr bool PIPE = (FUSE & 2) != 0;                 // key loop
  constexpr bool SPILL = (FUSE & 4) != 0;                // dense: also write the scaled logits (sink scoring)
  constexpr bool PER_HEAD = (FUSE & 8) != 0;             // FUSED: partial relevances per head, not per group of heads
  constexpr int BLOCKS = (FUSE & 32) != 0 ? kFusedMaxBlocks : ((FUSE & 16) != 0 ? kFusedManyBlocks : 256);  // FUSED: the most blocks to rank
  constexpr bool INNER = (FUSE & 64) != 0;               // FUSED: the relevances, too
  static_assert(!INNER || (FUSED && !PER_HEAD && WAVES > 4), "one workgroup per head");
  constexpr int kBufBytes = 2 * G::kStageBytes;          // one slot: K stage + V stage of a sub-tile
  static_assert(16 * D * 4 <= kBufBytes, "a wavefront's O tile fits its stage");
  __shared__ __attribute__((aligned(256))) char ldsA[WAVES * kBufBytes];
  __shared__ float2 ml_sh[WAVES][16];  // final merge: running maximum and sum per wavefront and query

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int split = PIPE ? blockIdx.x : blockIdx.y, h = PIPE ? blockIdx.y : blockIdx.x;
  const Counts counted(p);
  char* stageK = ldsA + wave * kBufBytes;  // the slot this wavefront owns
  char* stageV = stageK + G::kStageBytes;
  const uint16_t* Qh = p.Q + (int64_t)h * p.qsh;
  const uint16_t* Kh = p.K + (int64_t)h * p.ksh;
  const uint16_t* Vh = p.V + (int64_t)h * p.vsh;

  __shared__ __attribute__((aligned(16))) char topk_raw[FUSED ? sizeof(TopkShared) : 16];
  TopkShared& topk_sm = *reinterpret_cast<TopkShared*>(topk_raw);
  using Kept = KeptList<FUSED, BLOCKS>;
  __shared__ int32_t kept_beside[Kept::kEntriesBeside];
  typename Kept::Id* kept_sh = Kept::place(topk_raw, kept_beside);
  const typename Kept::Id* kept_blocks = kept_sh;
  if constexpr (!FUSED) kept_blocks = p.kept_blocks;
  __shared__ float dots_sh[INNER ? WAVES * kInnerBlocks : 1];
  // With the Top-C prologue ahead, the query rows are requested before it (their two round trips — row ids, then rows —
  // pass while the relevances are summed and ranked); without it they follow the first K/V requests (see below).
  bf16x8 q[G::kKSteps];
  int qrow_early = -1, few_sinks = -1;
  if (FUSED) {
    qrow_early = fetch_q_row(p.active_idx, 0, p.max_active, p.n_gen, lane);
    FirstParts<PER_HEAD && BLOCKS <= 256 ? 32 : 8, 64 * WAVES, BLOCKS> first;
    if constexpr (INNER) {
      const int entry = lane < p.n_focus_max ? p.kept_blocks[lane] : -1;
      few_sinks = request_few_sinks(p, lane);
      load_q_tile<D>(q, Qh, p.qsn, qrow_early, lane);
      relevance_parts<D, WAVES>(first, p, entry, counted.focus, dots_sh, wave, lane);
    } else {
      first_partials(first, p, PER_HEAD);
      few_sinks = request_few_sinks(p, lane);
      load_q_tile<D>(q, Qh, p.qsn, qrow_early, lane);
    }
    rank_blocks(p, first, PER_HEAD, counted.focus, kept_sh, topk_sm, blockIdx.x == 0 && blockIdx.y == 0);
  } else {
    few_sinks = request_few_sinks(p, lane);
  }
  __shared__ uint32_t kept_bits_sh[kBitmapBlocks / 32];
  __shared__ int sinks_unsorted_sh;
  static_assert(WAVES == 4 || (!PIPE && BLOCKS <= 256), "one split, a sub-tile per wavefront");
  static_assert(D == 128 || PIPE || WAVES > 4 ||
                    4 * (sizeof(ldsA) + sizeof(ml_sh) + sizeof(topk_raw) + sizeof(kept_beside) + sizeof(kept_bits_sh) + 16) <= 163840,
                "four workgroups share a compute unit (kAttnGroupsSmall)");
  const SinkUnion uni = prepare_union(p, split, kept_blocks, kept_bits_sh, &sinks_unsorted_sh);
  const uint32_t* kept_bits = uni.kept_bits;
  const int sinks_ascending = uni.ascending;

  // Order of the memory requests: the query row ids first (tiny, they return first), then the first
  // sub-tile's K and V rows as soon as its block id is known, then the query rows and the device-side count.
  const int st_end = p.n_sub;
  const SplitRounds rounds(p, split, h);
  const int st = split * WAVES + wave;
  const int qrow = FUSED ? qrow_early : fetch_q_row(p.active_idx, 0, p.max_active, p.n_gen, lane);
  SubTile t;
  t.kind = 0;
  t.row0 = 0;
  t.vmask = 0u;
  t.sink_row = 0;
  RoundList<typename Kept::Id> list{p, rounds, uni, kept_blocks, wave, lane, few_sinks};
  if (PIPE) {
    t = list.take();
    if (t.vmask != 0u) {
      issue_subtile<D>(Kh, p.ksn, t, stageK, lane);
      issue_subtile<D>(Vh, p.vsn, t, stageV, lane);
    }
  } else if (st < st_end) {
    t = locate_subtile(st, lane, p.M, p.N, p.B, p.n_b, p.sub_per_block, kept_blocks, p.n_keep, p.sink_idx, p.n_sink, kept_bits,
                          sinks_ascending, p.dense_rows, FUSED, few_sinks);
    if (t.vmask != 0u) {
      issue_subtile<D>(Kh, p.ksn, t, stageK, lane);
      issue_subtile<D>(Vh, p.vsn, t, stageV, lane);
    }
  }
  if (!FUSED) load_q_tile<D>(q, Qh, p.qsn, qrow, lane);
  const int n_act = counted.n_active(p);
  mask_q_tile<D>(q, 0, n_act, lane);

  float m_run = -INFINITY, l_run = 0.f;
  floatx4 o[G::kColTiles];
#pragma unroll
  for (int ct = 0; ct < G::kColTiles; ++ct) o[ct] = floatx4{0.f, 0.f, 0.f, 0.f};

  bool first = true;
  floatx4 kept_logits[2];  // SPILL: the raw logits of the sub-tile just multiplied, written out by the caller (see the key loops)
  auto consume = [&](const char* sK, const char* sV, uint32_t vmask, int row0) __attribute__((always_inline)) {  // one staged sub-tile into the running softmax
    floatx4 acc[2];
    qk_subtile<D>(acc, sK, q, lane);
    if (SPILL) {
      kept_logits[0] = acc[0];
      kept_logits[1] = acc[1];
    }
    float ps[8];
    const float alpha = softmax_step(acc, vmask, g, p.scale_log2, m_run, l_run, ps);
    // the running maximum settles after a few sub-tiles: the rescale is skipped when it would multiply by one
    if (!first && __ballot(alpha != 1.f) != 0ull) {
#pragma unroll
      for (int ct = 0; ct < G::kColTiles; ++ct) o[ct] *= alpha;
    }
    const bf16x8 pb = pack_bf16x8(ps);
    // O^T[dcol][query] += V^T . P^T
#pragma unroll
    for (int ct = 0; ct < G::kColTiles; ++ct) {
      const bf16x8 a = read_v_operand<D>(sV, ct, lane);
      o[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, pb, o[ct], 0, 0, 0);
    }
    first = false;
  };
  if (!PIPE) {
    // one sub-tile per wavefront at most (the launcher picks this variant only when a split holds no more sub-tiles
    // than the workgroup has wavefronts): no key loop, and none of its code — these launches are a few microseconds
    // long and start with a cold instruction cache, so every KB of code they walk through shows in the run time
    if (t.vmask != 0u) {
      wait_loads();
      consume(stageK, stageV, t.vmask, t.row0);
      if (SPILL) spill_logits(p.logits_out, h, p.dense_rows, p.max_active, t.row0, kept_logits, p.scale_log2, lane);  // contiguous rows only (dense)
    }
  } else {
    // One stage, whose K and V rows travel separately (see wide_attn_kernel): the next K rows are requested as soon as the present ones
    // are in registers, then the V rows likewise.  No barrier: the slots are private to the wavefront.
    // SPILL: the logits go out behind the request of the next V rows.  A whole sub-tile is two stores; they are counted, so that
    // nothing waits for them; those of a ragged one count for nothing and are waited for.
    SubTile tn = list.take();
    bool stored = false;  // two stores behind the V rows under way
    for (int i = 0; i < rounds.n_rounds; ++i) {
      const bool here = t.vmask != 0u, more = tn.vmask != 0u;  // wave-uniform
      floatx4 acc[2];
      bf16x8 kop[2][G::kKSteps], vop[G::kColTiles], pb;
      if (here) {
        if (SPILL && stored)
          wait_loads_but<G::kLoads + kSpillStores>();
        else
          wait_loads_but<G::kLoads>();  // all but the V rows
        read_k_operands16<D>(kop, stageK, lane);
      }
      if (more) issue_subtile<D>(Kh, p.ksn, tn, stageK, lane);
      if (here) {
#pragma unroll
        for (int kt = 0; kt < 2; ++kt) {
          acc[kt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int kk = 0; kk < G::kKSteps; ++kk) acc[kt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop[kt][kk], q[kk], acc[kt], 0, 0, 0);
        }
        float ps[8];
        const float alpha = softmax_step(acc, t.vmask, g, p.scale_log2, m_run, l_run, ps);
        if (!first && __ballot(alpha != 1.f) != 0ull) {
#pragma unroll
          for (int ct = 0; ct < G::kColTiles; ++ct) o[ct] *= alpha;
        }
        pb = pack_bf16x8(ps);
        first = false;
        if (!more)
          wait_loads();
        else if (SPILL && stored)
          wait_loads_but<G::kLoads + kSpillStores>();
        else
          wait_loads_but<G::kLoads>();  // all but the next K rows
        read_v_operands16<D>(vop, stageV, lane);
      }
      if (more) issue_subtile<D>(Vh, p.vsn, tn, stageV, lane);
      if (here) {
#pragma unroll
        for (int ct = 0; ct < G::kColTiles; ++ct) o[ct] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vop[ct], pb, o[ct], 0, 0, 0);
        if (SPILL) spill_logits(p.logits_out, h, p.dense_rows, p.max_active, t.row0, acc, p.scale_log2, lane);
      }
      stored = here && t.vmask == 0xffffffffu;
      t = tn;
      tn = list.take();
    }
  }

  // ---- merge the four wavefronts through LDS: each leaves its O tile [16][D] in its own stage.  The 16-byte chunks of a row are
  // permuted by its number: unpermuted, the sixteen rows of a store all begin at the same bank (2170 of
  // this kernel's 15 700 cycles; whole layer 32 heads 32K, 7 of 256 blocks 13.8 -> 13.0 us, 13 of 128 blocks 16.6 -> 15.4).
  constexpr int kVec = D / 64;  // chunks per thread in the merge: mc, mc + 16
  auto chunk_at = [&](int w, int row, int ch) __attribute__((always_inline)) {
    return reinterpret_cast<floatx4*>(ldsA + w * kBufBytes + (row * (D / 4) + (ch ^ row)) * 16);
  };
  const int mq = threadIdx.x >> 4, mc = threadIdx.x & 15;  // query this thread merges
  wait_loads();
  __syncthreads();  // every staged sub-tile has been consumed by everyone
#pragma unroll
  for (int ct = 0; ct < G::kColTiles; ++ct) *chunk_at(wave, c, 4 * ct + g) = o[ct];
  if (g == 0) ml_sh[wave][c] = make_float2(m_run, l_run);
  __syncthreads();
  float2 ml[WAVES];
  floatx4 ow[WAVES][kVec];
#pragma unroll
  for (int w = 0; w < WAVES; ++w) {
    ml[w] = ml_sh[w][WAVES == 4 ? mq : mq & 15];
#pragma unroll
    for (int i = 0; i < kVec; ++i) ow[w][i] = *chunk_at(w, WAVES == 4 ? mq : mq & 15, mc + 16 * i);
  }
  float mmax = ml[0].x;
#pragma unroll
  for (int w = 1; w < WAVES; ++w) mmax = fmaxf(mmax, ml[w].x);
  floatx4 acc_o[kVec];
#pragma unroll
  for (int i = 0; i < kVec; ++i) acc_o[i] = floatx4{0.f, 0.f, 0.f, 0.f};
  float lsum = 0.f;
#pragma unroll
  for (int w = 0; w < WAVES; ++w) {
    const float f = ml[w].y > 0.f ? __builtin_amdgcn_exp2f(ml[w].x - mmax) : 0.f;
    lsum += f * ml[w].y;
#pragma unroll
    for (int i = 0; i < kVec; ++i) acc_o[i] += f * ow[w][i];
  }
  const int a = mq;  // position in the active list
  if (a < n_act && (WAVES == 4 || a < 16)) {
    if (p.n_split == 1) {
      const float inv = lsum > 0.f ? 1.f / lsum : 0.f;
      uint16_t* dst = p.out + (int64_t)h * p.osh + (int64_t)a * p.osn + mc * 4;
#pragma unroll
      for (int i = 0; i < kVec; ++i)
        *reinterpret_cast<uint2*>(dst + 64 * i) =
            make_uint2(cvt_pk_bf16(acc_o[i][0] * inv, acc_o[i][1] * inv), cvt_pk_bf16(acc_o[i][2] * inv, acc_o[i][3] * inv));
      if (p.lse && mc == 0)
        p.lse[(int64_t)h * p.max_active + a] = lsum > 0.f ? (mmax + __builtin_amdgcn_logf(lsum)) * kLn2 : -INFINITY;
      if (p.lse2_out && mc == 0)
        p.lse2_out[(int64_t)h * p.q_pad + a] = lsum > 0.f ? mmax + __builtin_amdgcn_logf(lsum) : INFINITY;
    } else {
      const int64_t row = ((int64_t)h * p.q_pad + a) * p.n_split + split;
#pragma unroll
      for (int i = 0; i < kVec; ++i) *reinterpret_cast<floatx4*>(p.part_o + row * D + mc * 4 + 64 * i) = acc_o[i];
      if (mc == 0) *reinterpret_cast<float2*>(p.part_ml + 2 * row) = make_float2(lsum > 0.f ? mmax : -INFINITY, lsum);
    }
  }
}

// All operands of a sub-tile for the 32x32 tiles (read_k_operands16).
template <int D>
__device__ __forceinline__ void read_k_operands32(bf16x8 (&k)[D / 16], const char* stageK, int lane) {
  const uint32_t a = lds_address(stageK) + stage_off<D>(lane & 31, lane >> 5);  // chunk 2 ks + hh: 32 ks added to the swizzled place
  if constexpr (D == 128) {
    asm volatile(
        "ds_read_b128 %0, %8\n\tds_read_b128 %1, %9\n\tds_read_b128 %2, %10\n\tds_read_b128 %3, %11\n\t"
        "ds_read_b128 %4, %12\n\tds_read_b128 %5, %13\n\tds_read_b128 %6, %14\n\tds_read_b128 %7, %15\n\ts_waitcnt lgkmcnt(0)"
        : "=&v"(k[0]), "=&v"(k[1]), "=&v"(k[2]), "=&v"(k[3]), "=&v"(k[4]), "=&v"(k[5]), "=&v"(k[6]), "=&v"(k[7])
        : "v"(a), "v"(a ^ 32u), "v"(a ^ 64u), "v"(a ^ 96u), "v"(a ^ 128u), "v"(a ^ 160u), "v"(a ^ 192u), "v"(a ^ 224u)
        : "memory");
  } else {
    asm volatile(
        "ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\ts_waitcnt lgkmcnt(0)"
        : "=&v"(k[0]), "=&v"(k[1]), "=&v"(k[2]), "=&v"(k[3])
        : "v"(a), "v"(a ^ 32u), "v"(a ^ 64u), "v"(a ^ 96u)
        : "memory");
  }
}
template <int D>
__device__ __forceinline__ void read_v_operands32(bf16x8 (&v)[2][D / 32], const char* stageV, int lane) {
  const int s = lane & 15, b = lane >> 4;
  const int row = 4 * (b >> 1) + (s >> 2), col = 16 * (b & 1) + 4 * (s & 3);
  const uint32_t a = lds_address(stageV) + vstage_off<D>(row, col >> 3) + (col & 7) * 2;  // d tile dt: chunk 4 dt further, k-step ks: row 16 ks
  shortx4 r[2][D / 32][2];
  if constexpr (D == 128) {
    asm volatile(
        "ds_read_b64_tr_b16 %0, %16\n\tds_read_b64_tr_b16 %1, %16 offset:2048\n\t"
        "ds_read_b64_tr_b16 %2, %17\n\tds_read_b64_tr_b16 %3, %17 offset:2048\n\t"
        "ds_read_b64_tr_b16 %4, %18\n\tds_read_b64_tr_b16 %5, %18 offset:2048\n\t"
        "ds_read_b64_tr_b16 %6, %19\n\tds_read_b64_tr_b16 %7, %19 offset:2048\n\t"
        "ds_read_b64_tr_b16 %8, %16 offset:4096\n\tds_read_b64_tr_b16 %9, %16 offset:6144\n\t"
        "ds_read_b64_tr_b16 %10, %17 offset:4096\n\tds_read_b64_tr_b16 %11, %17 offset:6144\n\t"
        "ds_read_b64_tr_b16 %12, %18 offset:4096\n\tds_read_b64_tr_b16 %13, %18 offset:6144\n\t"
        "ds_read_b64_tr_b16 %14, %19 offset:4096\n\tds_read_b64_tr_b16 %15, %19 offset:6144\n\ts_waitcnt lgkmcnt(0)"
        : "=&v"(r[0][0][0]), "=&v"(r[0][0][1]), "=&v"(r[0][1][0]), "=&v"(r[0][1][1]), "=&v"(r[0][2][0]), "=&v"(r[0][2][1]),
          "=&v"(r[0][3][0]), "=&v"(r[0][3][1]), "=&v"(r[1][0][0]), "=&v"(r[1][0][1]), "=&v"(r[1][1][0]), "=&v"(r[1][1][1]),
          "=&v"(r[1][2][0]), "=&v"(r[1][2][1]), "=&v"(r[1][3][0]), "=&v"(r[1][3][1])
        : "v"(a), "v"(a ^ 64u), "v"(a ^ 128u), "v"(a ^ 192u)
        : "memory");
  } else {
    asm volatile(
        "ds_read_b64_tr_b16 %0, %8\n\tds_read_b64_tr_b16 %1, %8 offset:1024\n\t"
        "ds_read_b64_tr_b16 %2, %9\n\tds_read_b64_tr_b16 %3, %9 offset:1024\n\t"
        "ds_read_b64_tr_b16 %4, %8 offset:2048\n\tds_read_b64_tr_b16 %5, %8 offset:3072\n\t"
        "ds_read_b64_tr_b16 %6, %9 offset:2048\n\tds_read_b64_tr_b16 %7, %9 offset:3072\n\ts_waitcnt lgkmcnt(0)"
        : "=&v"(r[0][0][0]), "=&v"(r[0][0][1]), "=&v"(r[0][1][0]), "=&v"(r[0][1][1]), "=&v"(r[1][0][0]), "=&v"(r[1][0][1]),
          "=&v"(r[1][1][0]), "=&v"(r[1][1][1])
        : "v"(a), "v"(a ^ 64u)
        : "memory");
  }
#pragma unroll
  for (int ks = 0; ks < 2; ++ks)
#pragma unroll
    for (int dt = 0; dt < D / 32; ++dt) {
      struct { shortx4 a, b; } both = {r[ks][dt][0], r[ks][dt][1]};
      v[ks][dt] = __builtin_bit_cast(bf16x8, both);
    }
}

// One staged sub-tile of 32 keys against a tile of 32 queries (32x32x16 MFMA), into the running softmax.
//   S^T = K Q^T   lane (query = lane % 32, hh = lane / 32), register v: logit of key 8 (v / 4) + 4 hh + v % 4
//   O^T = V^T P^T the same registers, packed to bf16, are the B operand of k-step v / 8
// k_operand(ks) / v_operand(dt, ks) supply the A operands; l_run is this lane's share of the row sum (its 16 of the 32 keys).
// r_run is the same for the probabilities as they enter the PV product, rounded to bf16.  SUMS: bit 0 l_run, bit 1 r_run is kept.
// Bit 2: O is rescaled for every sub-tile, also by one.  Where the compiler kept two copies of O for the two sides of that branch (the
// 32-query tiles of a block entry at d = 64) the moves between them cost more than the products.
// First half: logits, running maximum and sums (l_run; r_run is only rescaled), the probabilities ps.
template <int D, int SUMS, class KOp>
__device__ __forceinline__ void probabilities32(const KOp k_operand, const bf16x8 (&q)[D / 16], uint32_t vmask, int hh, float scale_log2,
                                                float& m_run, float& l_run, float& r_run, floatx16 (&o)[D / 32], float (&ps)[16]) {
  constexpr int kKS = D / 16, kDT = D / 32;
  floatx16 acc;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
  for (int ks = 0; ks < kKS; ++ks) acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(k_operand(ks), q[ks], acc, 0, 0, 0);
  if (vmask != 0xffffffffu) {  // wave-uniform: slots that hold no key
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = ((vmask >> (8 * (v >> 2) + 4 * hh + (v & 3))) & 1u) ? acc[v] : -INFINITY;
  }
  float mx = fmaxf(acc[0], acc[1]);
#pragma unroll
  for (int v = 2; v < 16; ++v) mx = fmaxf(mx, acc[v]);
  const uintx2 sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
  mx = fmaxf(__uint_as_float(sw.x), __uint_as_float(sw.y)) * scale_log2;
  const float m_new = fmaxf(m_run, mx);
  const float m_use = m_new == -INFINITY ? 0.f : m_new;
  if ((SUMS & 4) || __ballot(m_new != m_run) != 0ull) {  // some running maximum of this wavefront moves (rare after the first sub-tiles)
    const float alpha = __builtin_amdgcn_exp2f(m_run - m_use);
    if (SUMS & 1) l_run *= alpha;
    if (SUMS & 2) r_run *= alpha;
#pragma unroll
    for (int dt = 0; dt < kDT; ++dt) o[dt] *= alpha;
    m_run = m_new;
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) ps[v] = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[v], scale_log2, -m_use));
  if (SUMS & 1) {
    float sum = ps[0] + ps[1];
#pragma unroll
    for (int v = 2; v < 16; v += 2) sum += ps[v] + ps[v + 1];
    l_run += sum;
  }
}
// the eight of k-step ks, packed
__device__ __forceinline__ uint4 pack_probabilities(const float (&ps)[16], int ks) {
  return make_uint4(cvt_pk_bf16(ps[8 * ks], ps[8 * ks + 1]), cvt_pk_bf16(ps[8 * ks + 2], ps[8 * ks + 3]),
                    cvt_pk_bf16(ps[8 * ks + 4], ps[8 * ks + 5]), cvt_pk_bf16(ps[8 * ks + 6], ps[8 * ks + 7]));
}
template <int D, int SUMS, class KOp, class VOp>
__device__ __forceinline__ void attend_subtile32(const KOp k_operand, const VOp v_operand, const bf16x8 (&q)[D / 16], uint32_t vmask,
                                                 int hh, float scale_log2, float& m_run, float& l_run, float& r_run,
                                                 floatx16 (&o)[D / 32]) {
  constexpr int kDT = D / 32;
  float ps[16];
  probabilities32<D, SUMS>(k_operand, q, vmask, hh, scale_log2, m_run, l_run, r_run, o, ps);
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const uint4 pk = pack_probabilities(ps, ks);
    if (SUMS & 2) r_run += add_bf16_pair(add_bf16_pair(0.f, pk.x), pk.y) + add_bf16_pair(add_bf16_pair(0.f, pk.z), pk.w);
    const bf16x8 pb = as_bf16x8(pk);
#pragma unroll
    for (int dt = 0; dt < kDT; ++dt) o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v_operand(dt, ks), pb, o[dt], 0, 0, 0);
  }
}

// fp32 O tile [32 queries][D] in LDS for the merge of several wavefronts: byte offset of 16-byte chunk ch of query row r.
// Swizzled so that neither the writes (32 rows, two chunks) nor the reads (consecutive chunks of a few rows) conflict: any 16 rows at
// one chunk, and any 16 chunks of one row, lie in 16 different groups of four banks (with 8 different ones a layer of 24 queries took
// 16.0 us instead of 15.6, one of 196 queries on 4 K/V heads 25.0 instead of 24.3).
template <int D>
__device__ __forceinline__ int o_chunk(int row, int ch) {
  return (row * (D / 4) + (ch ^ (row & (D / 4 - 1)))) * 16;
}
template <int D>
__device__ __forceinline__ void store_o_tile(char* dst, const floatx16 (&o)[D / 32], int qi, int hh) {
#pragma unroll
  for (int dt = 0; dt < D / 32; ++dt)
#pragma unroll
    for (int j = 0; j < 4; ++j)
      *reinterpret_cast<floatx4*>(dst + o_chunk<D>(qi, 8 * dt + 2 * j + hh)) =
          floatx4{o[dt][4 * j], o[dt][4 * j + 1], o[dt][4 * j + 2], o[dt][4 * j + 3]};
}

// More than 16 queries: the same work decomposition as the 16-query kernel — a sub-tile goes from the memory request to the
// MFMAs in one slot of LDS — with 32-query tiles on v_mfma_f32_32x32x16_bf16.  A 32x32 tile takes
// half the LDS operand reads and half the MFMA instructions of two 16-query tiles, so that the QK^T -> softmax -> PV chain of
// an in-order wavefront fits into the time its share of HBM needs for the next sub-tile (probabilities32).
// NT = 1 (up to 32 queries per query group), four wavefronts: a wavefront owns its slot; no barrier in the key loop.
// NT = 2 (up to 64), eight wavefronts: wavefronts s and s + 4 share slot s, each stages half of its rows (K / V) and carries
//   one query tile; two stages per slot, one barrier per round.  (One wavefront with both tiles needs 128 accumulator registers outside the
//   vector registers, and copying them for the rescale made its chain longer than the memory time.)  The second tile's
//   wavefronts only stage when the device-side count leaves it empty.
// MODE bit 0: Top-C in the prologue.  Bit 1: a slot walks several sub-tiles (key loop).  Bit 3: the rows are read by several query groups
// and should stay in the L2.  Bits 4 and 5 (with bit 0): more than 256 blocks to rank, up to kFusedManyBlocks or kFusedMaxBlocks.
// NT = 1 has one stage per slot, whose K and V rows travel separately: the next K rows are requested as soon as the present ones are in
// registers, then the V rows likewise, so that a wavefront always has one of the two under way.  Loads alone, in that order, read 538 MB in
// 77 us (7.0 TB/s); a pair of K and V requested at a time, when the pair before it has come, 80 us.  With the products around them what is left of that is
// (two stages per slot, pairs, before): 8256 keys, 32 heads, 28 queries 30.7 -> 29.9 us a call; 256 of 512 blocks, 256 response rows and
// 327 sinks, 25 queries 54.9 -> 54.0; 32 832 keys the same.  The rows of several query groups come from the L2, where waiting for both at
// once is the better one (196 queries on 4 K/V heads, 16 640 keys 25.9 and 26.3).
// Bound by HBM.  32 heads, 32 832 keys, all kept: 87 us with 28 queries (6.2 TB/s; 16-query tiles on shared sub-tiles took 94),
// 93 us with 64 (101); half of the 64-row blocks and 327 sinks: 51 us (57).
// Grid: one list (list_index).  Workgroups go to the XCDs round-robin, so the query groups of one (head, key split) pair are
// placed eight apart: they run on the same XCD at about the same time and its L2 serves their common K/V rows.
template <int D, int NT, int MODE>
__global__ __launch_bounds__(256 * NT, 2) void wide_attn_kernel(WIDE_FIRST_PARAMS, const AttnArgs args) {
  AttnArgs p = with_first(args, rel_part, active_idx, Q, counts, n_b, H, max_active, args.n_gen, n_split, n_sub);
  p.q_groups = q_groups;
  using G = Geo<D>;
  constexpr bool FUSED = (MODE & 1) != 0, PIPE = (MODE & 2) != 0;
  constexpr bool DOUBLE = NT == 2 && PIPE;                   // two stages per slot
  constexpr bool APART = NT == 1 && PIPE && (MODE & 8) == 0;  // K and V rows travel separately
  constexpr int BLOCKS = (MODE & 32) != 0 ? kFusedMaxBlocks : ((MODE & 16) != 0 ? kFusedManyBlocks : 256);
  constexpr int kPolicy = (MODE & 8) != 0 ? 0 : kStreamPolicy;
  constexpr int kKS = D / 16, kDT = D / 32;
  constexpr int kBufBytes = 2 * G::kStageBytes;  // K stage + V stage of a sub-tile
  constexpr int kOChunks = D / 4;                // 16-byte chunks of one fp32 output row
  static_assert(32 * D * 4 <= kBufBytes, "an O tile fits a slot");
  __shared__ __attribute__((aligned(256))) char ldsA[kWavesPerGroup * kBufBytes];
  __shared__ __attribute__((aligned(16))) char ldsB[DOUBLE ? kWavesPerGroup * kBufBytes : 16];
  __shared__ float2 ml_sh[kWavesPerGroup][32];
  __shared__ __attribute__((aligned(16))) char topk_raw[FUSED ? sizeof(TopkShared) : 16];
  using Kept = KeptList<FUSED, BLOCKS>;
  __shared__ int32_t kept_beside[Kept::kEntriesBeside];
  __shared__ uint32_t kept_bits_sh[kBitmapBlocks / 32];
  __shared__ int sinks_unsorted_sh;

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int slot = wave & (kWavesPerGroup - 1), tile = NT == 1 ? 0 : wave >> 2;
  const int qi = lane & 31, hh = lane >> 5;
  const int slot8 = list_index() >> 3;
  int first8 = slot8, qg = 0;
  if (p.q_groups > 1) {
    first8 = slot8 / p.q_groups;
    qg = slot8 - first8 * p.q_groups;
  }
  const int pair = first8 * 8 + (int)(blockIdx.x & 7u);
  if (pair >= p.n_split * p.H) return;  // whole workgroup
  const int h = pair / p.n_split, split = pair - h * p.n_split;
  const Counts counted(p);
  const int q0 = (qg * NT + tile) * 32;  // first query of this wavefront's tile
  const uint16_t* Qh = p.Q + (int64_t)h * p.qsh;
  const uint16_t* Kh = p.K + (int64_t)h * p.ksh;
  const uint16_t* Vh = p.V + (int64_t)h * p.vsh;

  int qrow = q0 + qi < p.max_active ? p.active_idx[q0 + qi] : -1;
  if (qrow >= p.n_gen) qrow = -1;
  bf16x8 q[kKS];  // B operand of K Q^T: lane (query, hh) holds Q[query][16 ks + 8 hh .. + 7]
  auto load_q = [&]() __attribute__((always_inline)) {
    const uint16_t* src = Qh + (int64_t)max(qrow, 0) * p.qsn + hh * 8;
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks) q[ks] = as_bf16x8(*reinterpret_cast<const uint4*>(src + ks * 16));
  };
  typename Kept::Id* kept_sh = Kept::place(topk_raw, kept_beside);
  const typename Kept::Id* kept_blocks = kept_sh;
  if constexpr (!FUSED) kept_blocks = p.kept_blocks;
  int few_sinks;
  if (FUSED) {  // the query rows travel while the blocks are ranked
    FirstParts<8, 256 * NT, BLOCKS> first;  // (per head, from a K scan: the other parts are requested when they are added)
    first_partials(first, p, p.rel_per_head);
    few_sinks = request_few_sinks(p, lane);
    if (qg > 0 && qg * NT * 32 >= counted.n_active(p)) return;  // a query group past the device-side count has nothing to do
    load_q();
    rank_blocks(p, first, p.rel_per_head, counted.focus, kept_sh, *reinterpret_cast<TopkShared*>(topk_raw), pair == 0 && qg == 0);
  } else {
    few_sinks = request_few_sinks(p, lane);
    if (qg > 0 && qg * NT * 32 >= counted.n_active(p)) return;
  }
  const SinkUnion uni = prepare_union(p, split, kept_blocks, kept_bits_sh, &sinks_unsorted_sh);

  const SplitRounds rounds(p, split, h);
  auto locate = [&](int sub) __attribute__((always_inline)) {
    SubTile t;
    t.kind = 0;
    t.row0 = 0;
    t.vmask = 0u;
    t.sink_row = 0;
    if (sub < p.n_sub)
      t = locate_subtile(sub, lane, p.M, p.N, p.B, p.n_b, p.sub_per_block, kept_blocks, p.n_keep, p.sink_idx, p.n_sink, uni.kept_bits,
                         uni.ascending, p.dense_rows, FUSED, few_sinks);
    return t;
  };
  auto request = [&](const SubTile& t, char* stage) __attribute__((always_inline)) {
    if (t.vmask == 0u) return;
    if (NT == 1 || tile == 0) issue_subtile<D, false, kPolicy>(Kh, p.ksn, t, stage, lane);
    if (NT == 1 || tile == 1) issue_subtile<D, true, kPolicy>(Vh, p.vsn, t, stage + G::kStageBytes, lane);
  };
  auto staged = [&]() __attribute__((always_inline)) {  // every requested row of this round is in LDS
    wait_loads();
    if (NT > 1) __syncthreads();
  };
  char* slotA = ldsA + slot * kBufBytes;
  RoundList<typename Kept::Id> list{p, rounds, uni, kept_blocks, slot, lane, few_sinks};
  SubTile t = APART ? list.take() : locate(PIPE ? rounds.sub(0, slot) : split * kWavesPerGroup + slot);
  request(t, slotA);
  if (!FUSED) load_q();
  const int n_act = counted.n_active(p);
  {
    const bool live = qrow >= 0 && q0 + qi < n_act;
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks) q[ks] = live ? q[ks] : as_bf16x8(make_uint4(0u, 0u, 0u, 0u));
  }
  float m_run = -INFINITY, l_run = 0.f;  // l_run: this lane's share of the row sum (its 16 of every 32 keys)
  floatx16 o[kDT];
#pragma unroll
  for (int dt = 0; dt < kDT; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[dt][v] = 0.f;

  // one staged sub-tile into the running softmax
  auto consume = [&](auto k_operand, auto v_operand, uint32_t vmask) __attribute__((always_inline)) {
    float unused = 0.f;
    attend_subtile32<D, 1>(k_operand, v_operand, q, vmask, hh, p.scale_log2, m_run, l_run, unused, o);
  };
  auto k_at = [&](const char* stage, int ks) __attribute__((always_inline)) {
    return as_bf16x8(*reinterpret_cast<const uint4*>(stage + stage_off<D>(qi, 2 * ks + hh)));
  };
  auto v_at = [&](const char* stage, int dt, int ks) __attribute__((always_inline)) {
    return read_v_operand32<D>(stage + G::kStageBytes, dt, ks, lane);
  };
  const bool tile_live = q0 < n_act;
  if (!PIPE) {  // one sub-tile per slot at most
    staged();
    if (t.vmask != 0u && tile_live)
      consume([&](int ks) { return k_at(slotA, ks); }, [&](int dt, int ks) { return v_at(slotA, dt, ks); }, t.vmask);
  } else if constexpr (APART) {
    SubTile tn = list.take();
    for (int i = 0; i < rounds.n_rounds; ++i) {
      const bool here = t.vmask != 0u, more = tn.vmask != 0u;  // wave-uniform
      bf16x8 kop[kKS], vop[2][kDT], pb[2];
      if (here) {
        wait_loads_but<G::kLoads>();  // all but the V rows
        read_k_operands32<D>(kop, slotA, lane);
      }
      if (more) issue_subtile<D, false, kPolicy>(Kh, p.ksn, tn, slotA, lane);
      if (here) {
        float ps[16];
        probabilities32<D, 1>([&](int ks) { return kop[ks]; }, q, t.vmask, hh, p.scale_log2, m_run, l_run, l_run, o, ps);
#pragma unroll
        for (int ks = 0; ks < 2; ++ks) pb[ks] = as_bf16x8(pack_probabilities(ps, ks));
        if (more)
          wait_loads_but<G::kLoads>();  // all but the next K rows
        else
          wait_loads();
        read_v_operands32<D>(vop, slotA + G::kStageBytes, lane);
      }
      if (more) issue_subtile<D, true, kPolicy>(Vh, p.vsn, tn, slotA + G::kStageBytes, lane);
      if (here) {
#pragma unroll
        for (int ks = 0; ks < 2; ++ks)
#pragma unroll
          for (int dt = 0; dt < kDT; ++dt) o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vop[ks][dt], pb[ks], o[dt], 0, 0, 0);
      }
      t = tn;
      tn = list.take();
    }
  } else {
    SubTile tn = locate(rounds.sub(1, slot));
    int i = 0;
    // One round: `t` sits in `cur`.  Between the arrival of its rows and the request of the next ones lies only what has to:
    // the operand reads the compiler would otherwise put behind the arrival of the next rows (the transposed V reads, which
    // it cannot tell from the stage being filled), or that the request overwrites.  The sub-tile after the next is located —
    // a block id from memory — once the request is out.
    auto round = [&](const char* cur, char* nxt) __attribute__((always_inline)) {
      staged();
      bf16x8 kop[kKS], vop[2][kDT];
#pragma unroll
      for (int ks = 0; ks < 2; ++ks)
#pragma unroll
        for (int dt = 0; dt < kDT; ++dt) vop[ks][dt] = v_at(cur, dt, ks);
      if (!DOUBLE) {
#pragma unroll
        for (int ks = 0; ks < kKS; ++ks) kop[ks] = k_at(cur, ks);
      }
      wait_lds_reads();
      request(tn, nxt);
      const SubTile t2 = locate(rounds.sub(i + 2, slot));
      if (t.vmask != 0u && tile_live)
        consume([&](int ks) { return DOUBLE ? k_at(cur, ks) : kop[ks]; }, [&](int dt, int ks) { return vop[ks][dt]; }, t.vmask);
      t = tn;
      tn = t2;
      ++i;
    };
    if (DOUBLE) {
      char* slotB = ldsB + slot * kBufBytes;
      while (i < rounds.n_rounds) {  // uniform over the workgroup
        round(slotA, slotB);
        if (i < rounds.n_rounds) round(slotB, slotA);
      }
    } else {
      while (i < rounds.n_rounds) round(slotA, slotA);
    }
  }

  // ---- merge the four slots, one query tile at a time, through LDS
  if (NT > 1) __syncthreads();  // the slots have been read by both wavefronts
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    const int qn = (qg * NT + n) * 32;
    if (qn >= n_act) break;      // uniform
    if (n > 0) __syncthreads();  // the previous tile has been read by everyone
    if (NT == 1 || tile == n) {
      store_o_tile<D>(slotA, o, qi, hh);
      const uintx2 sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_run), __float_as_uint(l_run), false, false);
      if (hh == 0) ml_sh[slot][qi] = make_float2(m_run, __uint_as_float(sw.x) + __uint_as_float(sw.y));
    }
    __syncthreads();
    constexpr int kPerQuery = 8 * NT;  // threads that share a query
    const int mq = threadIdx.x / kPerQuery, c0 = threadIdx.x % kPerQuery;  // thread = (query, chunks c0, c0 + kPerQuery, ...)
    float2 ml[kWavesPerGroup];
    float mmax = -INFINITY, lsum = 0.f;
#pragma unroll
    for (int w = 0; w < kWavesPerGroup; ++w) {
      ml[w] = ml_sh[w][mq];
      mmax = fmaxf(mmax, ml[w].x);
    }
    float f[kWavesPerGroup];
#pragma unroll
    for (int w = 0; w < kWavesPerGroup; ++w) {
      f[w] = ml[w].y > 0.f ? __builtin_amdgcn_exp2f(ml[w].x - mmax) : 0.f;
      lsum += f[w] * ml[w].y;
    }
    const int a = qn + mq;
    if (a < n_act) {
      const int64_t row = ((int64_t)h * p.q_pad + a) * p.n_split + split;
      const float inv = lsum > 0.f ? 1.f / lsum : 0.f;
#pragma unroll
      for (int i = 0; i < kOChunks / kPerQuery; ++i) {
        const int ch = c0 + kPerQuery * i;
        floatx4 s = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kWavesPerGroup; ++w) s += f[w] * *reinterpret_cast<const floatx4*>(ldsA + w * kBufBytes + o_chunk<D>(mq, ch));
        if (p.n_split == 1)
          *reinterpret_cast<uint2*>(p.out + (int64_t)h * p.osh + (int64_t)a * p.osn + ch * 4) =
              make_uint2(cvt_pk_bf16(s[0] * inv, s[1] * inv), cvt_pk_bf16(s[2] * inv, s[3] * inv));
        else
          *reinterpret_cast<floatx4*>(p.part_o + row * D + ch * 4) = s;
      }
      if (c0 == 0) {
        if (p.n_split == 1) {
          if (p.lse) p.lse[(int64_t)h * p.max_active + a] = lsum > 0.f ? (mmax + __builtin_amdgcn_logf(lsum)) * kLn2 : -INFINITY;
          if (p.lse2_out) p.lse2_out[(int64_t)h * p.q_pad + a] = lsum > 0.f ? mmax + __builtin_amdgcn_logf(lsum) : INFINITY;
        } else {
          *reinterpret_cast<float2*>(p.part_ml + 2 * row) = make_float2(lsum > 0.f ? mmax : -INFINITY, lsum);
        }
      }
    }
  }
}

// Merge of the per-split partial results: out = sum_s f_s O_s / sum_s f_s l_s, f_s = exp2(m_s - max m).
// One workgroup per (head, active row): thread = (split lane, 4 columns) and takes the splits sl, sl + lanes, ... in index
// order, kBatch loads in flight; the lanes' states meet in LDS and are added in lane order (a fixed order: deterministic).
// Heads are the fast grid axis, here and in the loop-free launches of sparse_attn_kernel: with a multiple of eight heads the
// workgroups of a head run on one XCD, whose L2 then holds the head's query rows and partial results (0.4 us of 10.9 at 32K).
// The loads do not wait for the device-side query count, which is only looked at when the row is stored, so up to
// kBatch * lanes splits (32 at d = 128) cost one memory round trip.  (A workgroup per 16 rows that walked the splits one
// after the other took 27 us at 130 splits of four heads, and as long as this one at 8.)
template <int D>
__global__ __launch_bounds__(256) void attn_combine_kernel(const float* __restrict__ part_o,
                                                           const float* __restrict__ part_ml,
                                                           const int32_t* __restrict__ counts, int max_active, int q_pad,
                                                           int n_split, uint16_t* __restrict__ out, int64_t osh, int64_t osn,
                                                           float* __restrict__ lse, float* __restrict__ lse2) {
  constexpr int kCols = D / 4, kLanes = 256 / kCols, kBatch = 4;
  __shared__ float2 ml_sh[kLanes];
  __shared__ __attribute__((aligned(16))) float o_sh[kLanes][D];
  const int a = grid_yz(), h = blockIdx.x;
  const int sl = threadIdx.x / kCols, mc = (threadIdx.x % kCols) * 4;
  const int n_act = counts ? min(max(counts[1], 0), max_active) : max_active;
  if (a >= max_active) return;  // (the grid's last slice)
  const int64_t row0 = ((int64_t)h * q_pad + a) * n_split;
  const float2* ml = reinterpret_cast<const float2*>(part_ml) + row0;
  const float* po = part_o + row0 * D + mc;
  floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, l = 0.f;
  for (int s0 = sl; s0 < n_split; s0 += kLanes * kBatch) {
    float2 v[kBatch];
    floatx4 x[kBatch];
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      const int s = s0 + u * kLanes;
      v[u] = make_float2(-INFINITY, 0.f);
      if (s < n_split) {
        v[u] = ml[s];
        x[u] = *reinterpret_cast<const floatx4*>(po + (int64_t)s * D);
      }
    }
#pragma unroll
    for (int u = 0; u < kBatch; ++u) {
      if (v[u].y > 0.f) {
        const float m_new = fmaxf(m, v[u].x);
        const float f_old = __builtin_amdgcn_exp2f(m - m_new), f = __builtin_amdgcn_exp2f(v[u].x - m_new);
        l = l * f_old + f * v[u].y;
        acc = acc * f_old + f * x[u];
        m = m_new;
      }
    }
  }
  if (mc == 0) ml_sh[sl] = make_float2(m, l);
  *reinterpret_cast<floatx4*>(&o_sh[sl][mc]) = acc;
  __syncthreads();
  if (threadIdx.x >= kCols || a >= n_act) return;  // rows past the count: their partial results were never written
  float2 lane_ml[kLanes];
  float mmax = -INFINITY;
#pragma unroll
  for (int i = 0; i < kLanes; ++i) {
    lane_ml[i] = ml_sh[i];
    mmax = fmaxf(mmax, lane_ml[i].x);
  }
  floatx4 o = floatx4{0.f, 0.f, 0.f, 0.f};
  float lsum = 0.f;
#pragma unroll
  for (int i = 0; i < kLanes; ++i) {
    const float f = lane_ml[i].y > 0.f ? __builtin_amdgcn_exp2f(lane_ml[i].x - mmax) : 0.f;
    lsum += f * lane_ml[i].y;
    o += f * *reinterpret_cast<const floatx4*>(&o_sh[i][mc]);
  }
  const float inv = lsum > 0.f ? 1.f / lsum : 0.f;
  *reinterpret_cast<uint2*>(out + (int64_t)h * osh + (int64_t)a * osn + mc) =
      make_uint2(cvt_pk_bf16(o[0] * inv, o[1] * inv), cvt_pk_bf16(o[2] * inv, o[3] * inv));
  if (mc == 0) {
    if (lse) lse[(int64_t)h * max_active + a] = lsum > 0.f ? (mmax + __builtin_amdgcn_logf(lsum)) * kLn2 : -INFINITY;
    if (lse2) lse2[(int64_t)h * q_pad + a] = lsum > 0.f ? mmax + __builtin_amdgcn_logf(lsum) : INFINITY;
  }
}

// Up to N splits: a wavefront per (head, active row), every lane with D / 64 columns of all of them: N loads, no LDS and no barrier.  The
// same operations in the same order as above, where every lane then has one split.  Bound by the one memory round trip and the
// launch.  Whole layer, above -> this way: 32 heads, 8 splits, 256 blocks 14.40 -> 14.27 us, 125 blocks 13.65 -> 13.38; d = 64, 7 splits
// 11.95 -> 11.15; 16 heads, d = 64, 14 splits 11.48 -> 11.22.  With more than 4 KB of partial results per row the single wavefront takes
// longer than four (d = 128: 16 heads, 13 splits 13.85 -> 13.94, 8 heads, 21 splits 12.8 -> 14.4), and four rows per workgroup take 0.05 more.
// Several query groups (4 heads, 252 rows: 25.7 and 26.0 us) keep the workgroup per row.
template <int D, int N>
__global__ __launch_bounds__(64) void attn_combine_few_kernel(const float* __restrict__ part_o, const float* __restrict__ part_ml,
                                                              const int32_t* __restrict__ counts, int max_active, int q_pad,
                                                              int n_split, uint16_t* __restrict__ out, int64_t osh, int64_t osn,
                                                              float* __restrict__ lse, float* __restrict__ lse2) {
  constexpr int kVec = D / 64;
  const int a = grid_yz(), h = blockIdx.x, mc = threadIdx.x * kVec;
  if (a >= max_active) return;  // (the grid's last slice)
  const int n_act = counts ? min(max(counts[1], 0), max_active) : max_active;
  const int64_t row0 = ((int64_t)h * q_pad + a) * n_split;
  const float2* ml = reinterpret_cast<const float2*>(part_ml) + row0;
  const float* po = part_o + row0 * D + mc;
  float2 v[N];
  float x[N][kVec];
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const int s = min(u, n_split - 1);
    v[u] = ml[s];
#pragma unroll
    for (int i = 0; i < kVec; ++i) x[u][i] = po[(int64_t)s * D + i];
  }
  if (a >= n_act) return;  // rows past the count: their partial results were never written
  float mmax = -INFINITY;
#pragma unroll
  for (int u = 0; u < N; ++u) {
    if (u >= n_split || !(v[u].y > 0.f)) v[u] = make_float2(-INFINITY, 0.f);
    mmax = fmaxf(mmax, v[u].x);
  }
  float o[kVec] = {}, lsum = 0.f;
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const float f = v[u].y > 0.f ? __builtin_amdgcn_exp2f(v[u].x - mmax) : 0.f;
    lsum += f * v[u].y;
#pragma unroll
    for (int i = 0; i < kVec; ++i) o[i] += f * (v[u].y > 0.f ? x[u][i] : 0.f);
  }
  const float inv = lsum > 0.f ? 1.f / lsum : 0.f;
  uint16_t* dst = out + (int64_t)h * osh + (int64_t)a * osn + mc;
  if constexpr (kVec == 2)
    *reinterpret_cast<uint32_t*>(dst) = cvt_pk_bf16(o[0] * inv, o[1] * inv);
  else
    *dst = (uint16_t)cvt_pk_bf16(o[0] * inv, 0.f);
  if (mc == 0) {
    if (lse) lse[(int64_t)h * max_active + a] = lsum > 0.f ? (mmax + __builtin_amdgcn_logf(lsum)) * kLn2 : -INFINITY;
    if (lse2) lse2[(int64_t)h * q_pad + a] = lsum > 0.f ? mmax + __builtin_amdgcn_logf(lsum) : INFINITY;
  }
}

// LOOP: the mode bits of the key loop
template <int D, int NT, int LOOP>
static void launch_wide_t(const AttnArgs& a, const SplitPlan& p, bool fused, hipStream_t st) {
  const dim3 grid = grid_list(query_group_list(p, a.H)), block(256 * NT);
  constexpr int kKeep = LOOP & 8;
  const bool many = a.n_b > 256, most = a.n_b > kFusedManyBlocks;
  if (fused && p.pipelined && most)
    WIDE_LAUNCH((wide_attn_kernel<D, NT, LOOP | 33>), grid, block, st, a);
  else if (fused && most)
    WIDE_LAUNCH((wide_attn_kernel<D, NT, kKeep | 33>), grid, block, st, a);
  else if (fused && p.pipelined && many)
    WIDE_LAUNCH((wide_attn_kernel<D, NT, LOOP | 17>), grid, block, st, a);
  else if (fused && many)
    WIDE_LAUNCH((wide_attn_kernel<D, NT, kKeep | 17>), grid, block, st, a);
  else if (fused && p.pipelined)
    WIDE_LAUNCH((wide_attn_kernel<D, NT, LOOP | 1>), grid, block, st, a);
  else if (fused)
    WIDE_LAUNCH((wide_attn_kernel<D, NT, kKeep | 1>), grid, block, st, a);
  else if (p.pipelined)
    WIDE_LAUNCH((wide_attn_kernel<D, NT, LOOP>), grid, block, st, a);
  else
    WIDE_LAUNCH((wide_attn_kernel<D, NT, kKeep>), grid, block, st, a);
}

// Few sub-tiles per head: one workgroup of more wavefronts takes them all, a sub-tile each, and there are no partial results and no launch
// that merges them (what a plan of two to four splits spends most on: a kernel boundary and a memory round trip, 3 us).  One compute unit
// then fetches the head's K and V rows, 128 KB at most (about 45 bytes a clock), and its LDS holds them: eight sub-tiles at d = 128,
// sixteen at d = 64, where the two ways meet.  Whole layer, splits -> this way: d = 64, 4 heads, 10 sub-tiles 10.8 -> 9.2 us; 32 heads, 6
// sub-tiles 11.1 -> 9.2, 13 of 256 blocks 12.0 -> 11.1, attention alone with 15 8.1 -> 8.0; 256 heads, 14 sub-tiles 16.9 -> 14.1; d = 128,
// 4 heads, 8 sub-tiles 11.9 -> 10.8, 64 heads 12.5 -> 12.0, 256 heads 19.9 -> 15.8.  More than 256 blocks (whose ranking takes every
// thread of a smaller workgroup) stay with the splits, ranked here or before: the bits of the output do not depend on that.  So do more
// heads than leave a plan with two splits (d = 64 more than 512, d = 128 more than 256): one workgroup of four wavefronts per head, with a
// key loop.  Twelve wavefronts, against sixteen for the same nine to twelve sub-tiles: 4 heads, whole layer 7.5 and 7.8 us, 32 heads 9.8 and
// 10.1, 128 heads 11.4 and 11.6, 256 heads 13.4 and 13.7.
// The probe layer goes the same way, or its output would not have the bits of the attention over all blocks (32-row tiles, heads, splits ->
// this way: d = 64, 8 tiles, 4 heads 11.8 -> 10.3 us, 11 tiles, 32 heads 15.5 -> 15.0, 16 tiles, 4 heads 12.1 -> 11.8, 32 heads 16.7 and 17.1, 128
// heads 32.0 -> 31.4; d = 128, 8 tiles, 4 heads 13.3 -> 12.8, 32 heads 16.5 -> 16.0, 128 heads 30.3 -> 29.2).
// Returns 0 for the plan's splits.  Scratch memory is asked for as for the splits.
static int one_split_waves(int head_dim, int n_b, const SplitPlan& p) {
  const int most = head_dim == 64 ? 16 : 8;
  if (p.q_tiles != 1 || p.n_split == 1 || p.pipelined || p.n_sub > most || n_b > 256) return 0;
  return p.n_sub <= 8 ? 8 : (p.n_sub <= 12 ? 12 : 16);
}
// The workgroup of one head writes its output while those of others still read their inputs, where with key splits the launch that merges
// them writes it when everyone has read everything.  Calls whose outputs share memory with an input, which the interface does not ask
// anyone to take, therefore keep the splits and give what they always gave.  (The counts are read by the merging launch, too.)
bool attention_outputs_apart(const void* Q, const int32_t* active_idx, int max_active, const void* K, const void* V, const focus_shape& s,
                             const int32_t* kept_blocks, int n_keep, const int32_t* sink_idx, int n_sink, const void* out, const float* lse) {
  const int64_t L = (int64_t)s.n_ctx + s.n_resp;
  const Extent read[] = {extent(Q, s.q_stride_h, s.q_stride_n, s.n_heads, s.n_gen, s.head_dim),
                         extent(K, s.k_stride_h, s.k_stride_n, s.n_heads, L, s.head_dim),
                         extent(V, s.v_stride_h, s.v_stride_n, s.n_heads, L, s.head_dim),
                         extent(active_idx, (int64_t)max_active * 4), extent(kept_blocks, (int64_t)n_keep * 4), extent(sink_idx, (int64_t)n_sink * 4)};
  const Extent o = extent(out, s.o_stride_h, s.o_stride_n, s.n_heads, max_active, s.head_dim), l = extent(lse, (int64_t)s.n_heads * max_active * 4);
  for (const Extent& r : read)
    if (o.meets(r) || l.meets(r)) return false;
  return true;
}
// Such a workgroup works the relevances of all heads out itself where its wavefronts do that in one go (16 blocks of a head each): a
// launch less, against one more memory round trip in this one.  Whole layer with that launch and without: d = 64, 4 heads, 16 blocks,
// 10 sub-tiles 9.2 -> 8.1 us; d = 128, 4 heads, 32 blocks, 8 sub-tiles 10.8 -> 10.4.
bool relevance_in_attention(const focus_shape& s, const SplitPlan& p) {
  const int n_b = ceil_div(s.n_ctx, s.block), waves = one_split_waves(s.head_dim, n_b, p);
  return (int64_t)s.n_heads * ceil_div(n_b, kInnerBlocks) <= waves;
}
template <int D, int WAVES>
static hipError_t launch_one_split(AttnArgs a, bool fused, hipStream_t st) {
  if (a.n_sub > WAVES) return hipErrorInvalidValue;  // no key loop: the rest would be left out
  const dim3 grid(a.H), block(64 * WAVES);
  a.n_split = 1;
  if (a.logits_out != nullptr)
    ATTN_LAUNCH((sparse_attn_kernel<D, 4, WAVES>), grid, block, st, a);
  else if (fused && a.kept_blocks != nullptr)
    ATTN_LAUNCH((sparse_attn_kernel<D, 65, WAVES>), grid, block, st, a);
  else if (fused && a.rel_per_head)
    ATTN_LAUNCH((sparse_attn_kernel<D, 9, WAVES>), grid, block, st, a);
  else if (fused)
    ATTN_LAUNCH((sparse_attn_kernel<D, 1, WAVES>), grid, block, st, a);
  else
    ATTN_LAUNCH((sparse_attn_kernel<D, 0, WAVES>), grid, block, st, a);
  return hipGetLastError();
}

template <int D>
static hipError_t launch_attn_t(const AttnArgs& a, const SplitPlan& p, bool fused, bool output_apart, hipStream_t st) {
  if (!p.pipelined && p.n_split * kWavesPerGroup < p.n_sub) return hipErrorInvalidValue;  // the loop-free variants: one sub-tile per wavefront
  if (fused && a.logits_out != nullptr) return hipErrorInvalidValue;
  const int waves = output_apart ? one_split_waves(D, a.n_b, p) : 0;
  if (fused && a.kept_blocks != nullptr && waves == 0) return hipErrorInvalidValue;
  if constexpr (D == 64) {
    if (waves == 16) return launch_one_split<D, 16>(a, fused, st);
    if (waves == 12) return launch_one_split<D, 12>(a, fused, st);
  }
  if (waves != 0) return launch_one_split<D, 8>(a, fused, st);
  const dim3 grid = p.pipelined ? dim3(p.n_split, a.H) : dim3(a.H, p.n_split), block(256);
  if (p.q_tiles_per_group > 1) {
    if (a.logits_out != nullptr) return hipErrorInvalidValue;  // logits are spilled for one 16-query tile only
    if (query_group_list(p, a.H) > kMaxList) return hipErrorInvalidValue;
    if (p.q_tiles_per_group > 2)
      launch_wide_t<D, 2, 2>(a, p, fused, st);
    else if (p.q_groups > 1)
      launch_wide_t<D, 1, 2 | 8>(a, p, fused, st);
    else
      launch_wide_t<D, 1, 2>(a, p, fused, st);
  } else if (a.logits_out != nullptr) {  // dense probe layer with the logits spilled
    if (p.pipelined)
      ATTN_LAUNCH((sparse_attn_kernel<D, 6, 4>), grid, block, st, a);
    else
      ATTN_LAUNCH((sparse_attn_kernel<D, 4, 4>), grid, block, st, a);
  } else if (fused && a.rel_per_head && a.n_b > 256) {
    if (p.pipelined && a.n_b > kFusedManyBlocks)
      ATTN_LAUNCH((sparse_attn_kernel<D, 43, 4>), grid, block, st, a);
    else if (a.n_b > kFusedManyBlocks)
      ATTN_LAUNCH((sparse_attn_kernel<D, 41, 4>), grid, block, st, a);
    else if (p.pipelined)
      ATTN_LAUNCH((sparse_attn_kernel<D, 27, 4>), grid, block, st, a);
    else
      ATTN_LAUNCH((sparse_attn_kernel<D, 25, 4>), grid, block, st, a);
  } else if (fused && p.pipelined && a.n_b > kFusedManyBlocks)
    ATTN_LAUNCH((sparse_attn_kernel<D, 35, 4>), grid, block, st, a);
  else if (fused && a.n_b > kFusedManyBlocks)
    ATTN_LAUNCH((sparse_attn_kernel<D, 33, 4>), grid, block, st, a);
  else if (fused && p.pipelined && a.n_b > 256)
    ATTN_LAUNCH((sparse_attn_kernel<D, 19, 4>), grid, block, st, a);
  else if (fused && a.n_b > 256)
    ATTN_LAUNCH((sparse_attn_kernel<D, 17, 4>), grid, block, st, a);
  else if (fused && p.pipelined && a.rel_per_head)
    ATTN_LAUNCH((sparse_attn_kernel<D, 11, 4>), grid, block, st, a);
  else if (fused && p.pipelined)
    ATTN_LAUNCH((sparse_attn_kernel<D, 3, 4>), grid, block, st, a);
  else if (fused && a.rel_per_head)
    ATTN_LAUNCH((sparse_attn_kernel<D, 9, 4>), grid, block, st, a);
  else if (fused)
    ATTN_LAUNCH((sparse_attn_kernel<D, 1, 4>), grid, block, st, a);
  else if (p.pipelined)
    ATTN_LAUNCH((sparse_attn_kernel<D, 2, 4>), grid, block, st, a);
  else
    ATTN_LAUNCH((sparse_attn_kernel<D, 0, 4>), grid, block, st, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || p.n_split == 1) return e;
  if (p.q_groups == 1 && p.n_split <= 8)
    hipLaunchKernelGGL((attn_combine_few_kernel<D, 8>), grid_x_yz(a.H, a.max_active), dim3(64), 0, st, a.part_o, a.part_ml, a.counts, a.max_active,
                       a.q_pad, a.n_split, a.out, a.osh, a.osn, a.lse, a.lse2_out);
  else if (p.q_groups == 1 && p.n_split * D <= 1024)  // (d = 64)
    hipLaunchKernelGGL((attn_combine_few_kernel<D, 1024 / D>), grid_x_yz(a.H, a.max_active), dim3(64), 0, st, a.part_o, a.part_ml, a.counts, a.max_active,
                       a.q_pad, a.n_split, a.out, a.osh, a.osn, a.lse, a.lse2_out);
  else
    hipLaunchKernelGGL(attn_combine_kernel<D>, grid_x_yz(a.H, a.max_active), dim3(256), 0, st, a.part_o, a.part_ml, a.counts, a.max_active,
                       a.q_pad, a.n_split, a.out, a.osh, a.osn, a.lse, a.lse2_out);
  return hipGetLastError();
}

hipError_t launch_sparse_attn(const void* Q, const int32_t* active_idx, const int32_t* counts, int max_active,
                              const void* K, const void* V, const focus_shape& s, const int32_t* kept_blocks, int n_keep,
                              const int32_t* sink_idx, int n_sink, const SplitPlan& p, void* out, float* lse,
                              float* part_o, float* part_ml, const FusedTopC* fused, hipStream_t st,
                              const DenseProbe* probe) {
  if (max_active < 1) return hipErrorInvalidValue;
  AttnArgs a;
  a.dense_rows = probe ? s.n_ctx + s.n_resp : 0;
  a.logits_out = probe ? probe->logits_out : nullptr;
  a.lse2_out = probe ? probe->lse2_out : nullptr;
  a.Q = static_cast<const uint16_t*>(Q);
  a.K = static_cast<const uint16_t*>(K);
  a.V = static_cast<const uint16_t*>(V);
  a.active_idx = active_idx;
  a.counts = counts;
  a.kept_blocks = kept_blocks;
  a.sink_idx = sink_idx;
  a.out = static_cast<uint16_t*>(out);
  a.lse = lse;
  a.part_o = part_o;
  a.part_ml = part_ml;
  a.qsh = s.q_stride_h; a.qsn = s.q_stride_n;
  a.ksh = s.k_stride_h; a.ksn = s.k_stride_n;
  a.vsh = s.v_stride_h; a.vsn = s.v_stride_n;
  a.osh = s.o_stride_h; a.osn = s.o_stride_n;
  a.H = s.n_heads; a.M = s.n_ctx; a.N = s.n_resp; a.B = s.block;
  a.n_b = ceil_div(s.n_ctx, s.block);
  a.n_gen = s.n_gen; a.n_keep = n_keep; a.n_sink = n_sink; a.max_active = max_active;
  a.sub_per_block = ceil_div(s.block, kSubTile);
  a.n_sub = p.n_sub; a.n_split = p.n_split; a.q_pad = p.q_pad;
  a.q_groups = p.q_groups;
  a.scale_log2 = kLog2e / sqrtf((float)s.head_dim);
  a.head_turn = 0xffffffffu / (uint32_t)s.n_heads;
  a.split_rounds = ceil_div(p.n_sub, kWavesPerGroup) / p.n_split;
  a.split_rounds_more = ceil_div(p.n_sub, kWavesPerGroup) % p.n_split;
  if (fused) a.kept_blocks = fused->kbar ? fused->focus_idx : nullptr;
  a.rel_part = fused ? (fused->kbar ? fused->kbar : fused->rel_part) : nullptr;
  a.rel_per_head = fused && fused->per_head;
  a.scores_out = fused ? fused->scores_out : nullptr;
  a.kept_out = fused ? fused->kept_out : nullptr;
  a.n_focus_max = fused ? fused->n_focus_max : 0;
  const bool apart = attention_outputs_apart(Q, active_idx, max_active, K, V, s, kept_blocks, n_keep, sink_idx, n_sink, out, lse);
  return s.head_dim == 128 ? launch_attn_t<128>(a, p, fused != nullptr, apart, st) : launch_attn_t<64>(a, p, fused != nullptr, apart, st);
}

// =====================================================================================================
// Block-entry refresh (Alg. 1, I_active = all positions): dense bidirectional attention of EVERY row of Q over every
// key — the one MFMA-bound launch of the method (4 n_q L d flops per head against 2 L d 2 bytes of K and V).
// A workgroup holds 256 consecutive queries, 32 per wavefront, and walks the key axis in 32-row sub-tiles shared by
// its eight wavefronts.  LDS holds a ring of eight K and eight V sub-tiles: while four are multiplied the other four are
// filled, one per iteration through registers, and there is one barrier per four sub-tiles — behind a barrier all wavefronts
// wait for their first operands at the same time and neither the matrix cores nor the vector ALU have work, and between
// barriers the two wavefronts of a SIMD drift apart, so that the vector work of one runs beside the MFMAs of the other.
// (32 heads, 8192 rows: 1052 us with a barrier per sub-tile, 1018 with one per four on normal-distributed data, 830 and 746
// on zeros: the difference between the two kinds of data is the chip's power limit.)  Both products use the 32x32x16 MFMA:
//   S^T = K Q^T   lane (query = lane % 32, hh = lane / 32) register v holds the logit of key 8 (v / 4) + 4 hh + v % 4,
//                 so a query's 32 logits sit in two lanes and the row maximum costs one cross-lane exchange;
//   O^T = V^T P^T the same registers, packed to bf16 eight at a time, are the B operand of k-step s = v / 8; the A
//                 operand is read transposed from the row-major staged V with the key slots in that same order.
// The loop is bound by the vector ALU (exp2 and the multiply-adds around it), so everything else is kept out of it:
// row addresses are one scalar base per sub-tile plus per-lane offsets computed once, the running sum is taken by
// v_dot2 over the packed bf16 pairs (two values per instruction, and the very values that enter the PV product),
// the rescale of O runs only when some running maximum in the wavefront moved, and the ragged last sub-tile has a
// loop body of its own.  No index lists, no key splits across workgroups: each normalises and writes its own rows.
// One-dimensional grid over the (head, query block) list, dealt to the XCDs in contiguous eighths (see the kernel).
// PARTS = 2: a half block of 128 queries.  Four wavefronts carry its tiles over the even key sub-tiles, four over the odd ones, each four with
// rings of their own (half as long: a barrier per two sub-tiles), and the two states of a tile are added at the end.  (PARTS = 4: a quarter, 64
// queries, every fourth sub-tile, a barrier each.)  A
// workgroup then fetches and stores twice the rows per product and takes 0.60 us where a block takes 1.04 (32-row sub-tile of 256 workgroups at
// d = 128, 8192 keys), which is less than an empty half of a round costs.  LSE: the log-sum-exps are wanted; they are then those of the unrounded sums.
// The queries that would leave a round of workgroups mostly empty go there or to refresh_tail_kernel (cut_refresh).
// COPY: the workgroups behind those of the items make the layer's cache refresh, where this is the layer's last attention launch, instead of a
// launch of their own (which short prompts feel: block entry, 32 heads, 1160 rows 51.6 -> 42.9 us, 8192 rows 1032 -> 1020; 8 heads, 5823 rows
// 165 -> 155; d = 64: 32 heads, 1811 rows 49.5 -> 45.7, 8 heads, 14 913 rows 514 -> 504).  At d = 64 the rows of K and V are requested one after the
// other: both at once take the registers of a second workgroup (14 913 rows 525).
// =====================================================================================================
struct RefreshArgs {
  const uint16_t* Q;
  const uint16_t* K;
  const uint16_t* V;
  uint16_t* out;
  float* lse;  // [H, n_q] natural log, or null
  int64_t qsh, qsn, ksh, ksn, vsh, vsn, osh, osn;
  int n_q, L;
  int n_qb, n_work;    // whole query blocks per head; work items (head, query block) of refresh_attn_kernel
  int n_heads, n_tail;  // query tiles left to refresh_tail_kernel
  // parts of blocks (refresh_attn_kernel<., 2 | 4, .>), of part_tiles tiles: so many of whole blocks, then so many of every head's last tiles
  int n_part_whole, n_part_head, part_tiles;
  float scale_log2;
};

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>): a loop whose index is a constant expression
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F>
__device__ __forceinline__ void static_for(F&& f) {
  static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// keeps the computation of x in front of this point (and of the scheduling fences after it)
__device__ __forceinline__ void pin(float& x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ void pin(int& x) { asm volatile("" : "+v"(x)); }

// Eight wavefronts of 32 queries: two per SIMD, and 256 queries share every staged sub-tile.  (Four wavefronts of 64 queries —
// each LDS operand feeding two MFMAs, one wavefront per SIMD with 444 registers — gives the same sharing with half the LDS
// reads, but a lone wavefront cannot cover its own dependent vector-ALU chains: 0.82 against 1.01 PFLOP/s.)
constexpr int kRefreshWaves = 8;  // wavefronts per workgroup
constexpr int kRefreshBlock = 4;  // sub-tiles between two barriers

template <int D, int PARTS, bool LSE, bool COPY>
__global__ __launch_bounds__(64 * kRefreshWaves, 2) void refresh_attn_kernel(const RefreshArgs p, const CacheRefresh copy) {
  using G = Geo<D>;
  constexpr int kKS = D / 16;                    // k-steps of K Q^T
  constexpr int kDT = D / 32;                    // 32-wide d tiles of V^T P^T
  constexpr int NB = kRefreshBlock / PARTS, kRing = 2 * NB;
  constexpr int kPartWaves = kRefreshWaves / PARTS;  // query tiles of a workgroup
  constexpr int kShare = kPartWaves / 2;         // wavefronts that share the K (or the V) rows of a sub-tile
  constexpr int NL = G::kLoads / kShare;         // loads per wavefront and sub-tile
  static_assert(G::kLoads % kShare == 0 && NL >= 1, "every wavefront stages at least one load");
  // K sub-tile j sits in slot (j - 1) mod kRing of its ring, V sub-tile j in slot j mod kRing: iteration t reads slot t mod kRing of both
  __shared__ __attribute__((aligned(16))) char ringsK[PARTS * kRing * G::kStageBytes];
  __shared__ __attribute__((aligned(16))) char ringsV[PARTS * kRing * G::kStageBytes];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int part = PARTS == 1 ? 0 : wave / kPartWaves, tile = PARTS == 1 ? wave : wave % kPartWaves;
  const int qi = lane & 31, hh = lane >> 5;
  // Workgroups are handed to the 8 XCDs round-robin in launch order, and each XCD has its own L2.  Launch slot i is
  // therefore given work item (i % 8) * chunk + i / 8 of the (head, query block) list: an XCD walks one contiguous
  // eighth of the list, so the workgroups resident on it at any time are neighbouring query blocks of ONE head and
  // stream the same K/V rows through its L2 together.
  const int n_items = PARTS == 1 ? p.n_work : p.n_part_whole + p.n_part_head * p.n_heads;
  const int chunk = (n_items + 7) >> 3;
  if (COPY && (int)blockIdx.x >= 8 * chunk) {  // the layer's cache refresh on the side, as in refresh_tail_kernel
    const int half = threadIdx.x >> 8, item = 2 * ((int)blockIdx.x - 8 * chunk) + half;
    const bool live = item < copy.n_chunks * copy.n_heads;
    const int ch = live ? item / copy.n_chunks : 0;
    static_assert(2 * 2048 * sizeof(float) <= sizeof(ringsK), "both halves' partial means fit");
    cache_refresh_chunk<D, D == 128>(copy, live ? item - ch * copy.n_chunks : 0, ch, threadIdx.x & 255, live, reinterpret_cast<float*>(ringsK) + half * 2048);
    return;
  }
  const int work = (int)(blockIdx.x & 7u) * chunk + (int)(blockIdx.x >> 3);
  if (work >= n_items) return;  // whole workgroup
  int h, tile0;  // first query tile
  if (PARTS == 1) {
    h = work / p.n_qb;
    tile0 = (work - h * p.n_qb) * kRefreshWaves;
  } else if (work < p.n_part_whole) {
    const int block = p.n_work + work / PARTS;
    h = block / p.n_qb;
    tile0 = (block - h * p.n_qb) * kRefreshWaves + work % PARTS * kPartWaves;
  } else {
    const int i = work - p.n_part_whole;
    h = i / p.n_part_head;
    tile0 = p.n_qb * kRefreshWaves + (i - h * p.n_part_head) * kPartWaves;
  }
  const int q_row = (tile0 + tile) * 32 + qi;
  // Sub-tiles: n_keys of the head; a part takes those with its remainder mod PARTS, n_tiles for each of them (one may be past the end)
  const int n_keys = (p.L + kSubTile - 1) / kSubTile;
  const int n_tiles = (n_keys + PARTS - 1) / PARTS;
  const int n_full = p.L / kSubTile;
  char* ringK = ringsK + part * (kRing * G::kStageBytes);
  char* ringV = ringsV + part * (kRing * G::kStageBytes);

  // this wavefront's share of every sub-tile: the first half of the wavefronts split the K rows, the second half the
  // V rows.  Row addresses: a scalar base that moves by 32 rows per sub-tile plus per-lane byte offsets fixed for the launch.
  const bool is_v = tile >= kShare;
  const int first = (tile % kShare) * NL;
  const char* src = reinterpret_cast<const char*>(is_v ? p.V + (int64_t)h * p.vsh : p.K + (int64_t)h * p.ksh);
  const int64_t row_bytes = (is_v ? p.vsn : p.ksn) * 2;
  const int64_t tile_bytes = row_bytes * kSubTile;
  auto swz = [&](int slot) { return is_v ? vstage_swz<D>(slot) : (slot & (G::kChunks - 1)); };  // chunk permutation of a staged row
  uint32_t voff[NL];
#pragma unroll
  for (int i = 0; i < NL; ++i) {
    const int slot = (first + i) * G::kRowsPerLoad + lane / G::kChunks;
    voff[i] = (uint32_t)slot * (uint32_t)row_bytes + (((lane % G::kChunks) ^ swz(slot)) << 4);
  }
  const int lead_k = is_v ? 0 : 1;
  // element e = sub-tile e + 1 of K, sub-tile e of V: what ring slot e mod kRing holds
  auto fetch = [&](int e, uintx4 (&r)[NL]) __attribute__((always_inline)) {
    int t = (e + lead_k) * PARTS + part;
    if (PARTS > 1) t = min(t, n_keys - 1);  // past the end: any rows of the key set, all masked
    const char* base = src + (int64_t)t * tile_bytes;
    if (t >= n_full) {  // the ragged last sub-tile: slots past the end read its last row instead (masked below)
      const int last = p.L - t * kSubTile - 1;
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const int slot = (first + i) * G::kRowsPerLoad + lane / G::kChunks;
        voff[i] = (uint32_t)min(slot, last) * (uint32_t)row_bytes + (((lane % G::kChunks) ^ swz(slot)) << 4);
      }
    }
#pragma unroll
    for (int i = 0; i < NL; ++i) r[i] = __builtin_nontemporal_load(reinterpret_cast<const uintx4*>(base + voff[i]));
  };
  char* my_ring = (is_v ? ringV : ringK) + first * 1024 + lane * 16;
  auto store = [&](int slot, const uintx4 (&r)[NL]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < NL; ++i) *reinterpret_cast<uintx4*>(my_ring + slot * G::kStageBytes + i * 1024) = r[i];
  };
  auto exists = [&](int e) { return e + lead_k < n_tiles; };

  // prologue: K sub-tile 0 (element -1) and the first block of elements, all requested at once
  uintx4 r[NL];
  {
    uintx4 pr[NB + 1][NL];
    if (!is_v) fetch(-1, pr[NB]);
#pragma unroll
    for (int e = 0; e < NB; ++e)
      if (exists(e)) fetch(e, pr[e]);
    if (exists(NB)) fetch(NB, r);
    if (!is_v) store(kRing - 1, pr[NB]);
#pragma unroll
    for (int e = 0; e < NB; ++e)
      if (exists(e)) store(e, pr[e]);
  }
  bf16x8 q[kKS];  // B operand of K Q^T: lane (query, hh) holds Q[query][16 ks + 8 hh .. + 7]
  {
    const uint16_t* qsrc = p.Q + (int64_t)h * p.qsh + (int64_t)min(q_row, p.n_q - 1) * p.qsn + hh * 8;
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks) {
      const uint4 v = *reinterpret_cast<const uint4*>(qsrc + ks * 16);
      q[ks] = as_bf16x8(q_row < p.n_q ? v : make_uint4(0u, 0u, 0u, 0u));
    }
  }
  // Below every finite scaled logit (the scale is less than one) but finite itself: keys with a logit of -inf, all that a lane may have seen so far,
  // then get a probability of 0 and an alpha of 1 or 0, where a maximum of -inf would give NaN.
  float m_run = -FLT_MAX, l_run = 0.f;   // l_run: this lane's share of the row sum (its 16 of every 32 keys)
  float u_run = 0.f;                     // LSE: the same of the probabilities before they are rounded
  floatx16 o[kDT];
#pragma unroll
  for (int dt = 0; dt < kDT; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[dt][v] = 0.f;
  int koff[kKS];  // byte offset of the K operand of k-step s within a slot
#pragma unroll
  for (int s = 0; s < kKS; ++s) {
    koff[s] = stage_off<D>(qi, 2 * s + hh);
    pin(koff[s]);
  }
  int vaddr[kDT];  // LDS address of the V operand of d tile dt in slot 0 (read_v_operand32)
#pragma unroll
  for (int dt = 0; dt < kDT; ++dt) {
    const int row = 4 * (lane >> 5) + ((lane & 15) >> 2), col = 32 * dt + 16 * ((lane >> 4) & 1) + 4 * (lane & 3);
    vaddr[dt] = (int)lds_address(ringV) + vstage_off<D>(row, col >> 3) + (col & 7) * 2;
    pin(vaddr[dt]);
  }
  auto v_operand = [&](int slot, int dt, int ks) __attribute__((always_inline)) {  // rows 16 ks, 16 ks + 8 further: the same swizzle
    typedef shortx4 __attribute__((address_space(3))) * lds_ptr;
    const uint32_t at = (uint32_t)(vaddr[dt] + slot * G::kStageBytes + 16 * ks * G::kRowBytes);
    struct { shortx4 a, b; } both = {__builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(uintptr_t)at),
                                     __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(uintptr_t)(at + 8 * G::kRowBytes))};
    return __builtin_bit_cast(bf16x8, both);
  };
  // scaled row maximum of one sub-tile's logits.  Slots past the end of a ragged sub-tile hold copies of its last
  // row, so they cannot raise the maximum and need no masking here.
  auto row_max_lane = [&](const floatx16& a) __attribute__((always_inline)) {
    float mx = fmaxf(a[0], a[1]);
#pragma unroll
    for (int v = 2; v < 16; ++v) mx = fmaxf(mx, a[v]);
    return mx;
  };
  auto row_max = [&](float mx) __attribute__((always_inline)) {
    const uintx2 sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
    return fmaxf(__uint_as_float(sw.x), __uint_as_float(sw.y)) * p.scale_log2;
  };
  auto rescale = [&](float mx) __attribute__((always_inline)) {
    if (__ballot(mx > m_run) != 0ull) {  // some running maximum of this wavefront moves (rare after the first sub-tiles)
      const float m_new = fmaxf(m_run, mx);
      const float alpha = __builtin_amdgcn_exp2f(m_run - m_new);  // 0 where m_new is the first finite logit
      m_run = m_new;
      l_run *= alpha;
      if (LSE) u_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < kDT; ++dt) o[dt] *= alpha;
    }
  };

  __syncthreads();
  floatx16 acc;
  float mx;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
  for (int ks = 0; ks < kKS; ++ks) {
    const bf16x8 a = as_bf16x8(*reinterpret_cast<const uint4*>(ringK + (kRing - 1) * G::kStageBytes + koff[ks]));
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, q[ks], acc, 0, 0, 0);
  }
  mx = row_max(row_max_lane(acc));

  // One iteration, written as NS slots of one LDS operand and one MFMA each — K Q^T of sub-tile t + 1 first, then
  // V^T P^T of sub-tile t — with scheduling fences between the slots: a wavefront issues in order, so the vector work
  // of the other sub-tile (exponentials of sub-tile t beside the first MFMAs, the row maximum of sub-tile t + 1 beside
  // the last ones) has to sit between the MFMAs in program order or it would wait behind all of them.  The
  // LDS operand of slot s + kLead is requested in slot s, across iterations within a block.  n_valid < 32 only in the last
  // iteration (kLast), which has no K Q^T part.
  constexpr int NS = kKS + 2 * kDT;             // operand slots per iteration
  constexpr int kLead = 3;
  bf16x8 ahead[kLead];                          // operands of the next iteration's first slots
  // R: ring slot of this iteration, or -1: t mod kRing.  kFirst: first of a block, behind the barrier.  kMore: the next iteration belongs to the same block.
  auto body = [&](int t, auto slot_tag, auto first_tag, auto more_tag, auto last_tag, int n_valid) __attribute__((always_inline)) {
    constexpr int R = decltype(slot_tag)::value;
    constexpr bool kFirst = decltype(first_tag)::value, kMore = decltype(more_tag)::value, kLast = decltype(last_tag)::value;
    constexpr int S0 = kLast ? kKS : 0;           // first slot of this iteration
    if (kFirst) __syncthreads();                  // the block is staged; everyone is done with the previous one
    rescale(mx);
    const int ring = R >= 0 ? R : (t & (kRing - 1));
    const char* sK = ringK + ring * G::kStageBytes;
    bf16x8 op[NS + kLead];
    auto read_op = [&](auto sc) __attribute__((always_inline)) {
      constexpr int s = decltype(sc)::value;
      if constexpr (s < kKS)
        op[s] = as_bf16x8(*reinterpret_cast<const uint4*>(sK + koff[s]));
      else if constexpr (s < NS)
        op[s] = v_operand(ring, (s - kKS) % kDT, (s - kKS) / kDT);
      else if constexpr (kMore)
        ahead[s - NS] = as_bf16x8(*reinterpret_cast<const uint4*>(sK + G::kStageBytes + koff[s - NS]));
    };
    floatx16 next;
    uint32_t pk[8];
    float mxn = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) next[v] = 0.f;
    auto probabilities = [&](int v0, int v1) __attribute__((always_inline)) {  // logits v0 .. v1 - 1 -> packed bf16, added to the row sum
#pragma unroll
      for (int v = v0; v < v1; v += 2) {
        float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[v], p.scale_log2, -m_run));
        float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(acc[v + 1], p.scale_log2, -m_run));
        if (kLast) {  // a ragged sub-tile: slots past the end count for nothing
          const int key = 8 * (v >> 2) + 4 * hh + (v & 3);
          p0 = key < n_valid ? p0 : 0.f;
          p1 = key + 1 < n_valid ? p1 : 0.f;
        }
        pk[v >> 1] = cvt_pk_bf16(p0, p1);
        l_run = add_bf16_pair(l_run, pk[v >> 1]);
        if (LSE) u_run += p0 + p1;
      }
    };
    if (kLast) probabilities(0, 16);
    if constexpr (kFirst) {
      static_for<kLead>([&](auto sc) { read_op(std::integral_constant<int, decltype(sc)::value + S0>{}); });
    } else {
#pragma unroll
      for (int i = 0; i < kLead; ++i) op[i] = ahead[i];
    }
    __builtin_amdgcn_sched_barrier(0);
    static_for<NS - S0>([&](auto sc) {
      constexpr int s = decltype(sc)::value + S0;
      read_op(std::integral_constant<int, s + kLead>{});
      if constexpr (s < kKS) {
        next = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[s], q[s], next, 0, 0, 0);
      } else {
        constexpr int ks = (s - kKS) / kDT, dt = (s - kKS) % kDT;
        const bf16x8 pb = as_bf16x8(make_uint4(pk[4 * ks], pk[4 * ks + 1], pk[4 * ks + 2], pk[4 * ks + 3]));
        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[s], pb, o[dt], 0, 0, 0);
      }
      if constexpr (!kLast) {
        if constexpr (s < kKS + kDT) {  // pair i of the logits of sub-tile t: slot i (kKS + kDT) / 8
          static_for<8>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            if constexpr (i * (kKS + kDT) / 8 == s) {
              probabilities(2 * i, 2 * i + 2);
              pin(l_run);
            }
          });
        }
        if constexpr (s == kKS) {  // element t + NB to its slot, then request the one after
          if (exists(t + NB)) {
            store(R >= 0 ? (R + NB) % kRing : ((t + NB) & (kRing - 1)), r);
            if (exists(t + NB + 1)) fetch(t + NB + 1, r);
          }
        }
        if constexpr (s == NS - 3) mxn = row_max_lane(next);
        if constexpr (s == NS - 2) mxn = row_max(mxn);
      }
      __builtin_amdgcn_sched_barrier(0);
    });
    if (!kLast) {
      mx = mxn;
      acc = next;
    }
  };
  using std::integral_constant;
  constexpr std::false_type no{};
  constexpr std::true_type yes{};
  const int n_iter = n_tiles - 1;
  int t = 0;
  for (; t + kRing <= n_iter; t += kRing)  // straight-line: both halves of the rings
    static_for<kRing>([&](auto ic) {
      constexpr int i = decltype(ic)::value;
      body(t + i, integral_constant<int, i>{}, integral_constant<bool, i % NB == 0>{}, integral_constant<bool, i % NB != NB - 1>{}, no, kSubTile);
    });
  for (; t < n_iter; ++t) body(t, integral_constant<int, -1>{}, yes, no, no, kSubTile);
  // last sub-tile (possibly ragged): its logits are in acc already
  const int n_last = p.L - ((n_tiles - 1) * PARTS + part) * kSubTile;
  if (PARTS == 1 || n_last > 0)  // wave-uniform
    body(n_tiles - 1, integral_constant<int, -1>{}, yes, no, yes, n_last);
  else
    __syncthreads();  // (body's)

  // lane (query, hh) register v of d tile dt holds O^T[32 dt + 8 (v / 4) + 4 hh + v % 4][query]: four consecutive
  // output columns per register quad.  The two lanes of a query add their halves of the row sum.
  const uintx2 sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_run), __float_as_uint(l_run), false, false);
  float l = __uint_as_float(sw.x) + __uint_as_float(sw.y), l_exact = l;
  if (LSE) {
    const uintx2 uw = __builtin_amdgcn_permlane32_swap(__float_as_uint(u_run), __float_as_uint(u_run), false, false);
    l_exact = __uint_as_float(uw.x) + __uint_as_float(uw.y);
  }
  if constexpr (PARTS > 1) {  // the parts of a tile hold the same elements in the same lanes: through LDS, 16 bytes of a lane at a time
    constexpr int kPartBytes = kPartWaves * 32 * D * 4;
    static_assert(PARTS / 2 * kPartBytes <= (int)sizeof(ringsK) && (PARTS / 2 - 1) * kPartBytes + (PARTS - 1) * kPartWaves * 64 * 16 <= (int)sizeof(ringsV), "the parts fit");
    auto o_of = [&](int other) __attribute__((always_inline)) {  // parts 1 .. PARTS / 2 in the place of the K rings, the others in that of the V rings
      char* at = other <= PARTS / 2 ? ringsK + (other - 1) * kPartBytes : ringsV + (other - 1 - PARTS / 2) * kPartBytes;
      return reinterpret_cast<floatx4*>(at) + tile * (32 * D / 4) + lane;
    };
    auto ml_of = [&](int other) __attribute__((always_inline)) {
      return reinterpret_cast<floatx4*>(ringsV + (PARTS / 2 - 1) * kPartBytes) + ((other - 1) * kPartWaves + tile) * 64 + lane;
    };
    __syncthreads();  // the rings have been read by everyone
    if (part != 0) {
      floatx4* dst = o_of(part);
#pragma unroll
      for (int i = 0; i < 4 * kDT; ++i)
        dst[64 * i] = floatx4{o[i >> 2][4 * (i & 3)], o[i >> 2][4 * (i & 3) + 1], o[i >> 2][4 * (i & 3) + 2], o[i >> 2][4 * (i & 3) + 3]};
      *ml_of(part) = floatx4{m_run, l, l_exact, 0.f};
    }
    __syncthreads();
    if (part != 0) return;
    floatx4 ml[PARTS];
    ml[0] = floatx4{m_run, l, l_exact, 0.f};
    float f[PARTS];
#pragma unroll
    for (int w = 1; w < PARTS; ++w) {
      ml[w] = *ml_of(w);
      m_run = fmaxf(m_run, ml[w][0]);
    }
    l = 0.f;
    l_exact = 0.f;
#pragma unroll
    for (int w = 0; w < PARTS; ++w) {
      f[w] = ml[w][1] > 0.f ? __builtin_amdgcn_exp2f(ml[w][0] - m_run) : 0.f;
      l += f[w] * ml[w][1];
      l_exact += f[w] * ml[w][2];
    }
#pragma unroll
    for (int i = 0; i < 4 * kDT; ++i) {
      floatx4 x = floatx4{o[i >> 2][4 * (i & 3)], o[i >> 2][4 * (i & 3) + 1], o[i >> 2][4 * (i & 3) + 2], o[i >> 2][4 * (i & 3) + 3]} * f[0];
#pragma unroll
      for (int w = 1; w < PARTS; ++w) x += f[w] * o_of(w)[64 * i];
#pragma unroll
      for (int j = 0; j < 4; ++j) o[i >> 2][4 * (i & 3) + j] = x[j];
    }
  }
  if (q_row < p.n_q) {
    const float inv = l > 0.f ? 1.f / l : 0.f;
    uint16_t* dst = p.out + (int64_t)h * p.osh + (int64_t)q_row * p.osn + 4 * hh;
#pragma unroll
    for (int dt = 0; dt < kDT; ++dt)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        *reinterpret_cast<uint2*>(dst + 32 * dt + 8 * j) = make_uint2(cvt_pk_bf16(o[dt][4 * j] * inv, o[dt][4 * j + 1] * inv),
                                                                      cvt_pk_bf16(o[dt][4 * j + 2] * inv, o[dt][4 * j + 3] * inv));
    if ((PARTS == 1 || LSE) && p.lse && hh == 0)
      p.lse[(int64_t)h * p.n_q + q_row] = l_exact > 0.f ? (m_run + __builtin_amdgcn_logf(l_exact)) * kLn2 : -INFINITY;
  }
}

// The query tiles that refresh_attn_kernel does not take (see cut_refresh): one 32-query tile per workgroup, the
// key sub-tiles dealt to its eight wavefronts in turn.  A wavefront stages its own sub-tiles (no barrier in the key loop; the
// operands are all in registers before the next sub-tile is requested into the same stage), the eight states are merged at the
// end.  Tail tiles: those of whole blocks that the other kernel does not take, then every head's last few tiles.
// Rows are normalised as in refresh_attn_kernel, by the sum of the rounded probabilities (the quotient is then a weighted mean of V
// rows, and a common offset of V cancels in its rounding error: with V = 4 + noise that error is a quarter of what the unrounded sum
// leaves).  The log-sum-exp, in which nothing cancels, is that of the unrounded sum; LSE: it is wanted.
// The workgroups behind those of the tail tiles make the layer's cache refresh, two chunks each (copy; none without it): the tiles
// rarely fill the chip and leave the memory idle, while the copy needs nothing else.  32 heads: 8256 rows, tiles 77 us and copy 48
// us one after the other, 32 832 rows 282 and 185; 4 heads, 1056 rows, d = 64: a launch less.
// Bound by the vector ALU: a sub-tile of a tile takes a wavefront about a thousand cycles.  d = 64: O is rescaled for every sub-tile, which takes
// 90 register moves and 30 registers less than doing it where a maximum has moved, so that two workgroups fit a compute unit.  Block
// entry: 4 heads, 1056 rows 10.1 -> 9.5 us; 8 heads, 1056 rows 16.7 -> 13.8; 16 heads, 1532 rows 32.5 -> 25.3; 4 heads, 6032 rows 84 -> 67.
template <int D, bool LSE>
__global__ __launch_bounds__(64 * kRefreshWaves, D == 64 ? 4 : 2) void refresh_tail_kernel(const RefreshArgs p, const CacheRefresh copy) {
  using G = Geo<D>;
  constexpr int kKS = D / 16, kDT = D / 32, kOChunks = D / 4;
  constexpr int kBufBytes = 2 * G::kStageBytes;
  __shared__ __attribute__((aligned(16))) char lds[kRefreshWaves * kBufBytes];
  __shared__ float2 mr_sh[kRefreshWaves][32];  // running maximum, sum of the rounded probabilities
  __shared__ float l_sh[LSE ? kRefreshWaves : 1][32];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qi = lane & 31, hh = lane >> 5;
  const int n_tail_groups = (p.n_tail + 7) & ~7;
  if ((int)blockIdx.x >= n_tail_groups) {
    const int half = threadIdx.x >> 8, item = 2 * ((int)blockIdx.x - n_tail_groups) + half;
    const bool live = item < copy.n_chunks * copy.n_heads;
    const int h = live ? item / copy.n_chunks : 0;
    static_assert(2 * 2048 * sizeof(float) <= sizeof(lds), "both halves' partial means fit");
    cache_refresh_chunk<D>(copy, live ? item - h * copy.n_chunks : 0, h, threadIdx.x & 255, live, reinterpret_cast<float*>(lds) + half * 2048);
    return;
  }
  // contiguous eighths of the tile list to the XCDs, as in refresh_attn_kernel
  const int chunk = (p.n_tail + 7) >> 3;
  const int item = (int)(blockIdx.x & 7u) * chunk + (int)(blockIdx.x >> 3);
  if (item >= p.n_tail) return;  // whole workgroup
  const int done = p.n_work * kRefreshWaves + p.n_part_whole * p.part_tiles;  // tiles of whole blocks: taken, and left
  const int n_left = p.n_heads * p.n_qb * kRefreshWaves - done;
  int h, tile;
  if (item < n_left) {
    const int block = (done + item) / kRefreshWaves;
    h = block / p.n_qb;
    tile = done + item - h * p.n_qb * kRefreshWaves;
  } else {
    const int first = p.n_qb * kRefreshWaves + p.n_part_head * p.part_tiles, per_head = (p.n_q + 31) / 32 - first;
    h = (item - n_left) / per_head;
    tile = first + (item - n_left) - h * per_head;
  }
  const uint16_t* Kh = p.K + (int64_t)h * p.ksh;
  const uint16_t* Vh = p.V + (int64_t)h * p.vsh;
  const int n_tiles = (p.L + kSubTile - 1) / kSubTile;
  char* stage = lds + wave * kBufBytes;
  auto tile_of = [&](int t) __attribute__((always_inline)) {
    SubTile s;
    s.kind = 0;
    s.sink_row = 0;
    s.row0 = t * kSubTile;
    s.vmask = low_mask(p.L - s.row0);
    return s;
  };
  auto request = [&](int t) __attribute__((always_inline)) {
    const SubTile s = tile_of(t);
    issue_subtile<D, false, 0>(Kh, p.ksn, s, stage, lane);
    issue_subtile<D, true, 0>(Vh, p.vsn, s, stage + G::kStageBytes, lane);
  };
  if (wave < n_tiles) request(wave);
  const int q_row = tile * 32 + qi;
  bf16x8 q[kKS];
  {
    const uint16_t* qsrc = p.Q + (int64_t)h * p.qsh + (int64_t)min(q_row, p.n_q - 1) * p.qsn + hh * 8;
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks) q[ks] = as_bf16x8(*reinterpret_cast<const uint4*>(qsrc + ks * 16));
  }
  float m_run = -INFINITY, l_run = 0.f, r_run = 0.f;
  floatx16 o[kDT];
#pragma unroll
  for (int dt = 0; dt < kDT; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[dt][v] = 0.f;
  for (int t = wave; t < n_tiles; t += kRefreshWaves) {
    wait_loads();
    bf16x8 kop[kKS], vop[2][kDT];
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks) kop[ks] = as_bf16x8(*reinterpret_cast<const uint4*>(stage + stage_off<D>(qi, 2 * ks + hh)));
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int dt = 0; dt < kDT; ++dt) vop[ks][dt] = read_v_operand32<D>(stage + G::kStageBytes, dt, ks, lane);
    wait_lds_reads();
    if (t + kRefreshWaves < n_tiles) request(t + kRefreshWaves);
    attend_subtile32<D, (LSE ? 3 : 2) | (D == 64 ? 4 : 0)>([&](int ks) { return kop[ks]; }, [&](int dt, int ks) { return vop[ks][dt]; }, q,
                                     low_mask(p.L - t * kSubTile), hh, p.scale_log2, m_run, l_run, r_run, o);
  }
  store_o_tile<D>(stage, o, qi, hh);  // the wavefront's own stage, read for the last time above
  const uintx2 sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(r_run), __float_as_uint(r_run), false, false);
  if (hh == 0) mr_sh[wave][qi] = make_float2(m_run, __uint_as_float(sw.x) + __uint_as_float(sw.y));
  if (LSE) {
    const uintx2 lw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_run), __float_as_uint(l_run), false, false);
    if (hh == 0) l_sh[wave][qi] = __uint_as_float(lw.x) + __uint_as_float(lw.y);
  }
  __syncthreads();
  const int mq = threadIdx.x >> 4, c0 = threadIdx.x & 15;  // thread = (query, chunks c0, c0 + 16, ...)
  float f[kRefreshWaves], mmax = -INFINITY, rsum = 0.f, lsum = 0.f;
#pragma unroll
  for (int w = 0; w < kRefreshWaves; ++w) mmax = fmaxf(mmax, mr_sh[w][mq].x);
#pragma unroll
  for (int w = 0; w < kRefreshWaves; ++w) {
    const float2 mr = mr_sh[w][mq];
    f[w] = mr.y > 0.f ? __builtin_amdgcn_exp2f(mr.x - mmax) : 0.f;
    rsum += f[w] * mr.y;
    if (LSE) lsum += f[w] * l_sh[w][mq];
  }
  const int row = tile * 32 + mq;
  if (row >= p.n_q) return;
  const float inv = rsum > 0.f ? 1.f / rsum : 0.f;
#pragma unroll
  for (int i = 0; i < kOChunks / 16; ++i) {
    const int ch = c0 + 16 * i;
    floatx4 s = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < kRefreshWaves; ++w) s += f[w] * *reinterpret_cast<const floatx4*>(lds + w * kBufBytes + o_chunk<D>(mq, ch));
    *reinterpret_cast<uint2*>(p.out + (int64_t)h * p.osh + (int64_t)row * p.osn + ch * 4) =
        make_uint2(cvt_pk_bf16(s[0] * inv, s[1] * inv), cvt_pk_bf16(s[2] * inv, s[3] * inv));
  }
  if (LSE && c0 == 0) p.lse[(int64_t)h * p.n_q + row] = lsum > 0.f ? (mmax + __builtin_amdgcn_logf(lsum)) * kLn2 : -INFINITY;
}

// Which query tiles go to which kernel.  Every 256-query block takes the same time, so refresh_attn_kernel runs in rounds of 256
// blocks (one per compute unit; at d = 64 two fit, and take twice as long), and a round that is mostly empty costs more than half of a
// full one.  Half blocks of four tiles, every key sub-tile for half of the wavefronts, take two thirds of a block's time, quarters of two tiles
// a little over a third (d = 64, where two single tiles share a compute unit: no gain, not built).
// refresh_tail_kernel takes single 32-query tiles: an eighth of the key sub-tiles per wavefront, each about twice
// (d = 64: four times) as long because eight tiles no longer share the staged rows.  The ways
// to cut, the cheapest is taken (the cache refresh is left out, with which the cut must not change):
//   everything in blocks, the ragged one of each head included;
//   whole blocks, or whole rounds of them, and of the rest
//     all in halves (or quarters), with every head's last tiles in halves, the last of them padded or not;
//     whole rounds of halves (or quarters), and single tiles; or single tiles only.
// Cost of a launch (LaunchCost, us): a fixed part, one per round, and per key sub-tile of a round what a round of few workgroups takes, up to what
// a full one does, with the square of how full it is.  What grows is the clock's period: a full chip of matrix products on real
// data holds a lower clock than a few compute units (8192 keys, d = 128, us per sub-tile with 32, 128 and 256 workgroups: blocks 0.80, 0.84,
// 1.04, halves 0.49, 0.52, 0.60, quarters 0.33, 0.35, 0.39; on zeros, which hardly switch, 0.72, 0.72, 0.74, 0.44, 0.44, 0.45, 0.32, 0.30, 0.31; tiles do
// not feel it).  The figures are those that choose best among all ways to cut 648 block entries of 4 to 32 heads and 1K to 33K rows, each way
// timed: on average 0.03 % (d = 64: 0.3 %) above the fastest way, 2 % (7 %) at most; rounds of one price each, however full, were 1.1 %
// above it and up to 27 % (18 %), blocks and tiles only 7.5 % (2.7 %) and up to 49 % (30 %).  Blocks and tiles only, and with halves:
// d = 128: 32 heads, 2741 rows 185 -> 159 us, 2991 rows 219 -> 189, 4900 rows 487 -> 432; 8
// heads, 4096 rows 117 -> 88, 11 691 rows 669 -> 575; 4 heads, 5860 rows 117 -> 100, 8192 rows 219 -> 154; d = 64: 32 heads, 2991 rows 124 ->
// 115; 8 heads, 4096 rows 60.6 -> 52.5.  Quarters, where tiles took two rounds or more: d = 128, 8 heads, 1500 rows 31.1 -> 25.3; 4 heads, 2455 rows
// 38.0 -> 34.6, 3000 rows 45.5 -> 39.7, 4096 rows 63.4 -> 56.2.
// 32 heads, 8256 rows (33 blocks per head, 4.1 rounds): 1213 us all in blocks, 1106 us cut; 4 heads, 1056 rows, d = 64: 26 and 8.
// A launch has fewer than 2^32 threads (kMaxGroups workgroups): ways to cut with more tiles or parts than that are left out, and a cache refresh
// whose chunks do not fit behind the last attention launch (2^24 of them: block 1, 32 heads, half a million rows) has a launch of its own.
struct RefreshCut {
  int n_qb = 0, n_work = 0, parts = 2, part_whole = 0, part_head = 0;
  int64_t n_part = 0, n_tail = 0;
  float time = 0.f;
};
struct LaunchCost {
  float fixed, round, few, full;  // few, full: of a sub-tile in a round of few workgroups, and in a full one
  float of(int64_t n, float sub) const {  // n workgroups of `sub` key sub-tiles
    constexpr int kSlots = 256;
    if (n == 0) return 0.f;
    const float whole = (float)(n / kSlots), part = (float)(n % kSlots) / kSlots;
    return part > 0.f ? fixed + (whole + 1.f) * round + sub * (whole * full + few + (full - few) * part * part) : fixed + whole * (round + sub * full);
  }
};
static RefreshCut cut_refresh(int head_dim, int n_heads, int n_q, int L) {
  constexpr int kSlots = 256;
  constexpr int64_t kMaxGroups = ((int64_t(1) << 32) - 1) / (64 * kRefreshWaves);
  const int tiles = ceil_div(n_q, 32), last = tiles % kRefreshWaves;
  const float sub = (float)ceil_div(L, kSubTile);
  const bool d128 = head_dim == 128;
  const LaunchCost block = d128 ? LaunchCost{4.f, 3.f, 0.61f, 0.96f} : LaunchCost{12.f, 0.f, 0.43f, 0.54f};
  const LaunchCost half = d128 ? LaunchCost{7.f, 3.f, 0.4f, 0.57f} : LaunchCost{8.f, 0.f, 0.32f, 0.33f}, quarter = {6.f, 3.f, 0.28f, 0.34f};
  const LaunchCost single = d128 ? LaunchCost{3.f, 3.f, 0.195f, 0.195f} : LaunchCost{4.5f, 0.f, 0.114f, 0.114f};
  const int64_t whole = (int64_t)(tiles / kRefreshWaves) * n_heads, padded = (int64_t)ceil_div(tiles, kRefreshWaves) * n_heads;
  RefreshCut best;
  best.n_qb = ceil_div(tiles, kRefreshWaves);
  best.n_work = (int)padded;
  best.time = block.of(padded, sub);
  auto consider = [&](int64_t work, int parts, int64_t part_whole, int part_head) {
    const int part_tiles = kRefreshWaves / parts;
    RefreshCut c;
    c.n_qb = tiles / kRefreshWaves;
    c.n_work = (int)work;
    c.parts = parts;
    c.part_whole = (int)part_whole;
    c.part_head = part_head;
    c.n_part = part_whole + (int64_t)part_head * n_heads;
    c.n_tail = (parts * (whole - work) - part_whole) * part_tiles + (int64_t)std::max(0, last - part_head * part_tiles) * n_heads;
    if (c.n_part + 7 > kMaxGroups || c.n_tail + 7 > kMaxGroups) return;
    c.time = block.of(work, sub) + (parts == 2 ? half : quarter).of(c.n_part, sub) + single.of(c.n_tail, sub);
    if (c.time < best.time) best = c;
  };
  const int64_t rest = whole % kSlots;
  for (int64_t work : {whole, whole - rest}) {
    consider(work, 2, 0, 0);
    for (int parts = 2; parts <= (d128 ? 4 : 2); parts *= 2) {
      const int64_t n = parts * (whole - work);
      for (int part_head = 0; part_head <= ceil_div(last, kRefreshWaves / parts); ++part_head) consider(work, parts, n, part_head);
      consider(work, parts, n - n % kSlots, 0);
    }
  }
  return best;
}
template <int D>
static hipError_t launch_refresh_t(RefreshArgs& a, const focus_shape& s, const CacheRefresh* copy, hipStream_t st) {
  constexpr int64_t kMaxGroups = ((int64_t(1) << 32) - 1) / (64 * kRefreshWaves);
  const RefreshCut cut = cut_refresh(D, s.n_heads, s.n_gen, s.n_ctx + s.n_resp);
  a.n_heads = s.n_heads;
  a.n_qb = cut.n_qb;
  a.n_work = cut.n_work;
  a.n_part_whole = cut.part_whole;
  a.n_part_head = cut.part_head;
  a.part_tiles = kRefreshWaves / cut.parts;
  a.n_tail = (int)cut.n_tail;
  const dim3 block(64 * kRefreshWaves);
  const int64_t copies = copy ? ceil_div64((int64_t)copy->n_chunks * copy->n_heads, 2) : 0;
  auto list = [](int64_t n) { return (int64_t)8 * ceil_div64(n, 8); };
  if (copy != nullptr && list(cut.n_tail > 0 ? cut.n_tail : (cut.n_part > 0 ? cut.n_part : cut.n_work)) + copies > kMaxGroups) {
    hipError_t e = launch_cache_refresh(*copy, D, st);
    if (e != hipSuccess) return e;
    copy = nullptr;
  }
  if (cut.n_work > 0) {
    if (copy != nullptr && cut.n_part + cut.n_tail == 0)
      hipLaunchKernelGGL((refresh_attn_kernel<D, 1, false, true>), dim3((uint32_t)(list(cut.n_work) + copies)), block, 0, st, a, *copy);
    else
      hipLaunchKernelGGL((refresh_attn_kernel<D, 1, false, false>), dim3((uint32_t)list(cut.n_work)), block, 0, st, a, CacheRefresh{});
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (cut.n_part > 0) {
    const bool with = copy != nullptr && cut.n_tail == 0;
    const dim3 grid((uint32_t)(list(cut.n_part) + (with ? copies : 0)));
    const CacheRefresh with_copy = with ? *copy : CacheRefresh{};
    auto launch = [&](auto parts) {
      if (a.lse)
        hipLaunchKernelGGL((refresh_attn_kernel<D, decltype(parts)::value, true, true>), grid, block, 0, st, a, with_copy);
      else
        hipLaunchKernelGGL((refresh_attn_kernel<D, decltype(parts)::value, false, true>), grid, block, 0, st, a, with_copy);
    };
    if (cut.parts == 2)
      launch(std::integral_constant<int, 2>{});
    else if constexpr (D == 128)
      launch(std::integral_constant<int, 4>{});
    else
      return hipErrorInvalidValue;
    hipError_t e = hipGetLastError();
    if (e != hipSuccess || cut.n_tail == 0) return e;
  }
  if (cut.n_tail == 0) return hipSuccess;
  const dim3 grid((uint32_t)(list(cut.n_tail) + (copy ? copies : 0)));
  // d = 64: up to 128 tiles, which is what long prompts leave over, have a compute unit each (LDS that nobody uses sees to it): they are the
  // last to finish, and a chunk beside them costs more than it gains.  Layer with and without, medians of 24 pairs in turn: 32 heads, 4104
  // rows 193.8 and 195.8 us, 8256 rows 660.4 and 663.8; 8 heads, 8256 rows 209.1 and 210.0; 16 heads, 16 404 rows 1255.7 and 1258.9; 4
  // heads, 16 404 rows 394.1 and 395.3.
  const uint32_t alone = D == 64 && copy && cut.n_tail <= 128 ? 32768 : 0;
  if (a.lse)
    hipLaunchKernelGGL((refresh_tail_kernel<D, true>), grid, block, alone, st, a, copy ? *copy : CacheRefresh{});
  else
    hipLaunchKernelGGL((refresh_tail_kernel<D, false>), grid, block, alone, st, a, copy ? *copy : CacheRefresh{});
  return hipGetLastError();
}

hipError_t launch_refresh_attn(const void* Q, const void* K, const void* V, const focus_shape& s, void* out, float* lse,
                               hipStream_t st, const CacheRefresh* copy) {
  RefreshArgs a;
  a.Q = static_cast<const uint16_t*>(Q);
  a.K = static_cast<const uint16_t*>(K);
  a.V = static_cast<const uint16_t*>(V);
  a.out = static_cast<uint16_t*>(out);
  a.lse = lse;
  a.qsh = s.q_stride_h; a.qsn = s.q_stride_n;
  a.ksh = copy ? copy->nsh : s.k_stride_h; a.ksn = copy ? copy->nsn : s.k_stride_n;
  a.vsh = copy ? copy->nsh : s.v_stride_h; a.vsn = copy ? copy->nsn : s.v_stride_n;
  a.osh = s.o_stride_h; a.osn = s.o_stride_n;
  a.n_q = s.n_gen;
  a.L = s.n_ctx + s.n_resp;
  a.scale_log2 = kLog2e / sqrtf((float)s.head_dim);
  if (s.head_dim == 128) return launch_refresh_t<128>(a, s, copy, st);
  return launch_refresh_t<64>(a, s, copy, st);
}

// =====================================================================================================
// Probe-layer logits (Eq. 6, first half): logits[h, j, q] = log2(e) * Q[h, i_q] . K[h, j] / sqrt(d) for every key
// j in [0, L), and per (head, query, split) the maximum and the sum of exp2(logit - maximum).
// =====================================================================================================
struct LogitArgs {
  const uint16_t* Q;
  const uint16_t* K;
  const int32_t* active_idx;
  const int32_t* counts;
  float* logits;      // [H, ceil(L / 4), 16, 4]: see spill_logits  (mode 0, at most 16 queries)
  float* part_ml;     // [H, n_split, q_pad, 2]                (modes 0, 1)
  const float* lse2;  // [H, q_pad] base-2 log-sum-exp per row (mode 2)
  float* colpart;     // [q_groups * H, L]                     (mode 2)
  int64_t qsh, qsn, ksh, ksn;
  int H, L, n_gen, max_active;
  int n_sub, n_split, q_pad;
  float scale_log2;
  SelectArgs sel;  // SELECT only
};

// select_positions; lane a of `row` receives the a-th active position (a < their number, which is returned)
__device__ __forceinline__ int select_rows(const SelectArgs& s, int n_gen, int max_active, int lane, bool writer, int& row) {
  const unsigned long long active = select_positions(s, n_gen, max_active, lane, writer);
  const unsigned long long below = (1ull << lane) - 1ull;
  const int n = (int)__popcll(active);
  // the active lanes go to the front, the others behind them
  const int to = ((active >> lane) & 1ull) ? (int)__popcll(active & below) : n + (int)__popcll(~active & below);
  row = __builtin_amdgcn_ds_permute(to << 2, lane);
  return n;
}

// keys [32 st, 32 st + 32) of the first L
__device__ __forceinline__ SubTile key_subtile(int st, int L) {
  SubTile t;
  t.kind = 0;
  t.sink_row = 0;
  t.row0 = st * kSubTile;
  t.vmask = low_mask(min(L - t.row0, kSubTile));
  return t;
}

// Up to 16 active queries: the scaled logits are written out (re-reading 64 bytes per key and head is cheaper than a second pass
// over K) together with the per-split softmax statistics.
// SELECT: every wavefront makes the query selection itself, beside its first K rows, instead of reading what a launch of its own
// has written; the first workgroup writes the lists for everyone else (a step of 4 heads at 1K: one launch of 3 us less).
// STAGES = 2: the sub-tile after the next travels as well; which launches take it, and what it gives, at logits_in_two_stages.
template <int D, bool SELECT, int STAGES>
__global__ __launch_bounds__(256, 2) void qk_logits_kernel(const uint16_t* K, int64_t ksh, int64_t ksn, const int32_t* active_idx, int L,
                                                           int n_sub, int n_split, int max_active, int n_gen, const LogitArgs args) {
  LogitArgs p = args;  // what the first requests need comes in registers, as in the attention kernels
  p.K = K;
  p.ksh = ksh;
  p.ksn = ksn;
  p.active_idx = active_idx;
  p.L = L;
  p.n_sub = n_sub;
  p.n_split = n_split;
  p.max_active = max_active;
  p.n_gen = n_gen;
  using G = Geo<D>;
  __shared__ __attribute__((aligned(256))) char lds[STAGES * kWavesPerGroup * G::kStageBytes];
  __shared__ float ml_sh[kWavesPerGroup][16][2];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int c = lane & 15, g = lane >> 4;
  const int split = blockIdx.x, h = blockIdx.y;
  char* stageK = lds + wave * G::kStageBytes;
  const uint16_t* Qh = p.Q + (int64_t)h * p.qsh;
  const uint16_t* Kh = p.K + (int64_t)h * p.ksh;

  int st = split * kWavesPerGroup + wave;
  const int st_end = p.n_sub, st_step = p.n_split * kWavesPerGroup;
  int qrow = -1;
  if (!SELECT) qrow = fetch_q_row(p.active_idx, 0, p.max_active, p.n_gen, lane);
  SubTile t = key_subtile(st < st_end ? st : 0, p.L);
  if (st < st_end) issue_subtile<D>(Kh, p.ksn, t, stageK, lane);
  int n_act;
  if (SELECT) {
    int row;
    n_act = select_rows(p.sel, p.n_gen, p.max_active, lane, wave == 0 && (split | h) == 0, row);
    row = __shfl(row, c, kWave);
    qrow = c < n_act ? row : -1;
  }

  bf16x8 q[G::kKSteps];
  load_q_tile<D>(q, Qh, p.qsn, qrow, lane);
  if (!SELECT) n_act = p.counts ? min(max(p.counts[1], 0), p.max_active) : p.max_active;
  mask_q_tile<D>(q, 0, n_act, lane);

  float m_run = -INFINITY, l_run = 0.f;
  if constexpr (STAGES == 2) {
    // the stores of a whole sub-tile's logits are counted, so that nothing waits for them; a ragged one's are waited for
    char *here = stageK, *there = stageK + kWavesPerGroup * G::kStageBytes;
    int next = st + st_step;
    SubTile tn = key_subtile(next < st_end ? next : 0, p.L);
    if (next < st_end) issue_subtile<D>(Kh, p.ksn, tn, there, lane);
    bool stored = false;  // the stores behind the rows under way
    while (st < st_end) {
      if (next >= st_end)
        wait_loads();
      else if (stored)
        wait_loads_but<G::kLoads + kSpillStores>();
      else
        wait_loads_but<G::kLoads>();
      bf16x8 kop[2][G::kKSteps];
      read_k_operands16<D>(kop, here, lane);
      const int after = next + st_step;
      const SubTile ta = key_subtile(after < st_end ? after : 0, p.L);
      if (after < st_end) issue_subtile<D>(Kh, p.ksn, ta, here, lane);
      floatx4 acc[2];
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        acc[kt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kk = 0; kk < G::kKSteps; ++kk) acc[kt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kop[kt][kk], q[kk], acc[kt], 0, 0, 0);
      }
      float ps[8];
      softmax_step(acc, t.vmask, g, p.scale_log2, m_run, l_run, ps);
      spill_logits(p.logits, h, p.L, p.max_active, t.row0, acc, p.scale_log2, lane);
      stored = after < st_end && t.vmask == 0xffffffffu;
      t = tn;
      tn = ta;
      st = next;
      next = after;
      char* const other = here;
      here = there;
      there = other;
    }
  }
  while (st < st_end) {  // (STAGES = 1)
    const SubTile cur = t;
    wait_loads();
    floatx4 acc[2];
    qk_subtile<D>(acc, stageK, q, lane);
    // the staged rows are consumed: the next sub-tile can stream in while the results are written
    st += st_step;
    if (st < st_end) {
      t = key_subtile(st, p.L);
      wait_lds_reads();
      issue_subtile<D>(Kh, p.ksn, t, stageK, lane);
    }
    float ps[8];
    softmax_step(acc, cur.vmask, g, p.scale_log2, m_run, l_run, ps);
    spill_logits(p.logits, h, p.L, p.max_active, cur.row0, acc, p.scale_log2, lane);
  }

  if (g == 0) {
    ml_sh[wave][c][0] = m_run;
    ml_sh[wave][c][1] = l_run;
  }
  __syncthreads();
  if (threadIdx.x < 16) {
    float mmax = -INFINITY;
#pragma unroll
    for (int w = 0; w < kWavesPerGroup; ++w) mmax = fmaxf(mmax, ml_sh[w][threadIdx.x][0]);
    float lsum = 0.f;
#pragma unroll
    for (int w = 0; w < kWavesPerGroup; ++w) {
      const float l = ml_sh[w][threadIdx.x][1];
      if (l > 0.f) lsum += l * __builtin_amdgcn_exp2f(ml_sh[w][threadIdx.x][0] - mmax);
    }
    const int64_t row = ((int64_t)h * p.n_split + split) * 16 + threadIdx.x;
    *reinterpret_cast<float2*>(p.part_ml + 2 * row) = make_float2(lsum > 0.f ? mmax : -INFINITY, lsum);
  }
}

// More than 16 active queries: spilling 64 floats and more per key and head would outweigh K, so K is scanned twice.
// MODE 1: per-split softmax statistics.
// MODE 2: with the row log-sum-exps known, the probabilities are formed on the fly and summed over the workgroup's queries;
//         colpart[qg * H + h, j] = sum_i P[h, i, j].
// MODE 3: the same from the statistics of MODE 1, of which every workgroup forms the log-sum-exps of its queries itself, beside its
//         first K rows (lse_in_logits).
// A workgroup has NT tiles of 32 queries (32x32x16 MFMA) and four slots, one per wavefront, which walk the key sub-tiles; the
// operands of a sub-tile are read from its slot once, into registers, and the next one is requested before they are multiplied.
// MODE 1 computes K Q^T (a lane holds one query's logits: the running maximum is one exchange), MODE 2 Q K^T (a lane holds one
// key's probabilities: the sum over the queries stays in its registers).  Tiles past the device-side count are skipped.
// SELECT (MODE 1) as in qk_logits_kernel.
// Grid as in wide_attn_kernel: the query groups of one (head, key split) pair run on one XCD and share its rows there.
// 32 heads, 32 832 keys, both passes and what follows them: 113 -> 106 us with 28 of 36 queries (bound by HBM), 8 256 keys, 60
// queries 69 -> 44; 4 K/V heads, 16 640 keys, 196 queries 64 -> 36; 8 K/V heads, 60 064 keys, 400 queries 330 -> 198 (16-query tiles,
// each wavefront fetching all query rows, query groups far apart in time).
template <int D, int NT, int MODE, bool SELECT>
__global__ __launch_bounds__(256, NT == 1 ? 4 : 2) void wide_logits_kernel(const uint16_t* K, int64_t ksh, int64_t ksn,
                                                                           const int32_t* active_idx, int L, int n_sub, int n_split,
                                                                           int max_active, int n_gen, int q_groups, const LogitArgs args) {
  LogitArgs p = args;
  p.K = K;
  p.ksh = ksh;
  p.ksn = ksn;
  p.active_idx = active_idx;
  p.L = L;
  p.n_sub = n_sub;
  p.n_split = n_split;
  p.max_active = max_active;
  p.n_gen = n_gen;
  using G = Geo<D>;
  constexpr int kKS = D / 16;
  constexpr bool SUMS = MODE >= 2;
  __shared__ __attribute__((aligned(16))) char lds[kWavesPerGroup * G::kStageBytes];
  __shared__ __attribute__((aligned(16))) char stageQ[NT * G::kStageBytes];
  float2 (*ml_sh)[NT * 32] = reinterpret_cast<float2 (*)[NT * 32]>(stageQ);  // [4][NT * 32], once the queries are in registers
  static_assert(kWavesPerGroup * sizeof(float2) * 32 <= G::kStageBytes, "fits");

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qi = lane & 31, hh = lane >> 5;
  const int slot8 = list_index() >> 3;
  const int pair = (slot8 / q_groups) * 8 + (int)(blockIdx.x & 7u), qg = slot8 % q_groups;
  if (pair >= n_split * p.H) return;  // whole workgroup
  const int h = pair / n_split, split = pair - h * n_split;
  const int q_base = qg * NT * 32;
  char* stageK = lds + wave * G::kStageBytes;
  const uint16_t* Qh = p.Q + (int64_t)h * p.qsh;
  const uint16_t* Kh = p.K + (int64_t)h * p.ksh;

  int st = split * kWavesPerGroup + wave;
  const int st_end = p.n_sub, st_step = p.n_split * kWavesPerGroup;
  // The query rows go through LDS, a quarter per wavefront: four wavefronts fetching all of them moved more bytes than K where
  // a wavefront walks a handful of sub-tiles.  Staged like K rows; load i of a wavefront covers kRowsPerLoad rows.
  constexpr int kQLoads = NT * 32 / (kWavesPerGroup * G::kRowsPerLoad);
  const int q_sub = lane / G::kChunks, q_pos = lane % G::kChunks;
  int qrow[kQLoads];
  bool live[NT];  // this lane's query of tile n exists
  if (!SELECT) {
#pragma unroll
    for (int i = 0; i < kQLoads; ++i) {
      const int a = q_base + (wave * kQLoads + i) * G::kRowsPerLoad + q_sub;
      qrow[i] = a < p.max_active ? p.active_idx[a] : 0;
    }
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      const int a = q_base + n * 32 + qi, row = a < p.max_active ? p.active_idx[a] : -1;
      live[n] = row >= 0 && row < p.n_gen;
    }
  }
  SubTile t = key_subtile(st < st_end ? st : 0, p.L);
  if (st < st_end) issue_subtile<D>(Kh, p.ksn, t, stageK, lane);
  int n_act;
  if (SELECT) {
    int row;
    n_act = select_rows(p.sel, p.n_gen, p.max_active, lane, wave == 0 && (pair | qg) == 0, row);
#pragma unroll
    for (int i = 0; i < kQLoads; ++i) {
      const int a = q_base + (wave * kQLoads + i) * G::kRowsPerLoad + q_sub, r = __shfl(row, a & (kWave - 1), kWave);
      qrow[i] = a < n_act ? r : 0;
    }
  } else {
    n_act = p.counts ? min(max(p.counts[1], 0), p.max_active) : p.max_active;
  }
  {
    typedef const __attribute__((address_space(1))) void* gptr_t;
    typedef __attribute__((address_space(3))) void* lptr_t;
#pragma unroll
    for (int i = 0; i < kQLoads; ++i) {
      const int slot = (wave * kQLoads + i) * G::kRowsPerLoad + q_sub;
      const uint16_t* src = Qh + (int64_t)min(max(qrow[i], 0), p.n_gen - 1) * p.qsn + (q_pos ^ (slot & (G::kChunks - 1))) * 8;
      __builtin_amdgcn_global_load_lds((gptr_t)src, (lptr_t)(stageQ + (wave * kQLoads + i) * 1024), 16, 0, 0);
    }
  }
  float neg_lse[SUMS ? NT : 1][16];  // minus the log-sum-exp of query 8 (v / 4) + 4 hh + v % 4; -inf for rows that do not exist
  auto set_lse = [&](int n, int v, int a, float z) __attribute__((always_inline)) {
    neg_lse[n][v] = (a < n_act && z < INFINITY) ? -z : -INFINITY;  // exp2(x - inf) = 0: the row contributes nothing
  };
  if (MODE == 2) {
#pragma unroll
    for (int n = 0; n < NT; ++n) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int a = q_base + n * 32 + 8 * (v >> 2) + 4 * hh + (v & 3);
        set_lse(n, v, a, p.lse2[(int64_t)h * p.q_pad + min(a, p.q_pad - 1)]);
      }
    }
  }
  // MODE 3: thread = (query, split lane) adds up its share of the statistics; they meet in stageQ once the queries are in registers
  constexpr int kRowLanes = 256 / (NT * 32);
  RowState mine{-INFINITY, 0.f};
  if (MODE == 3)
    mine = add_row_splits(reinterpret_cast<const float2*>(p.part_ml) + (int64_t)h * n_split * p.q_pad + q_base + threadIdx.x % (NT * 32),
                          p.q_pad, threadIdx.x / (NT * 32), kRowLanes, n_split);
  wait_loads();
  __syncthreads();
  bf16x8 q[NT][kKS];  // lane (query, hh) holds Q[query][16 ks + 8 hh .. + 7]
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    const bool exists = q_base + n * 32 + qi < n_act && (SELECT || live[n]);
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks) {
      const uint4 v = *reinterpret_cast<const uint4*>(stageQ + n * G::kStageBytes + stage_off<D>(qi, 2 * ks + hh));
      q[n][ks] = as_bf16x8(exists ? v : make_uint4(0u, 0u, 0u, 0u));
    }
  }
  if (MODE == 3) {
    float2* lane_sh = reinterpret_cast<float2*>(stageQ);  // [kRowLanes][NT * 32]
    float* lse_sh = reinterpret_cast<float*>(stageQ + 256 * sizeof(float2));
    static_assert(256 * sizeof(float2) + NT * 32 * sizeof(float) <= NT * G::kStageBytes, "fits");
    __syncthreads();  // every wavefront has its queries in registers
    lane_sh[threadIdx.x] = make_float2(mine.m, mine.l);
    __syncthreads();
    if (threadIdx.x < NT * 32) lse_sh[threadIdx.x] = lse_of(add_row_splits(lane_sh + threadIdx.x, NT * 32, 0, 1, kRowLanes));
    __syncthreads();
#pragma unroll
    for (int n = 0; n < NT; ++n) {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int i = n * 32 + 8 * (v >> 2) + 4 * hh + (v & 3);
        set_lse(n, v, q_base + i, lse_sh[i]);
      }
    }
  }

  float m_run[NT], l_run[NT];  // MODE 1; l_run: this lane's share of the row sum (its 16 of every 32 keys)
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    m_run[n] = -INFINITY;
    l_run[n] = 0.f;
  }
  while (st < st_end) {
    const SubTile cur = t;
    wait_loads();
    bf16x8 kop[kKS];
#pragma unroll
    for (int ks = 0; ks < kKS; ++ks) kop[ks] = as_bf16x8(*reinterpret_cast<const uint4*>(stageK + stage_off<D>(qi, 2 * ks + hh)));
    st += st_step;
    wait_lds_reads();
    if (st < st_end) {
      t = key_subtile(st, p.L);
      issue_subtile<D>(Kh, p.ksn, t, stageK, lane);
    }
    float colsum = 0.f;
#pragma unroll
    for (int n = 0; n < NT; ++n) {
      if (n > 0 && q_base + n * 32 >= n_act) break;  // uniform
      floatx16 acc;
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[v] = 0.f;
#pragma unroll
      for (int ks = 0; ks < kKS; ++ks)
        acc = MODE == 1 ? __builtin_amdgcn_mfma_f32_32x32x16_bf16(kop[ks], q[n][ks], acc, 0, 0, 0)
                        : __builtin_amdgcn_mfma_f32_32x32x16_bf16(q[n][ks], kop[ks], acc, 0, 0, 0);
      if (SUMS) {
#pragma unroll
        for (int v = 0; v < 16; ++v) colsum += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[v], p.scale_log2, neg_lse[n][v]));
      } else {
        if (cur.vmask != 0xffffffffu) {  // wave-uniform: slots that hold no key
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[v] = ((cur.vmask >> (8 * (v >> 2) + 4 * hh + (v & 3))) & 1u) ? acc[v] : -INFINITY;
        }
        float mx = fmaxf(acc[0], acc[1]);
#pragma unroll
        for (int v = 2; v < 16; ++v) mx = fmaxf(mx, acc[v]);
        const uintx2 sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(mx), __float_as_uint(mx), false, false);
        const float m_new = fmaxf(m_run[n], fmaxf(__uint_as_float(sw.x), __uint_as_float(sw.y)) * p.scale_log2);
        const float m_use = m_new == -INFINITY ? 0.f : m_new;
        l_run[n] *= __builtin_amdgcn_exp2f(m_run[n] - m_use);
        m_run[n] = m_new;
        float sum[2] = {0.f, 0.f};
#pragma unroll
        for (int v = 0; v < 16; ++v) sum[v & 1] += __builtin_amdgcn_exp2f(__builtin_fmaf(acc[v], p.scale_log2, -m_use));
        l_run[n] += sum[0] + sum[1];
      }
    }
    if (SUMS) {
      const uintx2 sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(colsum), __float_as_uint(colsum), false, false);
      if (hh == 0 && ((cur.vmask >> qi) & 1u))
        p.colpart[((int64_t)qg * p.H + h) * p.L + cur.row0 + qi] = __uint_as_float(sw.x) + __uint_as_float(sw.y);
    }
  }
  if (SUMS) return;

  __syncthreads();  // every wavefront has its queries in registers: stageQ is free for the statistics
#pragma unroll
  for (int n = 0; n < NT; ++n) {
    const uintx2 sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(l_run[n]), __float_as_uint(l_run[n]), false, false);
    if (hh == 0) ml_sh[wave][n * 32 + qi] = make_float2(m_run[n], __uint_as_float(sw.x) + __uint_as_float(sw.y));
  }
  __syncthreads();
  if (threadIdx.x < NT * 32) {
    float mmax = -INFINITY;
#pragma unroll
    for (int w = 0; w < kWavesPerGroup; ++w) mmax = fmaxf(mmax, ml_sh[w][threadIdx.x].x);
    float lsum = 0.f;
#pragma unroll
    for (int w = 0; w < kWavesPerGroup; ++w) {
      const float2 v = ml_sh[w][threadIdx.x];
      if (v.y > 0.f) lsum += v.y * __builtin_amdgcn_exp2f(v.x - mmax);
    }
    if (q_base + (int)threadIdx.x < p.q_pad) {
      const int64_t row = ((int64_t)h * p.n_split + split) * p.q_pad + q_base + threadIdx.x;
      *reinterpret_cast<float2*>(p.part_ml + 2 * row) = make_float2(lsum > 0.f ? mmax : -INFINITY, lsum);
    }
  }
}

// One query tile: two stages per wavefront where the workgroups (two of them share a compute unit then, four with one stage) are
// resident at once all the same, or are many and long.  Sink chain with one stage and with two: 32 heads, 8256 keys, 16 splits 29.4 and
// 28.7 us, 4160 keys, 8 splits 20.9 and 19.9; 16 heads, 8256 keys 20.2 and 19.2; 4 heads, 32 832 keys 21.1 and 20.2; 32 heads, 131 136
// keys, 4096 workgroups of eight rounds 264 and 259; but 15 986 keys, 1024 workgroups of four rounds 43.4 and 44.2, 32 832 keys, 4128 of
// two 75.3 and 81.0.  The same, 4096 workgroups of 32 to 128 heads: 49 216 keys, three rounds 106 and 108; 65 600, four 137.5 and 136.0;
// 98 368, six 201.5 and 197.4; 120 064, seven 240.5 and 233.3 (so the line could lie lower, at four rounds); eight and more: 64 heads,
// 65 600 keys 272 and 265, 128 heads, 32 832 keys 285 and 278, d = 64 185 and 183; 64 heads, d = 64, 80 064 keys 219 and 215; 32 heads,
// 200 064 keys 914 and 904.
static bool logits_in_two_stages(const SplitPlan& p, int n_heads) {
  const int rounds = ceil_div(p.n_sub, kWavesPerGroup);
  return rounds >= 4 * p.n_split && ((int64_t)p.n_split * n_heads <= 512 || rounds >= 8 * p.n_split);
}

template <int D>
static hipError_t launch_logits_t(const LogitArgs& a, const SplitPlan& p, int mode, bool select, hipStream_t st) {
#define LOGITS_ARGS a.K, a.ksh, a.ksn, a.active_idx, a.L, a.n_sub, a.n_split, a.max_active, a.n_gen
  if (p.q_tiles_per_group == 1) {  // one tile spills its logits, several take two passes
    if (mode != 0) return hipErrorInvalidValue;
    const dim3 grid(p.n_split, a.H);
    const bool two = logits_in_two_stages(p, a.H);
    if (select && two)
      hipLaunchKernelGGL((qk_logits_kernel<D, true, 2>), grid, dim3(256), 0, st, LOGITS_ARGS, a);
    else if (select)
      hipLaunchKernelGGL((qk_logits_kernel<D, true, 1>), grid, dim3(256), 0, st, LOGITS_ARGS, a);
    else if (two)
      hipLaunchKernelGGL((qk_logits_kernel<D, false, 2>), grid, dim3(256), 0, st, LOGITS_ARGS, a);
    else
      hipLaunchKernelGGL((qk_logits_kernel<D, false, 1>), grid, dim3(256), 0, st, LOGITS_ARGS, a);
    return hipGetLastError();
  }
  if (mode == 0 || query_group_list(p, a.H) > kMaxList) return hipErrorInvalidValue;
  if (a.q_pad != p.q_groups * p.q_tiles_per_group * kQTile) return hipErrorInvalidValue;  // MODE 3 reads the statistics of whole query groups
  const dim3 grid = grid_list(query_group_list(p, a.H));
#define WIDE_LOGITS(NT)                                                                                                 \
  if (mode == 2 && a.part_ml != nullptr)                                                                                \
    hipLaunchKernelGGL((wide_logits_kernel<D, NT, 3, false>), grid, dim3(256), 0, st, LOGITS_ARGS, p.q_groups, a);      \
  else if (mode == 2)                                                                                                   \
    hipLaunchKernelGGL((wide_logits_kernel<D, NT, 2, false>), grid, dim3(256), 0, st, LOGITS_ARGS, p.q_groups, a);      \
  else if (select)                                                                                                      \
    hipLaunchKernelGGL((wide_logits_kernel<D, NT, 1, true>), grid, dim3(256), 0, st, LOGITS_ARGS, p.q_groups, a);       \
  else                                                                                                                  \
    hipLaunchKernelGGL((wide_logits_kernel<D, NT, 1, false>), grid, dim3(256), 0, st, LOGITS_ARGS, p.q_groups, a)
  if (p.q_tiles_per_group == 2) {
    WIDE_LOGITS(1);
  } else {
    WIDE_LOGITS(2);
  }
#undef WIDE_LOGITS
#undef LOGITS_ARGS
  return hipGetLastError();
}

// Up to four batches of statistics per thread: about as long as a launch of lse_combine_kernel would take (sink chain with that launch
// and without: 4 heads, 8256 keys, 36 queries, 65 splits 22.2 and 21.1 us; 65 600 keys, d = 64, 192 splits 28.8 and 30.0; 32 heads,
// 32 832 keys, 24 splits 105.2 and 102.6).
bool lse_in_logits(const SplitPlan& p) { return p.n_split <= 4 * kSplitsInFlight * (p.q_tiles_per_group == 2 ? 8 : 4); }

// mode 0: logits + part_ml out; mode 1: part_ml out; mode 2: lse2 in, colpart out (0: qk_logits_kernel; 1, 2: wide_logits_kernel)
hipError_t launch_qk_logits(const void* Q, const int32_t* active_idx, const int32_t* counts, int max_active,
                            const void* K, const focus_shape& s, const SplitPlan& p, int mode, float* logits,
                            float* part_ml, const float* lse2, float* colpart, hipStream_t st, const SelectArgs* select) {
  if (max_active < 1 || (select != nullptr && (mode == 2 || s.n_gen > kSelectInLogitsGen))) return hipErrorInvalidValue;
  LogitArgs a;
  a.sel = select ? *select : SelectArgs{};
  a.Q = static_cast<const uint16_t*>(Q);
  a.K = static_cast<const uint16_t*>(K);
  a.active_idx = active_idx;
  a.counts = counts;
  a.logits = logits;
  a.part_ml = part_ml;
  a.lse2 = lse2;
  a.colpart = colpart;
  a.qsh = s.q_stride_h; a.qsn = s.q_stride_n;
  a.ksh = s.k_stride_h; a.ksn = s.k_stride_n;
  a.H = s.n_heads; a.L = s.n_ctx + s.n_resp; a.n_gen = s.n_gen; a.max_active = max_active;
  a.n_sub = p.n_sub; a.n_split = p.n_split; a.q_pad = p.q_pad;
  a.scale_log2 = kLog2e / sqrtf((float)s.head_dim);
  return s.head_dim == 128 ? launch_logits_t<128>(a, p, mode, select != nullptr, st) : launch_logits_t<64>(a, p, mode, select != nullptr, st);
}

}  // namespace focus
