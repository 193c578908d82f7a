// Block-entry cache refresh: the copy of one chunk of rows with its block mean, shared by the kernel that does nothing else and by
// the block-entry attention launch that does it on the side.
#pragma once

#include "focus_common.h"
#include "focus_kernels.h"

namespace focus {

// Block-entry cache refresh (Alg. 1: every position is recomputed when a block starts): all M + N rows of the K and V
// caches take the new states, and the block means of the M prompt keys (Sec. 5.3) come out of the same pass, so the
// new K is read once.  256 threads per (chunk b of B rows, head h); chunks [0, n_b) are the prompt blocks, the rest
// cover the response rows (copied only).  The mean is accumulated in exactly the order block_means_kernel uses
// (thread (rr, c): rows rr, rr + RPP, ... of its 16-byte column slice; then the RPP partial rows in order), so the
// two kernels give bit-identical K_bar.  t = thread 0 .. 255; `red`: RPP rows of D floats; `live` = false: no chunk (the barrier
// is met all the same).  TOGETHER: the rows of K and V are requested at once (one memory round trip instead of two, twice the registers), for
// the few workgroups that run beside an attention launch; a launch of nothing else is bound by the memory and wants many small ones.
typedef unsigned uintx4_t __attribute__((ext_vector_type(4)));
template <int D, bool TOGETHER = false>
__device__ __forceinline__ void cache_refresh_chunk(const CacheRefresh& p, int b, int h, int t, bool live, float* red) {
  constexpr int TPR = D / 8;
  constexpr int RPP = 256 / TPR;
  constexpr int UNROLL = 8;
  const bool prompt = b < p.n_b;
  const int r0 = prompt ? b * p.B : p.M + (b - p.n_b) * p.B;
  const int len = live ? min(p.B, (prompt ? p.M : p.L) - r0) : 0;
  const int c = t % TPR, rr = t / TPR;
  const uint16_t* ksrc = p.Kn + (int64_t)h * p.nsh + (int64_t)r0 * p.nsn + c * 8;
  const uint16_t* vsrc = p.Vn + (int64_t)h * p.nsh + (int64_t)r0 * p.nsn + c * 8;
  uint16_t* kdst = p.Kc + (int64_t)h * p.ksh + (int64_t)r0 * p.ksn + c * 8;
  uint16_t* vdst = p.Vc + (int64_t)h * p.vsh + (int64_t)r0 * p.vsn + c * 8;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  for (int r = rr; r < len; r += RPP * UNROLL) {
    uint4 v[UNROLL], w[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const int row = r + u * RPP;
      v[u] = row < len ? load_stream16(ksrc + (int64_t)row * p.nsn) : make_uint4(0, 0, 0, 0);
    }
    if constexpr (TOGETHER) {
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) {
        const int row = r + u * RPP;
        if (row < len) w[u] = load_stream16(vsrc + (int64_t)row * p.nsn);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const int row = r + u * RPP;
      add_bf16x8(acc, v[u]);
      if (row < len) __builtin_nontemporal_store(__builtin_bit_cast(uintx4_t, v[u]), reinterpret_cast<uintx4_t*>(kdst + (int64_t)row * p.ksn));
    }
    if constexpr (TOGETHER) {
#pragma unroll
      for (int u = 0; u < UNROLL; ++u) {
        const int row = r + u * RPP;
        if (row < len) __builtin_nontemporal_store(__builtin_bit_cast(uintx4_t, w[u]), reinterpret_cast<uintx4_t*>(vdst + (int64_t)row * p.vsn));
      }
    }
  }
  for (int r = rr; !TOGETHER && r < len; r += RPP * UNROLL) {
    uint4 v[UNROLL];
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const int row = r + u * RPP;
      if (row < len) v[u] = load_stream16(vsrc + (int64_t)row * p.nsn);
    }
#pragma unroll
    for (int u = 0; u < UNROLL; ++u) {
      const int row = r + u * RPP;
      if (row < len) __builtin_nontemporal_store(__builtin_bit_cast(uintx4_t, v[u]), reinterpret_cast<uintx4_t*>(vdst + (int64_t)row * p.vsn));
    }
  }
  if (!p.kbar) return;  // uniform over the launch
#pragma unroll
  for (int e = 0; e < 8; ++e) red[rr * D + c * 8 + e] = acc[e];
  __syncthreads();
  if (live && prompt && t < D) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < RPP; ++i) s += red[i * D + t];
    p.kbar[((int64_t)h * p.n_b + b) * D + t] = s / (float)len;
  }
}

}  // namespace focus
