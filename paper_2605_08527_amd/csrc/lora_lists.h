// The row tiles' lists of extra contraction tiles for the large-batch GEMM (gemm_wide.hip).
#pragma once
#include "gemm_args.h"

namespace marlaas {

// The list of one row tile by one wave, a lane per adapter.  The rows are grouped by adapter, so the segments
// that intersect a tile belong to consecutive adapters; each is cut into 64-wide pieces of its 2 r_pad extra
// contraction values.  Record 0 holds the count (-1: more than the list holds).
__device__ __forceinline__ void lora_tile_list(const int32_t* __restrict__ seg_off, int n_adapters, const AdapterEntry* __restrict__ table,
                                               int which, int rows, int tile, int lane, LoraTile* __restrict__ out) {
  LoraTile* o = out + (int64_t)tile * (LT_MAX + 1);
  const int64_t m0 = (int64_t)tile * rows;
  const int64_t T_lora = seg_off[n_adapters];
  const int64_t m_end = m0 + rows < T_lora ? m0 + rows : T_lora;
  int cnt = 0;
  if (m0 < m_end) {
    for (int t0 = segment_of(seg_off, n_adapters, (int)m0); t0 < n_adapters; t0 += 64) {
      const int t = t0 + lane;
      int64_t lo = 0, hi = 0;
      int pieces = 0;
      AdapterEntry e;
      e.rank = 0;
      if (t < n_adapters) {
        lo = seg_off[t]; hi = seg_off[t + 1];
        if (lo < m0) lo = m0;
        if (hi > m_end) hi = m_end;
        e = table[t];
        if (hi > lo) pieces = (2 * ((e.rank + 15) & ~15) + 63) / 64;
      }
      int inc = pieces;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) { const int v = __shfl_up(inc, d); if (lane >= d) inc += v; }
      for (int p = 0, at = cnt + inc - pieces; p < pieces && at < LT_MAX; ++p, ++at) {
        LoraTile r;
        r.L = (uint64_t)(uintptr_t)(which ? e.B : e.A);
        r.lo = (int32_t)lo; r.hi = (int32_t)hi; r.kc = p * 64; r.rank = e.rank; r.pad[0] = r.pad[1] = 0;
        o[1 + at] = r;
      }
      cnt += __shfl(inc, 63);
      if (__ballot(t < n_adapters && (int64_t)seg_off[t + 1] < m_end) != ~0ull) break;   // the tile ends inside these
    }
  }
  if (lane == 0) {
    LoraTile r;
    r.L = 0; r.lo = cnt > LT_MAX ? -1 : cnt; r.hi = r.kc = r.rank = 0; r.pad[0] = r.pad[1] = 0;
    o[0] = r;
  }
}

}  // namespace marlaas
