// Expand of 16 rows by their own adapters' factors on the matrix instructions, for the kernels that finish
// rows of several adapters at once (few rows, some more rows, decode).
#pragma once
#include "common.h"

namespace marlaas {

// u as a two-term bf16 split, hi = bf16(u), lo = bf16(u - hi) (relative error 2^-17).
// Four ranks of a row: the first terms at p, the second ones `lo` values behind.
__device__ __forceinline__ void store_split4(bf16_t* p, int lo, f32x4 v) {
  uint32_t h[2], l[2];
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const uint32_t h0 = float_to_bf16_bits(v[2 * e]), h1 = float_to_bf16_bits(v[2 * e + 1]);
    h[e] = h0 | (h1 << 16);
    l[e] = float_to_bf16_bits(v[2 * e] - __uint_as_float(h0 << 16)) | ((uint32_t)float_to_bf16_bits(v[2 * e + 1] - __uint_as_float(h1 << 16)) << 16);
  }
  *(uint2*)p = make_uint2(h[0], h[1]);
  *(uint2*)(p + lo) = make_uint2(l[0], l[1]);
}
// Eight ranks of a row that store_split4 left at p; zeros where `mine` is not set.
__device__ __forceinline__ void load_split(const bf16_t* p, int lo_at, bool mine, bf16x8& hi, bf16x8& lo) {
  union { uint4 u; bf16x8 v; } h, l;
  h.u = *(const uint4*)p; l.u = *(const uint4*)(p + lo_at);
  h.u.x = mine ? h.u.x : 0; h.u.y = mine ? h.u.y : 0; h.u.z = mine ? h.u.z : 0; h.u.w = mine ? h.u.w : 0;
  l.u.x = mine ? l.u.x : 0; l.u.y = mine ? l.u.y : 0; l.u.z = mine ? l.u.z : 0; l.u.w = mine ? l.u.w : 0;
  hi = h.v; lo = l.v;
}
// Eight ranks of a row's fp32 u; zeros where `mine` is not set.
__device__ __forceinline__ void split_u(const float* u, bool mine, bf16x8& hi, bf16x8& lo) {
  const f32x4 ua = *(const f32x4*)u, ub = *(const f32x4*)(u + 4);
  const float uv[8] = {ua[0], ua[1], ua[2], ua[3], ub[0], ub[1], ub[2], ub[3]};
  union { uint32_t w[4]; bf16x8 v; } h, l;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float v0 = mine ? uv[2 * e] : 0.f, v1 = mine ? uv[2 * e + 1] : 0.f;
    const uint32_t h0 = float_to_bf16_bits(v0), h1 = float_to_bf16_bits(v1);
    h.w[e] = h0 | (h1 << 16);
    l.w[e] = float_to_bf16_bits(v0 - __uint_as_float(h0 << 16)) | ((uint32_t)float_to_bf16_bits(v1 - __uint_as_float(h1 << 16)) << 16);
  }
  hi = h.v; lo = l.v;
}

// y[cb] (16 columns each; lane: row lane % 16, columns 4 (lane / 16) .. + 3) += u L of the rows' adapters.
//   cnt      octets (8 ranks of one adapter) of the block's adapters; lane group lg supplies octet k0 + lg
//   t_row    adapter of this lane's row; split(q, mine, hi, lo): ranks q .. q + 7 of its u in two terms, zeros where not `mine`
//   oct(i)   adapter << 8 | first rank of octet i
//   load(i, cb)  8 ranks of octet i in column lane % 16 of block cb (zeros beyond the last column)
//   pre[k]   load(4 k + lg, cb) where 4 k + lg < cnt, requested before; further steps are requested KB at a time
// One product takes four octets, whose adapters may differ: the others' u is 0.  0 times a factor that is
// infinite or not a number is not 0, so where a sum comes out like that the block is done again, one
// adapter at a time, and a row takes its own adapter's products only: the same bits as with finite factors
// for everyone else.  The test costs eight fused multiply-adds a call.
template <int NCB, int KB, typename Split, typename Oct, typename Load>
__device__ __forceinline__ void expand_octets(f32x4 (&y)[NCB], uint4 (&pre)[KB][NCB], int cnt, int lg, int t_row, Split split, Oct oct, Load load) {
  union Frag { uint4 u; bf16x8 v; };
  f32x4 was[NCB];
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) was[cb] = y[cb];
  for (int b0 = 0; b0 < cnt; b0 += 4 * KB) {
#pragma unroll
    for (int k = 0; k < KB; ++k)
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb)
        if (b0 > 0) pre[k][cb] = b0 + 4 * k + lg < cnt ? load(b0 + 4 * k + lg, cb) : make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int k = 0; k < KB; ++k) {
      const int k0 = b0 + 4 * k;
      if (k0 >= cnt) break;
      const bool valid = k0 + lg < cnt;
      const int o = oct(valid ? k0 + lg : 0);
      bf16x8 hi, lo;
      split(o & 255, valid && t_row == o >> 8, hi, lo);
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        Frag f;
        f.u = pre[k][cb];
        y[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.v, lo, y[cb], 0, 0, 0);
        y[cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.v, hi, y[cb], 0, 0, 0);
      }
    }
  }
  float z = 0.f;                                                 // (0 unless a sum is infinite or not a number)
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
    for (int v = 0; v < 4; ++v) z = fmaf(y[cb][v], 0.f, z);
  if (__builtin_expect(__ballot(z != 0.f) == 0, 1)) return;
#pragma unroll
  for (int cb = 0; cb < NCB; ++cb) y[cb] = was[cb];
#pragma unroll 1
  for (int k0 = 0; k0 < cnt; k0 += 4) {
    const bool valid = k0 + lg < cnt;
    const int i = valid ? k0 + lg : 0;
    const int o = oct(i);
    const int t = valid ? o >> 8 : -1;
    bf16x8 hi, lo;
    split(o & 255, valid && t_row == t, hi, lo);
    int before = -1;
#pragma unroll 1
    for (int j = 0; j < 4; ++j) {
      const int tj = __builtin_amdgcn_readlane(t, 16 * j);       // (an adapter's octets are neighbours)
      if (tj < 0 || tj == before) continue;
      before = tj;
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        Frag f, g;                                               // (g: an infinite factor meets only the leading term of u,
        f.u = make_uint4(0, 0, 0, 0);                            // as it would the unsplit u)
        if (t == tj) f.u = load(i, cb);
        const uint32_t w[4] = {f.u.x, f.u.y, f.u.z, f.u.w};
        uint32_t d[4];
#pragma unroll
        for (int e = 0; e < 4; ++e)
          d[e] = ((w[e] & 0x7f80u) == 0x7f80u ? 0u : w[e] & 0xffffu) | ((w[e] & 0x7f800000u) == 0x7f800000u ? 0u : w[e] & 0xffff0000u);
        g.u = make_uint4(d[0], d[1], d[2], d[3]);
        f32x4 s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(g.v, lo, y[cb], 0, 0, 0);
        s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.v, hi, s, 0, 0, 0);
#pragma unroll
        for (int v = 0; v < 4; ++v) y[cb][v] = t_row == tj ? s[v] : y[cb][v];
      }
    }
  }
}

}  // namespace marlaas
