// u = scale x L of a few rows inside the kernels that finish a call in one launch (few rows, some more rows).
#pragma once
#include "common.h"
#include "agent_memory.h"

namespace marlaas {

// One workgroup's share of u: 16 ranks (q0 ..) of one adapter for its rows [row0, row1) of a row tile, which
// lie in one or two neighbouring 16-row blocks, over part `split` of S of the contraction.
struct ShrinkJob {
  const bf16_t* L;                 // the adapter's factor [rank][Kc]
  float scale;
  int rank, q0, row0, row1, split;
};

// Whether a job requests its operands a row at a time (ROWS below): with more than four steps a wave, more than eight rows (of
// fewer, most lanes in operand order repeat the first row, which is no look-up of its own: 281 rows of 92 adapters of rank 64, q/k/v of
// 5992 + 976 + 976 columns, contraction 1864, 74.4 us with, 71.5 without; 408 rows of 50 adapters of rank 32, 4112 x 10648, 78.2 and 75.1;
// 34 rows of 19 of rank 64, 6432 x 3240, 23.8 and 23.1; from 18 steps a wave on more than four: 512 rows of 64 adapters of ranks 8 to 64, 5120 x
// 5120, with their regrouping 69.9, in operand order 71.4, 21 other sizes of such jobs 1.0025 of the time, from memory 1.0006, of
// shorter jobs 1.007, up to 1.17), and no more than 640 workgroups in the launch (beyond, nobody waits for a
// single job, and what counts is what all of them do: 382 rows of 9 adapters of rank 128, q/k/v of 5152 + 960 + 960 columns, contraction
// 1400, 47.8 and 43.3 us; of 420 sizes those of 384 to 800 workgroups take 0.992 of the time with, of more 1.014).
__host__ __device__ inline bool shrink_rows(int64_t Kc, int S, int rows, int workgroups) {
  const int64_t part = (((Kc + 31) >> 5) + S - 1) / S;
  return rows > (part >= 18 * 8 ? 4 : 8) && workgroups <= 640 && part > 4 * 8;
}
// Whether the consumers of the kernel for few rows request x a row at a time (rows_to_operand): from 17 rows on with more than eight
// 32-deep steps a wave; 8 to 16 rows only where rows lie a multiple of 2 KB apart (neighbours in operand order then share the L1's
// sets), by rows times steps.  980 sizes without and with it, 1 to 32 rows, a graph of 16 calls: 32 rows, 4096 x 4096, 16.2 and 13.7 us,
// 3072 x 1280 11.7 and 8.7, 17 to 32 rows of other pitches, nine to eleven steps 0.97 of the time, from memory 1.00, more of them 0.93
// to 0.98; 16 rows, 4096 x 4096, 12.4 and 11.5, 10 rows, 5120 values, 0.95, 4096 values 1.00; other pitches up to 16 rows 0.99 to
// 1.00, from memory 1.00 to 1.02; 1 to 6 rows 1.01 to 1.03.
inline bool thin_rows(int64_t T, int64_t Kc, int64_t lda) {
  const int64_t steps = ((Kc + 31) / 32 + 7) / 8;
  return T > 16 ? steps > 8 : T >= 8 && lda % 1024 == 0 && T * steps > 192;
}
// Eight waves share the part's 32-deep steps, their sums meet in `red` (8 x NB x 64) and are added in wave
// order: the bits do not depend on who computes the job.  u(): [row of the tile][r_stride] of this split; ask() requests what
// u() needs, behind the first operands, which would have to wait for it.  Every wave has called u() when the waves meet, so that
// behind the job whoever likes may change what u() reads.  No value is stored as zero bits.  tok0, tok1: tokens of row
// lane % 16 of the first and of the second block.
// ROWS (shrink_rows): operands are requested a row at a time and put in order through LDS
// (rows_to_operand): 157 rows, 14336 x 4096, 32 adapters of rank 16, 42.4 -> 40.2 us, q/k/v of 157 rows 26.5 -> 25.1, 512 rows, 5120 x
// 5120, 64 adapters, in tiles of 96 rows 55.8 -> 53.4; with four steps the trip costs what it saves (256 rows, 4096 x 4096, 21.4 and 21.5).
// UP: steps requested together (twice); NB: blocks a job can have.  All eight waves call it.
template <int UP, int NB, bool ROWS = false, typename Ask, typename At>
__device__ __forceinline__ void shrink_job(const ShrinkJob& j, const bf16_t* X, int64_t lda, int64_t Kc, int32_t tok0, int32_t tok1, int S,
                                           f32x4* red, Ask ask, At u, int r_stride, int wave, int lane) {
  constexpr int WAVES = 8;
  union Frag { uint4 u; bf16x8 v; };
  const int li = lane & 15, lg = lane >> 4;
  const int steps = (int)((Kc + 31) >> 5), part = (steps + S - 1) / S;
  const int k0 = j.split * part, k1 = k0 + part < steps ? k0 + part : steps;
  const int per = (part + WAVES - 1) / WAVES;
  const int s0 = k0 + wave * per, s1 = s0 + per < k1 ? s0 + per : k1;
  const int blk = j.row0 >> 4;
  const bool two = (j.row1 - 1) >> 4 > blk;
  // (rows of others read the job's first row in the block, in a tile of many adapters most of it, and are not stored;
  // one block of few rows has its start delayed by the exchange: 11.6 -> 11.7 us for 6 rows)
  if constexpr (NB > 1) {
    const int r0 = blk * 16 + li, r1 = r0 + 16;
    const int32_t first0 = __shfl(tok0, j.row0 & 15), first1 = __shfl(tok1, 0);
    if (r0 < j.row0 || r0 >= j.row1) tok0 = first0;
    if (r1 >= j.row1) tok1 = first1;
  }
  // (ROWS: lane / 4 is the row that a lane requests and lane % 4 its eight values, put in order through this wave's part of red)
  const int lr = ROWS ? lane >> 2 : li, lk = ROWS ? lane & 3 : lg;
  if (ROWS) { tok0 = __shfl(tok0, lr); tok1 = __shfl(tok1, lr); }
  const bool row_in = j.q0 + lr < j.rank;
  char* const stage = (char*)(red + wave * NB * 64);
  const bf16_t* lrow = j.L + (int64_t)(row_in ? j.q0 + lr : 0) * Kc;
  const bf16_t* xrow[2] = {X + (int64_t)tok0 * lda, X + (int64_t)tok1 * lda};
  f32x4 acc[NB];
#pragma unroll
  for (int b = 0; b < NB; ++b) acc[b] = f32x4{0.f, 0.f, 0.f, 0.f};
  Frag fa[UP][NB + 1], fb[UP][NB + 1];
  auto request = [&](Frag (&f)[UP][NB + 1], int s) {
#pragma unroll
    for (int i = 0; i < UP; ++i) {
      const int64_t k = (int64_t)(s + i) * 32 + 8 * lk;
#pragma unroll
      for (int b = 0; b <= NB; ++b) f[i][b].u = make_uint4(0, 0, 0, 0);
      if (s + i < s1 && k < Kc) {
        if (row_in) f[i][NB].u = *(const uint4*)(lrow + k);
#pragma unroll
        for (int b = 0; b < NB; ++b) if (b == 0 || two) f[i][b].u = *(const uint4*)(xrow[b] + k);
      }
    }
  };
  auto multiply = [&](Frag (&f)[UP][NB + 1]) {
#pragma unroll
    for (int i = 0; i < UP; ++i) {
      if (ROWS) {
#pragma unroll
        for (int b = 0; b <= NB; ++b) if (b != 1 || NB == 1 || two) f[i][b].u = rows_to_operand(stage, f[i][b].u, lane);
      }
#pragma unroll
      for (int b = 0; b < NB; ++b) acc[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f[i][NB].v, f[i][b].v, acc[b], 0, 0, 0);
    }
  };
  request(fa, s0);
  ask();
#pragma unroll 1
  for (int s = s0; s < s1; s += 2 * UP) {
    if (s + UP < s1) request(fb, s + UP);
    multiply(fa);
    if (s + UP < s1) {
      if (s + 2 * UP < s1) request(fa, s + 2 * UP);
      multiply(fb);
    }
  }
#pragma unroll
  for (int b = 0; b < NB; ++b) red[(wave * NB + b) * 64 + lane] = acc[b];
  float* const u_at = u();
  __syncthreads();
  if (wave < NB) {                                               // wave b finishes block blk + b
    f32x4 s = red[wave * 64 + lane];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) {
      const f32x4 o = red[(w * NB + wave) * 64 + lane];
      s[0] += o[0]; s[1] += o[1]; s[2] += o[2]; s[3] += o[3];
    }
    // lane: row li of the block, ranks q0 + 4 lg .. + 3
    const int row = (blk + wave) * 16 + li;
    if (row >= j.row0 && row < j.row1) {
      f32x4 f;
#pragma unroll
      for (int v = 0; v < 4; ++v) { const float z = j.scale * s[v]; f[v] = __float_as_uint(z) == 0u ? -0.f : z; }
      store4_agent(u_at + (int64_t)row * r_stride + j.q0 + 4 * lg, f);
    }
  }
}

// Four values of u in S pieces (1, 2 or 4), added in their order; false if they are not there after `polls` readings (a
// round trip through the fabric each; as many requests as pieces: four for one piece cost 51 rows of 64 adapters of rank 64, 1384 x
// 8344, 28.2 -> 29.0 us).
template <int S>
__device__ __forceinline__ bool read_u_pieces(const float* u, int64_t u_split, int polls, f32x4& v) {
  static_assert(S == 1 || S == 2 || S == 4, "");
  const float* u1 = u + u_split;
  const float* u2 = u1 + u_split;
  const float* u3 = u2 + u_split;
  for (int it = 0; it < polls; ++it) {
    f32x4 w[S];
    if constexpr (S == 1)
      asm volatile("global_load_dwordx4 %0, %1, off sc1\n\ts_waitcnt vmcnt(0)" : "=&v"(w[0]) : "v"(u) : "memory");
    else if constexpr (S == 2)
      asm volatile("global_load_dwordx4 %0, %2, off sc1\n\tglobal_load_dwordx4 %1, %3, off sc1\n\ts_waitcnt vmcnt(0)"
                   : "=&v"(w[0]), "=&v"(w[1]) : "v"(u), "v"(u1) : "memory");
    else
      asm volatile("global_load_dwordx4 %0, %4, off sc1\n\tglobal_load_dwordx4 %1, %5, off sc1\n\t"
                   "global_load_dwordx4 %2, %6, off sc1\n\tglobal_load_dwordx4 %3, %7, off sc1\n\ts_waitcnt vmcnt(0)"
                   : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]) : "v"(u), "v"(u1), "v"(u2), "v"(u3) : "memory");
    bool ok = true;
#pragma unroll
    for (int k = 0; k < S; ++k)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        ok &= __float_as_uint(w[k][j]) != 0u;
        v[j] = k == 0 ? w[0][j] : v[j] + w[k][j];
      }
    if (ok) return true;
  }
  return false;
}

__device__ __forceinline__ bool read_u(const float* u, int64_t u_split, int S, int polls, f32x4& v) {
  return S == 1 ? read_u_pieces<1>(u, u_split, polls, v) : S == 2 ? read_u_pieces<2>(u, u_split, polls, v) : read_u_pieces<4>(u, u_split, polls, v);
}

// The same values computed by the wave that wants them (they did not come in time: no workgroup depends on another
// one being scheduled), with the sums in the order of shrink_job.  Lane: ranks q .. q + 3 of row `row` of the tile,
// `miss` if it lacks them.  t_s, tok_s: adapter (-1: none) and token (-1: past the end) of the tile's rows.  All
// lanes of the wave call it.
__device__ __forceinline__ void u_again(const AdapterEntry* table, int which, const bf16_t* X, int64_t lda, int64_t Kc, int S, const int32_t* t_s,
                                        const int32_t* tok_s, int row, int q, bool miss, int lane, f32x4& v) {
  constexpr int WAVES = 8;
  const int li = lane & 15, lg = lane >> 4;
  const int steps = (int)((Kc + 31) >> 5), part = (steps + S - 1) / S, per = (part + WAVES - 1) / WAVES;
#pragma unroll 1
  for (uint64_t left = __ballot(miss); left; left = __ballot(miss)) {
    const int l = __ffsll((unsigned long long)left) - 1;
    const int r = __builtin_amdgcn_readlane(row, l), q0 = __builtin_amdgcn_readlane(q, l) & ~15;
    const int t = __builtin_amdgcn_readfirstlane(t_s[r]);
    const AdapterEntry e = table[t];
    const int32_t tk = tok_s[(r & ~15) + li], own = tok_s[r];
    const bf16_t* xr = X + (int64_t)(tk < 0 ? own : tk) * lda;
    const bool row_in = q0 + li < e.rank;
    const bf16_t* lr = (const bf16_t*)(which ? e.A : e.B) + (int64_t)(row_in ? q0 + li : 0) * Kc;
    f32x4 u = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
    for (int split = 0; split < S; ++split) {
      const int k0 = split * part, k1 = k0 + part < steps ? k0 + part : steps;
      f32x4 sum = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
      for (int w = 0; w < WAVES; ++w) {
        const int s0 = k0 + w * per, s1 = s0 + per < k1 ? s0 + per : k1;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int st = s0; st < s1; ++st) {
          union { uint4 u; bf16x8 v; } lf, xf;
          const int64_t k = (int64_t)st * 32 + 8 * lg;
          lf.u = xf.u = make_uint4(0, 0, 0, 0);
          if (k < Kc && row_in) lf.u = *(const uint4*)(lr + k);
          if (k < Kc) xf.u = *(const uint4*)(xr + k);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lf.v, xf.v, acc, 0, 0, 0);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) sum[i] = w == 0 ? acc[i] : sum[i] + acc[i];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float z = e.scale * sum[i], f = __float_as_uint(z) == 0u ? -0.f : z;
        u[i] = split == 0 ? f : u[i] + f;
      }
    }
    // lane li + 16 lg holds ranks q0 + 4 lg .. of row li of the block
    const bool mine = miss && (row & ~15) == (r & ~15) && (q & ~15) == q0 && t_s[row] == t;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float got = __shfl(u[i], (row & 15) + 4 * (q & 12));
      if (mine) v[i] = got;
    }
    if (mine) miss = false;
  }
}

}  // namespace marlaas
