// Decode of some 64 to 1000 rows on the packed weight: the whole call in one launch.
//
//   out_p[tok(m), :] = x[tok(m), :] W_p  +  u_p(m) L_{t,p}        for every projection p of the call
//
// A workgroup owns a tile of 16 RB rows x 32 WN columns; its eight waves are WN column groups of 32 times
// KG = 8 / WN contraction groups, so a weight fragment is read once, by the one wave that multiplies it,
// and the sums of the contraction groups meet in LDS.  x goes through LDS by DMA in a ring of 128-deep
// tiles, because every column group needs all of it.  What bounds it: the fabric between the memory and the
// eight L2s (256 rows of 4096 x 4096 fetch 66.7 MB by the counters: the weight 33.5, x 2.1 for each XCD, the
// factors and what is read again), and below its rate every dependent trip through it, 1 to 1.5 us each, and
// every launch, about 4 us.  So: no second launch, few contraction splits, tiles small enough that two
// workgroups share a compute unit (128 registers, 80 KB of LDS).
//
// Measured (microseconds, before: extended columns through the split kernel and a second launch): 256 rows
// 4096 x 4096 with 32 adapters of rank 16 28.4 -> 21.5, q/k/v of 4096 + 1024 + 1024 columns 42.0 -> 29.8, the
// four calls of a decoder layer (4096, ffn 14336) of 157 rows 252 -> 190, 512 rows of 64 adapters of ranks 8
// to 64, 5120 x 5120, 62 (weights from memory).  Stamps in the 256 rows (a workgroup in the middle, the last one): indices
// 2.0, 2.4; first tile 3.8, 6.3 (a producer shares the unit; u is out after 5.6, 7.2); loop done 15.0, 17.3; sums met
// 15.6, 17.8; u in LDS 17.4, 19.4; expanded 17.8, 19.9; stored 18.2, 20.3.  q/k/v: first tile 4.7, 13.7; loop 19.4, 25.9; u in LDS
// 21.7, 28.4; stored 22.6, 29.3.
// What the last changes gave, each against a build without it: turns instead of a count (agent_memory.h); u in two terms once a
// row, on its way into LDS, not once a wave (100 rows of 32 adapters of rank 64, 4096 x 4096, 28.9 -> 28.2; q/k/v and 256 rows of
// rank 16 no more than runs differ); octet steps requested together (KB below).
//
// Tall tiles (gemm_tall.hip): 96 x 128 in the registers that two workgroups a unit have, 128 160 and 256 x 128 with a unit each.  A
// unit's time goes by what comes into it, 32, 36 or 48 KB for 64 values of a contraction where two workgroups of 80 rows take 52, and by how
// even the tiles fall on the 256 units.  Products by inline assembly: left to the compiler, sums moved between registers and 96
// rows spilled 12 of them, requests under way among those.  512 rows of 64 adapters of ranks 8 to 64, 5120 x 5120, 61.1 -> 52.4 us in 240 tiles of 96
// rows (280 of 80 before); 157 rows, 4096 x 28672, 32 adapters of rank 16, 72 -> 62, weights from memory 80 -> 68.6; 256 rows 105 -> 78, from memory 112 -> 81.  A ring of six k-tiles in
// place of four is no faster (256 rows, 4096 x 14336, 35.0 and 36.7).
//
// Whatever crosses workgroups carries its own flag: it travels through areas of the context that are all
// zero bits when a launch finds them, no value is stored as zero bits (+0 becomes -0), and a reader reads until
// nothing is zero bits any more.
//   u: workgroups before the others ("producers") compute it, one per 16 ranks of an adapter and pair of
//     16-row blocks of a row tile (and piece of a long contraction).  There are as many as any grouping of the
//     rows needs and each finds its share in the segment map, so that a captured call serves the groupings
//     that the map object gets later.  Launches take turns over two areas, and each clears the other's (agent_memory.h).
//   partial sums: with ksplit > 1 the splits of a tile share out its 16 x 16 units; a split hands the
//     others' units over, reads its own ones' missing sums and clears them.
// The reading is bounded (MID_POLLS).  u that does not come in time is computed by the reader; so are missing
// sums, and the next launch then clears their area and computes all of its sums where they are wanted.  No workgroup depends
// on another one being scheduled, and either way the sums are added in the same order: the bits are the same.
#pragma once
#include "gemm_args.h"
#include "agent_memory.h"
#include "lora_expand.h"
#include "lora_shrink.h"
#include "mid_plan.h"

#include <atomic>

namespace marlaas {

// (a value the compiler cannot compute ahead of its use and keep in a register until then)
__device__ __forceinline__ int fresh(int v) { asm volatile("" : "+v"(v)); return v; }

// 16 bytes per lane from base + ofs (or p) to LDS bytes lds .. lds + 1023
__device__ __forceinline__ void dma16(uint32_t lds, const char* base, uint32_t ofs) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(lds), "v"(ofs), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ void dma16(uint32_t lds, const char* p) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(lds), "v"(p) : "memory", "m0");
}

// c += a b.  Tall tiles: by inline assembly, so that the sums stay where they are.
template <bool PLAIN>
__device__ __forceinline__ void md_product(f32x4& c, bf16x8 a, bf16x8 b) {
  if constexpr (PLAIN) c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
  else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b));
}

static constexpr int MD_THREADS = 512, MD_WAVES = MID_WAVES;

template <int RB, int WN>
struct MidShape {
  static constexpr int KG = MD_WAVES / WN, K = 32 * KG;           // contraction groups; contraction values of a k-tile
  static constexpr bool SPLITS = RB <= 5;               // (the contraction may be split over workgroups; the others are "tall")
  static constexpr int PER_UNIT = RB <= 6 ? 2 : 1;      // workgroups that a compute unit has room for
  static constexpr int NS = RB == 4 || (RB == 5 && WN == 4) || (RB > 6 && RB < 14) ? 4 : 3; // ring slots = k-tiles on the way (registers, LDS)
  static constexpr int SLOT = RB * 16 * K * 2;
  static constexpr int RED = RB * WN * 2 * (KG - 1) * 1024;       // exchange of the contraction groups
};

// Job `job` of a projection's shrink, counted over all row tiles (16 RB rows each): 16 ranks of an adapter for its
// rows in a pair of row blocks (32 rows of a tile from a multiple of 32 on).  Fills in *j (but for the split)
// and returns the row tile, -1: there are fewer jobs.  Rows are grouped by adapter, so a lane per adapter
// counts its pairs from its rows' ends alone; where the adapters are more than the lanes a thread counts
// those of two rows (tmp: 16 ints of LDS).  All waves call it.
template <int RB>
__device__ __forceinline__ int find_job(const GemmArgs& a, const AdapterEntry* table, int job, int32_t* tmp, int wave, int lane, ShrinkJob* j) {
  constexpr int BM = 16 * RB, PAIRS = (RB + 1) / 2;
  int lo = 0, hi = 0;                                            // rows of the job's adapter
  int pair = -1;                                                 // pair of row blocks, counted over all row tiles
  auto pair_of = [&](int m) { return (int)((uint32_t)m / BM * PAIRS + (uint32_t)m % BM / 32); };
  AdapterEntry e;
  e.A = e.B = nullptr; e.rank = 0; e.scale = 0.f;
  if (a.n_adapters <= 64) {
    const bool in = lane < a.n_adapters;
    const int so = in ? a.seg_off[lane] : 0, so1 = in ? a.seg_off[lane + 1] : 0;
    if (in) e = table[lane];
    const int p0 = pair_of(so), pairs = so1 > so ? pair_of(so1 - 1) - p0 + 1 : 0;
    const int jobs = pairs * ((e.rank + 15) >> 4);
    int inc = jobs;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) { const int v = __shfl_up(inc, d); if (lane >= d) inc += v; }
    const uint64_t hit = __ballot(inc - jobs <= job && job < inc);
    if (hit == 0) return -1;
    const int l = __ffsll((unsigned long long)hit) - 1;
    const int k = job - __shfl(inc - jobs, l), np = __shfl(pairs, l);
    lo = __shfl(so, l); hi = __shfl(so1, l);
    pair = __shfl(p0, l) + k % np;
    j->q0 = k / np * 16;
    j->rank = __shfl(e.rank, l); j->scale = __shfl(e.scale, l);
    const uint64_t fp = (uint64_t)(uintptr_t)(a.which ? e.A : e.B);
    j->L = (const bf16_t*)(((uint64_t)(uint32_t)__shfl((int)(fp >> 32), l) << 32) | (uint32_t)__shfl((int)fp, l));
  } else {
    const int m = 2 * (wave * 64 + lane);
    static_assert(MID_ROWS <= 2 * MD_THREADS && BM % 2 == 0, "two rows a thread");
    const int g0 = m < a.T ? a.grp_ids[m] : -1, g1 = m + 1 < a.T ? a.grp_ids[m + 1] : -1, gb = m > 0 && m < a.T ? a.grp_ids[m - 1] : -1;
    const int n0 = g0 >= 0 && (g0 != gb || m % BM % 32 == 0) ? (table[g0].rank + 15) >> 4 : 0;
    const int n1 = g1 >= 0 && g1 != g0 ? (table[g1].rank + 15) >> 4 : 0;
    int inc = n0 + n1;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) { const int v = __shfl_up(inc, d); if (lane >= d) inc += v; }
    if (lane == 63) tmp[wave] = inc;
    if (wave == 0 && lane < 2) tmp[MD_WAVES + lane] = -1;
    __syncthreads();
    int k = job - (inc - n0 - n1);
    for (int w = 0; w < wave; ++w) k -= tmp[w];
    if (k >= 0 && k < n0 + n1) { tmp[MD_WAVES] = k < n0 ? m : m + 1; tmp[MD_WAVES + 1] = k < n0 ? k : k - n0; }
    __syncthreads();
    const int row = tmp[MD_WAVES];
    if (row < 0) return -1;
    const int t = a.grp_ids[row];
    e = table[t];
    lo = row; hi = a.seg_off[t + 1];
    pair = pair_of(row);
    j->q0 = tmp[MD_WAVES + 1] * 16;
    j->rank = e.rank; j->scale = e.scale;
    j->L = (const bf16_t*)(a.which ? e.A : e.B);
    __syncthreads();                                             // (tmp is free)
  }
  const int tm = pair / PAIRS, m0 = tm * BM, r0 = pair % PAIRS * 32, end = r0 + 32 < BM ? r0 + 32 : BM;
  j->row0 = lo > m0 + r0 ? lo - m0 : r0;
  j->row1 = hi < m0 + end ? hi - m0 : end;
  return tm;
}

// LDS: the ring or, once it is free, the exchange of the sums and, behind it, the rows' u; in place of it where
// two workgroups would not fit a compute unit otherwise (80-row tiles of 64 columns: ranks above 48; 64 x 64 and 80 x
// 128: above 96); the rows' tables.
template <int RB, int WN>
__host__ __device__ inline int mid_tables(int r_stride) { return 16 * RB * 20 + RB * 4 + RB * 2 * r_stride * (int)sizeof(uint16_t); }
template <int RB, int WN>
__host__ __device__ inline int mid_sums(int r_stride) {
  const int u = 16 * RB * (r_stride + 4) * (int)sizeof(float), red = MidShape<RB, WN>::RED;
  return red + u + mid_tables<RB, WN>(r_stride) <= 160 / MidShape<RB, WN>::PER_UNIT * 1024 ? red + u : red > u ? red : u;
}

template <int RB, int WN>
__global__ __launch_bounds__(MD_THREADS, (2 * MidShape<RB, WN>::PER_UNIT)) void gemm_mid_kernel(GemmArgs a) {
  typedef MidShape<RB, WN> S_;
  constexpr int KG = S_::KG, MD_K = S_::K, UR = MD_K / 8, NS = S_::NS, SLOT = S_::SLOT, BM = 16 * RB, NR = (RB + KG - 1) / KG;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  const int us = a.r_stride + 4, oct_max = 2 * a.r_stride;       // (octet: 8 ranks of one adapter; so many can a 16-row block have)
  const int sums = mid_sums<RB, WN>(a.r_stride), base_bytes = NS * SLOT > sums ? NS * SLOT : sums;
  const bool apart = sums == S_::RED + BM * us * 4;
  f32x4* red = (f32x4*)smem;
  float* u_s = (float*)(smem + (apart ? S_::RED : 0));           // [BM][us]: the rows' u
  uint64_t* rL_s = (uint64_t*)(smem + base_bytes);               // per row: expand factor,
  int32_t* tok_s = (int32_t*)(rL_s + BM);                        // token (-1: past the end),
  int32_t* t_s = tok_s + BM;                                     // adapter (-1: none),
  int32_t* rank_s = t_s + BM;                                    // rank
  int32_t* cnt_s = rank_s + BM;                                  // [RB] octets of a row block (-1: plain expand)
  uint16_t* oct_s = (uint16_t*)(cnt_s + RB);                     // [RB][oct_max]: row of the tile << 8 | first rank
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lg = lane >> 4;
  const bool lora = a.n_adapters > 0 && a.table != nullptr;
  const int b = (int)blockIdx.x - a.prod0, S = a.n_split;        // the producers are workgroups prod0 ..
  const int64_t u_n = a.T * a.r_stride;                          // u: [projection][split][T][r_stride], scaled
  constexpr int UNITS = 2 * WN * RB;
  static_assert(!S_::SPLITS || UNITS * 256 <= MID_TILE_FLOATS, "room for the splits' sums");
  auto u_area = [&](int area) { return a.mid_u + area * (int64_t)MID_U_FLOATS; };
  const bool joins = lora || a.ksplit > 1;                       // (exchanges something)
  const int64_t u_all = lora ? (int64_t)a.n_proj * S * u_n : 0;
  const int64_t consumers = (int64_t)gridDim.x - a.n_prod;

  if (b >= 0 && b < a.n_prod) {
    // ---- producers: job b (of those that the rows can have, padded to whole rounds over the XCDs), and where the producers are
    // fewer every n_prod'th behind it
    bool asked = false;
    Turn turn;
    for (int v = b; v < a.n_jobs; v += a.n_prod) {
      const int pp = v / (a.proj_jobs * S);
      ShrinkJob job;
      job.split = v % S;
      const int tile = pp < a.n_proj ? find_job<RB>(a, a.table + a.proj[pp].tab0, v / S - pp * a.proj_jobs, (int32_t*)smem, wave, lane, &job) : -1;
      if (tile >= 0) {                                           // (there are as many as any grouping of T rows needs)
        const int64_t r0 = (int64_t)tile * BM + (job.row0 & ~15) + li, last = a.T - 1;
        const int64_t i0 = r0 < last ? r0 : last, i1 = r0 + 16 < last ? r0 + 16 : last;
        const int32_t tok0 = a.perm ? a.perm[i0] : (int32_t)i0, tok1 = a.perm ? a.perm[i1] : (int32_t)i1;
        int4 line;
        auto ask = [&] { if (!asked) line = *(const int4*)turn_line(a.turns); };
        auto at = [&] {
          if (!asked) turn = turn_of(line.x, line.y, line.z, line.w);
          return u_area(turn.area) + (pp * S + job.split) * u_n + (int64_t)tile * BM * a.r_stride;
        };
        if (shrink_rows(a.Kc, S, job.row1 - job.row0, (int)gridDim.x)) shrink_job<3, 2, true>(job, a.Aop, a.lda, a.Kc, tok0, tok1, S, red, ask, at, a.r_stride, wave, lane);
        else shrink_job<3, 2, false>(job, a.Aop, a.lda, a.Kc, tok0, tok1, S, red, ask, at, a.r_stride, wave, lane);
        asked = true;
      }
      if constexpr (S_::PER_UNIT > 1) break;
      else __syncthreads();                                      // (red and find_job's ints are free)
    }
    if (!asked) turn_missed(a.turns, u_all, tid == 0);
    else if (tid == 0) turn_over(a.turns, turn, u_all);
    return;
  }

  // ---- consumers.  Workgroup b runs on XCD b mod 8.  An XCD works on one contraction split, so that it pulls
  // only its own part of x through the fabric; the row tiles of a column tile are neighbours on one XCD and
  // share the weight through its L2.
  const int c = b < 0 ? (int)blockIdx.x : (int)blockIdx.x - a.n_prod, ng = 8 / a.ksplit;
  const int ks0 = c & (a.ksplit - 1), tm = (c >> 3) % a.tiles_m, tn = (c >> 3) / a.tiles_m * ng + (c & 7) / a.ksplit;
  if (tn >= a.tiles_n) {
    if (joins) {
      const Turn turn = turn_missed(a.turns, u_all, tid == 0);
      clear_share(u_area(1 - turn.area), turn.u_before, c, consumers);
      if (!turn.sums_ok) clear_share(a.partials, MID_PART_FLOATS, c, consumers);
    }
    return;
  }
  int p = 0;
  for (int q = 1; q < a.n_proj; ++q) if (tn >= a.proj[q].tile0) p = q;
  const int64_t m0 = (int64_t)tm * BM;
  const int64_t Nout = a.proj[p].Nout, ldb = a.proj[p].ldw;
  const AdapterEntry* table = a.table + a.proj[p].tab0;
  float* parts = a.partials + (int64_t)(tm * a.tiles_n) * (UNITS * 256) * a.ksplit;    // [tile][unit][split][lane] x 4
  const int steps = (int)((a.Kc + 31) >> 5);
  const bool lead = ks0 == 0 && tn == a.proj[p].tile0;
  const int g = wave / WN, wn = wave % WN;
  const int64_t n0 = (int64_t)(tn - a.proj[p].tile0) * (32 * WN) + 32 * wn;     // this wave's first column
  // the indices everything waits for go first (inline assembly: the compiler's own waits would count the
  // requests below in); row of this lane's part of its DMA requests, row tid of the tables
  // (UR: 16-byte units of a tile's row; a DMA request is 64 of them)
  constexpr int NI = (RB * UR / 4 + 7) / 8;                      // DMA requests of a wave per k-tile,
  const bool full = wave < RB * UR / 4 - 8 * (NI - 1);           // one less for the upper waves where they do not divide
  const int drow = lane / UR, dunit = lane % UR;
#define MD_DROW(i_) ((wave + 8 * (i_)) * (64 / UR) + drow)
#define MD_SWZ(r_) (UR == 16 ? (r_) & 15 : ((r_) >> 1) & 7)
  // (requested by every lane, whether needed or not: a value that a branch merges could be copied before it is there)
  int32_t tokr[NI], tok, gid, gid1;
  const int32_t* none = (const int32_t*)a.zero_line;
#pragma unroll
  for (int i = 0; i < NI; ++i) {
    int64_t m = m0 + MD_DROW(i);
    if (m >= a.T) m = a.T - 1;
    asm volatile("global_load_dword %0, %1, off" : "=v"(tokr[i]) : "v"(a.perm ? a.perm + m : none) : "memory");
  }
  const int64_t mrow = m0 + tid;
  const bool has_row = tid < BM && mrow < a.T;
  const int64_t mr = has_row ? mrow : 0;
  asm volatile("global_load_dword %0, %1, off" : "=v"(tok) : "v"(a.perm ? a.perm + mr : none) : "memory");
  asm volatile("global_load_dword %0, %1, off" : "=v"(gid) : "v"(lora ? a.grp_ids + mr : none) : "memory");
  asm volatile("global_load_dword %0, %1, off" : "=v"(gid1) : "v"(lora ? a.grp_ids + (mr > 0 ? mr - 1 : 0) : none) : "memory");
  // column block cb of this wave is block n0 / 16 + cb of the packed weight (blocks past the last one
  // repeat it: those columns are never stored)
  const bf16_t* wp[2];
#pragma unroll
  for (int cb = 0; cb < 2; ++cb) {
    const int64_t blocks = (Nout + 15) >> 4;
    int64_t nb = (n0 >> 4) + cb;
    if (nb >= blocks) nb = blocks - 1;
    wp[cb] = (const bf16_t*)a.proj[p].W + ((nb * ldb) << 9);
  }
  const int ktiles = (int)((a.Kc + MD_K - 1) / MD_K), chunk = (ktiles + a.ksplit - 1) / a.ksplit;
  bf16x8 wreg[NS][2];
  const int wofs = lane * 16;
  // Weight fragments of k-tile t_ (steps past the end read zeros).  dst_: "+v" inside the loops, which ties a
  // slot to its registers: the compiler must not move a value that is still on its way (the code generated
  // for nested loops with "=v" did, for one of many versions of the code behind them).
#define MD_W(t_, s_, dst_)                                                                                \
  do {                                                                                                    \
    const int _st = (t_) * KG + g;                                                                        \
    _Pragma("unroll") for (int _c = 0; _c < 2; ++_c) {                                                    \
      const bf16_t* _p = _st < steps ? wp[_c] + ((int64_t)_st << 9) : a.zero_line;                        \
      asm volatile("global_load_dwordx4 %0, %1, %2" : dst_(wreg[s_][_c]) : "v"(wofs), "s"(_p) : "memory"); \
    }                                                                                                     \
  } while (0)
  // x of k-tile t_ into slot s_: row r of the tile at 16 UR r, its 16-byte unit u at place u ^ MD_SWZ(r)
  // (units past the end read zeros)
#define MD_X(t_, s_)                                                                                      \
  do {                                                                                                    \
    const bool _past = (int64_t)((t_) + 1) * MD_K > a.Kc;                                                 \
    _Pragma("unroll") for (int _i = 0; _i < NI; ++_i)                                                        \
      if (_i + 1 < NI || full) {                                                                           \
        const char* _p = (const char*)a.Aop + (int64_t)(t_) * (MD_K * 2);                                 \
        const uint32_t _to = lds0 + (s_) * SLOT + (wave + 8 * _i) * 1024;                                 \
        if (!_past) {                                                                                     \
          dma16(_to, _p, xofs[_i]);                                                                       \
        } else {                                                                                          \
          const int _ln = fresh(lane), _r = (wave + 8 * _i) * (64 / UR) + _ln / UR;                       \
          const bool _in = (int64_t)(t_) * MD_K + 8 * (_ln % UR ^ MD_SWZ(_r)) < a.Kc;                     \
          dma16(_to, _in ? _p + xofs[_i] : (const char*)a.zero_line);                                     \
        }                                                                                                 \
      }                                                                                                   \
  } while (0)
  // The column tiles of an XCD start at different k-tiles: the first to ask for a piece of x waits for the
  // fabric, and started together they all wait for every piece.
#define MD_T(i_) (kt_b + ((i_) + rot < nt ? (i_) + rot : (i_) + rot - nt))
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)smem;
  uint32_t xofs[NI];                                             // (the host keeps them below 4 GB)
  f32x4 y[NR][2];
  Turn turn;
  const int cbo = ks0 & 1;                                       // with several splits this wave's own units are its
  const bool own = !S_::SPLITS || a.ksplit == 1 || ((g * WN * 2 + wn * 2 + cbo) & (a.ksplit - 1)) == ks0;   // column block cbo, if any
  // eight ranks of an octet of row block rb in column lane % 16 of column block cb
  auto factor = [&](int rb, int i, int cb) {
    const int o = oct_s[rb * oct_max + i], row = o >> 8;
    const int64_t n = n0 + cb * 16 + li;
    if (n >= Nout) return make_uint4(0, 0, 0, 0);
    return *(const uint4*)((const bf16_t*)(uintptr_t)rL_s[row] + (o & 255) + n * rank_s[row]);
  };
  // The expand factors' fragments of the first KB steps (of four octets) of this wave's row blocks depend on nothing that
  // has to be waited for.  Four steps where a wave has one row block and the registers for them (200 rows of 64 adapters of
  // rank 64, 2048 x 2048, 24.0 -> 23.2 us; 128 rows of 16 of rank 128 24.9 -> 24.5), as far as the block has octets for them:
  // requested under a lane's condition alone they cost the blocks with few (64 rows of 4 adapters of rank 16, 1024 x
  // 1024, 10.64, one step or as many as there are 10.28).
  constexpr int KB = NR == 1 ? 4 : 1;
  uint4 pre[NR][KB][2];
  auto request_factors = [&]() {
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      const int rb = j * KG + g, cnt = rb < RB ? __builtin_amdgcn_readfirstlane(cnt_s[rb]) : 0;
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        if (k > 0 && 4 * k >= cnt) break;
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
          pre[j][k][cb] = make_uint4(0, 0, 0, 0);
          if (4 * k + lg < cnt) pre[j][k][cb] = factor(rb, 4 * k + lg, cb);
        }
      }
    }
  };
  {
    const int kt_b = ks0 * chunk, kt_e = kt_b + chunk > ktiles ? ktiles : kt_b + chunk, nt = kt_e > kt_b ? kt_e - kt_b : 0;
    int rot = (c >> 3) / a.tiles_m % 8 * a.rot;
    if (rot >= nt) rot = 0;                                      // (the last split can be shorter than the others)
#pragma unroll
    for (int s = 0; s < NS; ++s) if (s < nt) MD_W(MD_T(s), s, "=v");
    {
      if (nt >= NS) wait_vm<NS * 2>(); else wait_vm<0>();   // the indices have arrived
#pragma unroll
      for (int i = 0; i < NI; ++i) {
        asm volatile("" : "+v"(tokr[i]));
        int64_t m = m0 + MD_DROW(i);
        if (m >= a.T) m = a.T - 1;
        xofs[i] = (uint32_t)(((a.perm ? (int64_t)tokr[i] : m) * a.lda + 8 * (dunit ^ MD_SWZ(MD_DROW(i)))) * 2);
      }
      asm volatile("" : "+v"(tok), "+v"(gid), "+v"(gid1));
      tok = !has_row ? -1 : a.perm ? tok : (int32_t)mrow;
      if (!has_row || !lora) gid = -1;
      if (tid == 0 || !lora) gid1 = -1;
    }
    // the rows' adapter entries go before the first x request: they are there when it is
    uint64_t eL, ers;
    {
      const char* en = gid >= 0 ? (const char*)(table + gid) : (const char*)a.zero_line;
      asm volatile("global_load_dwordx2 %0, %1, off" : "=v"(eL) : "v"(en + (a.which ? 8 : 0)) : "memory");
      asm volatile("global_load_dwordx2 %0, %1, off" : "=v"(ers) : "v"(en + 16) : "memory");
    }
#pragma unroll
    for (int s = 0; s < NS; ++s) if (s < nt) MD_X(MD_T(s), s);
    // (every wave waits: a register with a request under way must not look free to the compiler)
    if (nt >= NS) { if (full) wait_vm<NS * NI>(); else wait_vm<NS * (NI - 1)>(); } else wait_vm<0>();
    asm volatile("" : "+v"(eL), "+v"(ers));
    if (wave < (BM + 63) / 64) {
      // the rows' tables, and per 16-row block the octets of its adapters (a lane per row; the first row of
      // an adapter in the block appends the adapter's octets)
      const int rank = gid >= 0 ? (int)(uint32_t)ers : 0;
      const bool first = gid >= 0 && (gid != gid1 || li == 0);
      const int n_oct = first ? rank >> 3 : 0;
      int inc = n_oct, bad = rank & 7 ? 1 : 0;
#pragma unroll
      for (int d = 1; d < 16; d <<= 1) { const int v = __shfl_up(inc, d, 16), w = __shfl_up(bad, d, 16); if (li >= d) { inc += v; bad |= w; } }
      if (tid < BM) {
        tok_s[tid] = tok; t_s[tid] = gid; rank_s[tid] = rank; rL_s[tid] = eL;
        for (int q = 0, o = (tid >> 4) * oct_max + inc - n_oct; q < 8 * n_oct; q += 8, ++o) oct_s[o] = (uint16_t)(tid << 8 | q);
        if (li == 15) cnt_s[tid >> 4] = a.lform == FORM_NT && bad == 0 ? inc : -1;
      }
    }
    f32x4 acc[RB][2];
#pragma unroll
    for (int i = 0; i < RB; ++i) acc[i][0] = acc[i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
    bf16x8 xf[RB];
    // the wave's 32 values of a k-tile: row li of a block, unit 4 g + lg
    const uint32_t xa = lds0 + li * (16 * UR) + (((g * 4 + lg) ^ MD_SWZ(li)) << 4);
#define MD_READ(a_, i_) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(xf[i_]) : "v"(a_), "n"((i_) * 256 * UR))
#define MD_STEP(i_, s_)                                                                                   \
  if ((i_) < RB) {                                                                                        \
    constexpr int _i = (i_) < RB ? (i_) : 0;                                                              \
    asm volatile("" : "+v"(xf[_i]));                                                                      \
    md_product<S_::SPLITS>(acc[_i][0], wreg[s_][0], xf[_i]);                                              \
    md_product<S_::SPLITS>(acc[_i][1], wreg[s_][1], xf[_i]);                                              \
    __builtin_amdgcn_sched_barrier(0);                                                                    \
    MD_READ(_xn, _i);                                                                                     \
  }
    // k-tile i, in slot s_ = i mod NS.  The x fragments rotate: the ones multiplied were read a tile before,
    // each is replaced by its successor right after its products (the last tile's successors come from a
    // stale slot and are not used).  No product waits for reads: MD_SYNC has, in front of every body.
    // Requests complete in order; younger than the x of tile i + 1 are, besides the x of NS - 2 tiles, the
    // weights requested since: min(i, NS - 1) tiles.
#define MD_BODY(s_)                                                                                       \
  do {                                                                                                    \
    constexpr int sn = ((s_) + 1) % NS;                                                                   \
    const uint32_t _xn = xa + sn * SLOT;                                                                  \
    __builtin_amdgcn_sched_barrier(0);                                                                    \
    MD_STEP(0, s_); MD_STEP(1, s_); MD_STEP(2, s_); MD_STEP(3, s_); MD_STEP(4, s_);                             \
    MD_STEP(5, s_); MD_STEP(6, s_); MD_STEP(7, s_); MD_STEP(8, s_); MD_STEP(9, s_);                       \
    MD_STEP(10, s_); MD_STEP(11, s_); MD_STEP(12, s_); MD_STEP(13, s_); MD_STEP(14, s_); MD_STEP(15, s_); \
  } while (0)
  /* after it everyone's part of tile i + 1 is there, and nobody reads the slot of tile i any more */
#define MD_SYNC(s_)                                                                                       \
  do {                                                                                                    \
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");                                       \
    asm volatile("" : "+v"(wreg[s_][0]), "+v"(wreg[s_][1]));                                              \
  } while (0)
    constexpr int XH = (NS - 2) * NI, XL = (NS - 2) * (NI - 1), WA = (NS - 1) * 2;
#define MD_ANY(s_, first_)                                                                                \
  do {                                                                                                    \
    const int i = i0 + (s_);                                                                              \
    if (i < nt) {                                                                                         \
      if (i + NS > nt) wait_vm<0>();                                                                      \
      else if (first_) { if (full) wait_vm<XH + (s_) * 2>(); else wait_vm<XL + (s_) * 2>(); }            \
      else { if (full) wait_vm<XH + WA>(); else wait_vm<XL + WA>(); }                                     \
      MD_SYNC(s_);                                                                                        \
      if (i + NS < nt) MD_X(MD_T(i + NS), s_);                                                            \
      MD_BODY(s_);                                                                                        \
      if (i + NS < nt) MD_W(MD_T(i + NS), s_, "+v");                                                      \
    }                                                                                                     \
  } while (0)
#define MD_FIRST(s_) MD_ANY(s_, true)
#define MD_ITER(s_) MD_ANY(s_, false)
    // the same where neither the start nor the end is near (tile `tile` is requested)
#define MD_STEADY(s_)                                                                                     \
  do {                                                                                                    \
    if (full) wait_vm<XH + WA>(); else wait_vm<XL + WA>();                                                \
    MD_SYNC(s_);                                                                                          \
    MD_X(tile, s_);                                                                                       \
    MD_BODY(s_);                                                                                          \
    MD_W(tile, s_, "+v");                                                                                 \
    tile = tile + 1 < kt_e ? tile + 1 : kt_b;                                                             \
  } while (0)
    if (nt > 0) {
      if (nt < NS) wait_vm<0>(); else if (full) wait_vm<(NS - 1) * NI>(); else wait_vm<(NS - 1) * (NI - 1)>();
      asm volatile("s_barrier" ::: "memory");
#pragma unroll
      for (int i = 0; i < RB; ++i) MD_READ(xa, i);
    }
    int i0 = 0;
#define MD_ROUND(m_)                                                                                      \
  do {                                                                                                    \
    m_(0); m_(1); m_(2);                                                                                  \
    if constexpr (NS > 3) m_(3);                                                                          \
  } while (0)
    if (nt > 0) MD_ROUND(MD_FIRST);
    i0 = NS;
    int tile = MD_T(2 * NS);
#pragma unroll 1
    for (; i0 + 2 * NS <= nt; i0 += NS) MD_ROUND(MD_STEADY);
    // whose turn it is: the answer is there when the last k-tile is
    f32x4 line;
    asm volatile("global_load_dwordx4 %0, %1, off" : "=v"(line) : "v"(joins ? turn_line(a.turns) : none) : "memory");
#pragma unroll 1
    for (; i0 < nt; i0 += NS) MD_ROUND(MD_ITER);
    wait_vm<0>();
    asm volatile("" : "+v"(line));
    turn = turn_of(__float_as_uint(line[0]), __float_as_uint(line[1]), __float_as_uint(line[2]), __float_as_uint(line[3]));
    // (the last reads are not used, but until they are there their registers must not look free)
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
    for (int i = 0; i < RB; ++i) if (nt > 0) asm volatile("" : "+v"(xf[i]));
    if constexpr (!S_::SPLITS) {                                 // (products by inline assembly: nobody counts the wait states of their sums)
      asm volatile("s_nop 15\n\ts_nop 15" ::: "memory");
#pragma unroll
      for (int i = 0; i < RB; ++i) asm volatile("" : "+v"(acc[i][0]), "+v"(acc[i][1]));
    }
    __syncthreads();                                             // the ring is free
    // ---- the contraction groups' sums: row block i is finished by group i mod KG
#pragma unroll
    for (int i = 0; i < RB; ++i)
      if (i % KG != g) {
        const int d = (g - i % KG - 1) & (KG - 1);
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) red[(((i * WN + wn) * 2 + cb) * (KG - 1) + d) * 64 + lane] = acc[i][cb];
      }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RB; ++i)
      if (i % KG == g) {
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
          f32x4 s = acc[i][cb];
#pragma unroll
          for (int d = 0; d < KG - 1; ++d) {
            const f32x4 o = red[(((i * WN + wn) * 2 + cb) * (KG - 1) + d) * 64 + lane];
            s[0] += o[0]; s[1] += o[1]; s[2] += o[2]; s[3] += o[3];
          }
          y[i / KG][cb] = s;
        }
      }
  }
  if (S_::SPLITS && a.ksplit > 1) {
    // row block rb of this wave's own units as split q adds it up: its contraction groups' products, k-tile
    // after k-tile from where the column tile starts, then the groups from the one that finishes the block on
    auto split_sum = [&](int rb, int q) {
      union Frag { uint4 u; bf16x8 v; } wf, xf;
      const int kt_b = q * chunk, kt_e = kt_b + chunk > ktiles ? ktiles : kt_b + chunk, nt = kt_e > kt_b ? kt_e - kt_b : 0;
      int rot = (c >> 3) / a.tiles_m % 8 * a.rot;
      if (rot >= nt) rot = 0;
      const int32_t tk = tok_s[rb * 16 + li];
      const bf16_t* xr = a.Aop + (int64_t)(tk < 0 ? 0 : tk) * a.lda;
      const int64_t last = ((Nout + 15) >> 4) - 1, nb = (n0 >> 4) + cbo;
      const bf16_t* wr = (const bf16_t*)a.proj[p].W + (((nb < last ? nb : last) * ldb) << 9) + lane * 8;
      f32x4 s = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
      for (int d = 0; d < KG; ++d) {
        f32x4 part = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int i = 0; i < nt; ++i) {
          const int st = MD_T(i) * KG + ((rb + d) & (KG - 1));
          const int64_t k = (int64_t)st * 32 + 8 * lg;
          wf.u = xf.u = make_uint4(0, 0, 0, 0);
          if (st < steps) wf.u = *(const uint4*)(wr + ((int64_t)st << 9));
          if (k < a.Kc) xf.u = *(const uint4*)(xr + k);
          part = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf.v, xf.v, part, 0, 0, 0);
        }
#pragma unroll
        for (int v = 0; v < 4; ++v) s[v] = d == 0 ? part[v] : s[v] + part[v];
      }
#pragma unroll
      for (int v = 0; v < 4; ++v) s[v] = __float_as_uint(s[v]) == 0u ? -0.f : s[v];
      return s;
    };
    // ---- hand over the others' units, collect this split's
    float* tile = parts + (int64_t)tn * (UNITS * 256) * a.ksplit + lane * 4;
#pragma unroll
    for (int j = 0; j < NR; ++j)
#pragma unroll
      for (int cb = 0; cb < 2; ++cb)
        if (j * KG + g < RB && !(own && cb == cbo) && turn.sums_ok) {
          f32x4 f;
#pragma unroll
          for (int v = 0; v < 4; ++v) f[v] = __float_as_uint(y[j][cb][v]) == 0u ? -0.f : y[j][cb][v];
          store4_agent(tile + ((((j * KG + g) * WN + wn) * 2 + cb) * a.ksplit + ks0) * 256, f);
        }
    bool ok = true;
    f32x4 w[NR][3];                                              // the other splits' sums, in split order
    if (own) {
      ok = false;
      for (int it = 0; it < a.spin_limit && !ok && turn.sums_ok; ++it) {
#pragma unroll
        for (int j = 0; j < NR; ++j)
#pragma unroll
          for (int o = 0; o < 3; ++o) {
            const int rb = j * KG + g < RB ? j * KG + g : g, q = o + 1 < a.ksplit ? o + (o >= ks0) : ks0 == 0;
            load4_agent(w[j][o], tile + (((rb * WN + wn) * 2 + cbo) * a.ksplit + q) * 256);
          }
        wait_vm<0>();
        bool all = true;
#pragma unroll
        for (int j = 0; j < NR; ++j)
#pragma unroll
          for (int o = 0; o < 3; ++o) {
            asm volatile("" : "+v"(w[j][o]));
#pragma unroll
            for (int v = 0; v < 4; ++v) all &= __float_as_uint(w[j][o][v]) != 0u;
          }
        ok = __ballot(all) == ~0ull;
      }
    }
    if (own && ok) {
#pragma unroll
      for (int j = 0; j < NR; ++j) {
        const f32x4 mine = cbo ? y[j][1] : y[j][0];
        f32x4 sum;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          const f32x4 o = q == ks0 ? mine : q > ks0 ? w[j][q > 0 ? q - 1 : 0] : w[j][q < 3 ? q : 2];
#pragma unroll
          for (int v = 0; v < 4; ++v) sum[v] = q == 0 ? o[v] : q < a.ksplit ? sum[v] + o[v] : sum[v];
        }
        if (cbo) y[j][1] = sum; else y[j][0] = sum;
#pragma unroll
        for (int q = 0; q < 4; ++q)
          if (q < a.ksplit && q != ks0 && j * KG + g < RB)
            store4_agent(tile + ((((j * KG + g) * WN + wn) * 2 + cbo) * a.ksplit + q) * 256, f32x4{0.f, 0.f, 0.f, 0.f});
      }
    } else if (__builtin_expect(own, 0)) {
      // (not reached in practice) the other splits' share of these units again
      if (turn.sums_ok) turn_gave_up(a.turns, turn.number, lane);
#pragma unroll 1
      for (int j = 0; j < NR && j * KG + g < RB; ++j) {
        f32x4 mine = {0.f, 0.f, 0.f, 0.f}, sum = mine;
#pragma unroll
        for (int jj = 0; jj < NR; ++jj)
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const float y0 = y[jj][0][v], y1 = y[jj][1][v];
            if (jj == j) mine[v] = cbo ? y1 : y0;
          }
#pragma unroll 1
        for (int q = 0; q < a.ksplit; ++q) {
          const f32x4 o = split_sum(j * KG + g, q);
#pragma unroll
          for (int v = 0; v < 4; ++v) { const float x = q == ks0 ? mine[v] : o[v]; sum[v] = q == 0 ? x : sum[v] + x; }
        }
#pragma unroll
        for (int jj = 0; jj < NR; ++jj) if (jj == j) { if (cbo) y[jj][1] = sum; else y[jj][0] = sum; }
      }
    }
  }

  if (lora) {
    const float* u_p = u_area(turn.area) + p * S * u_n;
    request_factors();
    // (A reading of u and the factors of eight octets requested before the sums meet, with four requests a reading and the
    // count's answer put off, took 2.8 % longer over 190 sizes in every tiling, all of a thread's readings at once 1.4 %:
    // the code around them costs every wave more than the trips it saves, but for ranks of 128, 1 % shorter with the second.)
    if (!apart) __syncthreads();                                 // (the sums have met: their place is u's)
    const int uq = a.r_stride >> 2;
    for (int i = tid; i < BM * uq; i += MD_THREADS) {            // (whole waves)
      const int row = i / uq, q = (i - row * uq) * 4;
      const int rank = rank_s[row];
      f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
      bool ok = true;
      if (q < rank) ok = read_u(u_p + (m0 + row) * a.r_stride + q, u_n, S, a.spin_limit, v);
      if (__builtin_expect(__ballot(!ok) != 0, 0))               // (not reached in practice)
        u_again(table, a.which, a.Aop, a.lda, a.Kc, S, t_s, tok_s, row, q, !ok, lane, v);
#pragma unroll
      for (int j = 0; j < 4; ++j) if (q + j >= rank) v[j] = 0.f;
      if (cnt_s[row >> 4] >= 0) store_split4((bf16_t*)(u_s + row * us) + q, a.r_stride, v);     // (as the expand wants it)
      else *(f32x4*)(u_s + row * us + q) = v;
      if (a.u_out && lead && m0 + row < a.T && q < ((rank + 15) & ~15))
        *(f32x4*)(a.u_out + (m0 + row) * a.r_stride + q) = v;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < NR; ++j) {
      const int rb = j * KG + g;
      if (rb >= RB || !own) break;
      const int row = rb * 16 + li, cnt = cnt_s[rb];
      if (cnt >= 0) {
        expand_octets(y[j], pre[j], cnt, lg, t_s[row],
                      [&](int q, bool mine, bf16x8& hi, bf16x8& lo) { load_split((const bf16_t*)(u_s + row * us) + q, a.r_stride, mine, hi, lo); },
                      [&](int i) { const int o = oct_s[rb * oct_max + i]; return t_s[o >> 8] << 8 | (o & 255); },
                      [&](int i, int cb) { return factor(rb, i, cb); });
      } else if (t_s[row] >= 0) {
        // ranks that are no multiples of 8, or factors stored rank-major: plain fp32 expand of this lane's row
        const int rank = rank_s[row];
        const bf16_t* L = (const bf16_t*)(uintptr_t)rL_s[row];
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
          const int64_t n = n0 + cb * 16 + 4 * lg;
          if (n < Nout)
            for (int q = 0; q < rank; ++q) {
              const float uq1 = u_s[row * us + q];
#pragma unroll
              for (int v = 0; v < 4; ++v)
                y[j][cb][v] = fmaf(uq1, bf16_bits_to_float(a.lform == FORM_NT ? L[(n + v) * rank + q] : L[(int64_t)q * Nout + n + v]), y[j][cb][v]);
            }
        }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < NR; ++j) {
    if (j * KG + g >= RB || !own) break;
    const int32_t otok = tok_s[(j * KG + g) * 16 + li];
#pragma unroll
    for (int cb = 0; cb < 2; ++cb) {
      const int64_t n = n0 + cb * 16 + 4 * lg;
      if (otok < 0 || n >= Nout || (S_::SPLITS && a.ksplit > 1 && cb != cbo)) continue;   // (Nout is a multiple of 8: four columns are in or out together)
      if (a.out_is_f32) {
        *(f32x4*)((float*)a.proj[p].out + (int64_t)otok * a.proj[p].ldo + n) = y[j][cb];
      } else {
        uint2 o;
        o.x = float_to_bf16_bits(y[j][cb][0]) | ((uint32_t)float_to_bf16_bits(y[j][cb][1]) << 16);
        o.y = float_to_bf16_bits(y[j][cb][2]) | ((uint32_t)float_to_bf16_bits(y[j][cb][3]) << 16);
        *(uint2*)((bf16_t*)a.proj[p].out + (int64_t)otok * a.proj[p].ldo + n) = o;
      }
    }
  }
  if (joins) {                                                   // (nobody waits for these)
    if (tid == MD_THREADS - 1) turn_over(a.turns, turn, u_all);
    clear_share(u_area(1 - turn.area), turn.u_before, c, consumers);
    if (__builtin_expect(!turn.sums_ok, 0)) clear_share(a.partials, MID_PART_FLOATS, c, consumers);
  }
}

template <int RB, int WN>
static hipError_t launch_mid(const GemmArgs& a, int cu_count, hipStream_t stream) {
  constexpr int ring = MidShape<RB, WN>::NS * MidShape<RB, WN>::SLOT;
  const int sums = mid_sums<RB, WN>(a.r_stride);
  const size_t lds = (size_t)(ring > sums ? ring : sums) + mid_tables<RB, WN>(a.r_stride);
  static std::atomic<uint64_t> done_dev{0};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = 1ull << (dev & 63);
  if (!(done_dev.load(std::memory_order_acquire) & bit)) {
    e = hipFuncSetAttribute((const void*)gemm_mid_kernel<RB, WN>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
    done_dev.fetch_or(bit, std::memory_order_release);
  }
  const int ng = 8 / a.ksplit;
  const int consumers = 8 * ((a.tiles_n + ng - 1) / ng) * a.tiles_m;
  // Producers go first where all workgroups are on the chip at once or splits keep the consumers short: their
  // u is then there in time (100 rows, 4096 x 4096 in four splits: 26.4 us, after the consumers 29.3).  Else
  // after one consumer for each compute unit, which they would delay (512 rows, 4096 x 4096, 64 adapters:
  // 50 -> 40 us).  Where those consumers find only half of the chip free (another launch, a stream with fewer
  // compute units) they hold every place, give up waiting and compute their u themselves.
  GemmArgs g = a;
  g.n_jobs = a.n_prod;
  if (mid_alone(RB)) {
    // A workgroup takes a whole unit: producers are first, and no more than the units that the consumers leave, one job after
    // another, where that are 32 and up to five jobs each, which are through before the consumers' sums are (each first on a unit of
    // its own, as many consumers start behind them: 157 rows, 4096 x 28672, 32 adapters in two projections, 66.8 -> 61.7 us; 256 rows,
    // 4096 x 14336, 48.1 -> 42.6; 200 rows, 3000 x 14336, 40 adapters of rank 32, 43.8 -> 39.1).  Behind the consumers they would run on the same
    // units, but a launch beside this one could take those places.
    const int64_t free = mid_free_units(cu_count, consumers);
    g.prod0 = 0;
    if (mid_jobs_in_turn(free, a.n_prod)) g.n_prod = (int)free;
  } else {
    g.prod0 = a.n_prod + consumers <= 2 * cu_count || a.ksplit > 1 || consumers < cu_count ? 0 : cu_count;
  }
  hipLaunchKernelGGL((gemm_mid_kernel<RB, WN>), dim3(g.n_prod + consumers), dim3(MD_THREADS), lds, stream, g);
  return hipGetLastError();
}

}  // namespace marlaas
