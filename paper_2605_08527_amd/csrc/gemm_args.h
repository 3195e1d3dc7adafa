// Kernel arguments and LDS layout helpers shared by the GEMM kernels (large-batch, small-batch and
// decode) and the split-contraction finish kernels.
#pragma once
#include "common.h"

namespace marlaas {

struct GemmArgs {
  const bf16_t* Aop; int64_t lda;
  const bf16_t* Bop; int64_t ldb;
  int64_t T, Kc, Nout;
  const int32_t* perm;
  const int32_t* seg_off;
  int n_adapters;
  const AdapterEntry* table;
  int which;               // 0: L_t = entry.A, 1: L_t = entry.B
  const float* U; int r_stride;
  void* out; int64_t ldo;
  int tiles_m, tiles_n;
  // split-K (few row tiles, e.g. decode): workgroup (tile, ks) handles contraction values
  // [ks * kchunk, (ks + 1) * kchunk) and leaves its fp32 sums in `partials`
  // ([ks][tiles_m * 256][ldp], grouped row order); splitk_finish_kernel adds them up.
  int ksplit; int64_t kchunk; float* partials;
  int64_t ldp;             // row stride of the partial sums (tiles_n * tile width)
  int64_t pm;              // rows of one split's partial sums (tiles_m * tile height)
  const RowChunk* chunks; int n_chunks;   // row chunks of the grouped order (finish kernel)
  // Fused shrink of the small-batch path: every column tile also computes 32 columns of
  // X * [all adapters' shrink factors] (extended column e = rank offset of adapter t + q); the
  // finish kernel picks each row's own adapter, scales and writes u_out.
  const ExtCol* ext_cols; const int32_t* ext_roff; int n_ext;   // n_ext = sum of the ranks; 0: not fused
  // ExtCol::t counts entries of the whole adapter bank, `table` may start inside it: entry index
  // of table[0]; ext_roff[] are offsets in the bank's column space, ext_base the call's first one
  int ext_t0, ext_base;
  float* u_part; int64_t ldu;   // [ks][pm][ldu] fp32 partial sums of the extended columns
  float* u_out;                 // [T][r_stride] (may be null)
  // Several projections in one pass (small-batch kernels only; n_proj <= 1: the fields above
  // describe the only projection).  Column tile tn belongs to the last projection whose tile0 <=
  // tn; `table`, `ext_roff` and ExtCol::t then index [projection][adapter].
  int n_proj;
  int fin_cols;                 // column chunks of the finish kernel's grid, all projections
  // Decode kernel that finishes the call itself (fin_in_kernel = 1: no finish kernel runs; the
  // partial sums are then in accumulator order, [split][tile][unit][column block][lane] x 4).
  //   sync    : device counters, all zero between launches: per tile the splits whose partial
  //             sums are performed, then per tile the splits that are through with it; then per
  //             row tile the workgroups whose partial u is performed and those through with u
  //   grp_ids : adapter of every grouped row (-1: none)
  //   spin_limit: polls of the kernel's one bounded wait
  int fin_in_kernel, out_is_f32, lform, spin_limit;
  int32_t* sync;
  const int32_t* grp_ids;
  ExtRows ext;                  // the row tiles' shares of the extended columns
  int n_prod, n_split;          // few-row kernel: workgroups that compute u (a multiple of n_proj n_split), the splits of their contraction,
  int prod0, n_jobs, proj_jobs, rot;    // (the kernel for more rows: the first of those, their jobs, those of a projection; k-tiles between neighbouring column tiles' starts)
  const bf16_t* zero_line;      // 1024 readable zero bytes
  float* thin_u;                // and where it travels: [MAX_PROJ][THIN_SPLITS][THIN_ROWS][128], zero between launches
  int32_t* turns; float* mid_u; // the kernel for more rows: whose turn it is (agent_memory.h), and the two areas of [projection][split][T][r_stride]
  ProjEntry proj[MAX_PROJ];     // by value: read with wave-uniform loads from the kernel arguments
};

// Large-batch kernel (gemm_wide.hip).  LoraTile: one 64-wide piece of the extra contraction values
// [u_hi | u_lo] x [L_t ; L_t] of the adapter whose rows [lo, hi) lie in a row tile: its factor, first
// value, rank.  A row tile's list is LT_MAX + 1 records, record 0 holding the count in `lo` (-1: more
// than LT_MAX, the kernel then stages the expand through registers).
struct LoraTile { uint64_t L; int32_t lo, hi, kc, rank; int32_t pad[2]; };
static constexpr int LT_MAX = 127;
static_assert(sizeof(LoraTile) == 32, "two 16-byte DMA pieces");
enum { WIDE_LORA_NONE = 0, WIDE_LORA_LISTS = 1, WIDE_LORA_STAGED = 2 };
struct WideArgs {
  const bf16_t* A; int64_t lda;      // rows gathered through perm
  const bf16_t* B; int64_t ldb;
  int64_t T, Kc, Nout;
  const int32_t* perm; const int32_t* seg_off;
  int n_adapters; const AdapterEntry* table; int which;    // which: 0: L_t = entry.A, 1: L_t = entry.B
  int lora;                          // WIDE_LORA_*: none, by DMA from lists and U2, staged through registers from U
  const float* U; int r_stride;
  const bf16_t* U2;                  // [T][2 r_stride]: row m = [u_hi (r_pad) | u_lo (r_pad)] of its adapter
  const LoraTile* lora_tiles;
  const bf16_t* zero_line;           // 16 readable zero bytes that masked DMA lanes fetch
  void* out; int64_t ldo;
  float* partials;
  int tiles_m, tiles_n, rounds, tail_tiles, tail_split; int64_t tail_kchunk;
};
// rounds * 256 whole tiles of 32 mt rows x 256 columns, then tail_tiles tiles in tail_split pieces of
// tail_kchunk contraction values (the last one takes the rest).
struct WidePlan {
  int mt = 8, tiles_m = 0, tiles_n = 0, rounds = 0, tail_tiles = 0, tail_split = 1;
  int64_t tail_kchunk = 0;
  size_t part_bytes = 0;
  double us = 0.0;                   // estimated run time
};
WidePlan wide_plan(int64_t T, int64_t Kc, int64_t Nout, size_t max_bytes);    // (of partial sums; 0: nothing is split)
hipError_t launch_gemm_wide(WideArgs a, const WidePlan& p, int form, int lform, int out_is_f32, hipStream_t stream);
// Tile t in walking order -> its column tile (and row tile *tm): groups of 2048 rows share their column tiles.
__host__ __device__ inline int wide_tile(int t, int mt, int tiles_m, int tiles_n, int* tm) {
  const int GM = 64 / mt;
  const int per_group = GM * tiles_n;
  const int gid = t / per_group, first_m = gid * GM;
  const int gsz = (tiles_m - first_m) < GM ? (tiles_m - first_m) : GM;
  const int in_g = t - gid * per_group;
  *tm = first_m + in_g % gsz;
  return in_g / gsz;
}

typedef const __attribute__((address_space(1))) void* gptr_t;
typedef __attribute__((address_space(3))) void* lptr_t;

// LDS byte offset of 16-byte unit `unit` of row `row` in a [rows][64] bf16 tile.
__device__ __forceinline__ int swz_rowk(int row, int unit) {
  return row * 128 + ((unit ^ ((row >> 1) & 7)) << 4);
}
// 8 consecutive contraction values of one column from a [k][n] tile: two
// transposing 64-bit reads (each returns 4 consecutive k for this lane's column).
__device__ __forceinline__ bf16x8 lds_read_frag_tr(const char* p0, const char* p1) {
  typedef short4v __attribute__((address_space(3))) * lds_s4;
  short4v a = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)p0);
  short4v b = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s4)p1);
  union { short s[8]; bf16x8 v; } r;
  r.s[0] = a[0]; r.s[1] = a[1]; r.s[2] = a[2]; r.s[3] = a[3];
  r.s[4] = b[0]; r.s[5] = b[1]; r.s[6] = b[2]; r.s[7] = b[3];
  return r.v;
}

// s_waitcnt immediate that waits only for the vector-memory counter (6 bits, split 3:0 / 15:14)
#define VMCNT(n) (0x0F70 | ((n) & 15) | ((((n) >> 4) & 3) << 14))

// Extended column e of row tile tm (counted from the tile's first) -> column of the call, e past the
// end repeating the last `unit` columns; columns the tile carries; column (counted from the tile's
// first) of rank 0 of the adapter of projection p whose rank offset is roff.
__device__ __forceinline__ int ext_carried(const GemmArgs& a, int tm) { return a.ext.on ? a.ext.count[tm] : a.n_ext; }
__device__ __forceinline__ int ext_column(const GemmArgs& a, int tm, int e, int unit) {
  const int n = ext_carried(a, tm);
  if (e >= n) e = n - unit;
  if (e < 0) e = 0;
  if (!a.ext.on) return e;
  int p = 0;
  for (int q = 1; q < a.n_proj; ++q) if (e >= a.ext.start[tm][q]) p = q;
  return n > 0 ? a.ext.base[tm][p] + e - a.ext.start[tm][p] : 0;
}
__device__ __forceinline__ int ext_local(const GemmArgs& a, int tm, int p, int roff) {
  return roff - a.ext_base + (a.ext.on ? a.ext.start[tm][p] - a.ext.base[tm][p] : 0);
}

// Small-batch kernels: tile of the partial sums and of the finish kernel's grid.
static constexpr int SK_BM = 128, SK_BN = 128, SK_BX = 32;

// Decode kernel on a packed copy of the weight (gemm_decode.hip): same tiles, same partial-sum
// layout and same finish kernel as gemm_skinny_kernel.  Bop (and every ProjEntry::W) is the packed
// copy, ldb (ProjEntry::ldw) its k-steps per column block; the adapters' factors must be stored
// contraction-contiguous when the shrink is fused (n_ext > 0).
hipError_t launch_gemm_decode(const GemmArgs& a, hipStream_t stream);
// Its tile (row tile, column tile) and split of workgroup b.  Workgroup b runs on XCD b mod 8, and every XCD has its own L2.  Where the sizes allow it, an
// XCD works on ONE contraction split (and on every 8 / ksplit-th column tile): it then pulls only its own K-range of x (and of the shrink factors)
// through the fabric, instead of all of x once per XCD.  The row tiles of a column tile stay neighbours on one XCD and share the
// weight tile through its L2.  Otherwise: a compact run of (column tile, split, row tile).
__host__ __device__ inline void decode_tile(int b, int tiles_m, int tiles_n, int ksplit, int* tm, int* tn, int* ks) {
  const int G = tiles_m * tiles_n * ksplit, xcd = b & 7, idx = b >> 3;
  const int ng = 8 / ksplit;                     // XCDs that share a split
  if (ksplit <= 8 && ng * ksplit == 8 && tiles_n % ng == 0) {
    *ks = xcd % ksplit;
    *tm = idx % tiles_m;
    *tn = (idx / tiles_m) * ng + xcd / ksplit;
  } else {
    const int q = G >> 3, rem = G & 7;
    const int bbs = xcd * q + (xcd < rem ? xcd : rem) + idx;
    *tm = bbs % tiles_m;
    const int rest = bbs / tiles_m;
    *ks = rest % ksplit;
    *tn = rest / ksplit;
  }
}
// Whether u of an unsplit call is there without waiting for a workgroup that has no unit yet: a workgroup has a unit to itself until it
// is through, so the column tiles that carry the `ext` extended columns have to be among the first on their XCDs.
inline bool decode_u_comes_first(int tiles_m, int tiles_n, int ext, int cu_count) {
  const int carry = (ext + 31) / 32 < tiles_n ? (ext + 31) / 32 : tiles_n;
  if (tiles_m * tiles_n <= cu_count) return true;
  return (tiles_n % 8 == 0 ? (carry + 7) / 8 * tiles_m : carry * tiles_m) <= cu_count / 8;
}

// Few rows (T <= THIN_ROWS) on packed weights, one launch (gemm_thin.hip): every ProjEntry filled in
// (also for one projection; W packed, ldw its k-steps, tile0 set here), u_out = [T][r_stride] fp32 that
// receives the scaled u (one projection; may be null), sync = counters, n_prod = n_proj times the most 16-rank tiles that
// any grouping of T rows can use.  Factors of the shrink stored contraction-contiguous.
hipError_t launch_gemm_thin(GemmArgs a, hipStream_t stream);
// Up to MID_ROWS rows likewise (gemm_mid.hip); turns, mid_u, partials: the context's areas.
hipError_t launch_gemm_mid(GemmArgs a, const MidPlan& p, int cu_count, hipStream_t stream);
hipError_t launch_gemm_tall(const GemmArgs& a, const MidPlan& p, int cu_count, hipStream_t stream);    // (its taller tiles: gemm_tall.hip)

}  // namespace marlaas
