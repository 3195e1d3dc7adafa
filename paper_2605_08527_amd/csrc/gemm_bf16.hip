// Small batches without a packed weight: gemm_skinny_kernel + splitk_finish_kernel, and the choice
// between the GEMM kernels (this one, gemm_decode.hip, gemm_wide.hip).
//
//   out[tok(m), :] = Aop[tok(m), :] * Bop  +  u(m) * L_t          (m in the segment of adapter t)
//
// 128 x 128 tiles with the contraction split over workgroups, fp32 partial sums, and the shrink
// computed by the same kernel as 32 extended columns per column tile; the finish kernel adds the
// splits, applies the expand in fp32 and scatters the rows.  transpose_bf16_kernel: per-call
// transposed copy of a weight that is stored output-contiguous, for large batches.
#include "mid_plan.h"

#include <atomic>
#include <cstring>

namespace marlaas {

static constexpr int BK = 64;          // k-tile

// ---------------------------------------------------------------------------------------------
// Small batches (decode): the weight is streamed once from HBM and is the dominant traffic.  With
// few rows the 256 x 256 tile needs many contraction splits to fill the chip, and the fp32
// partial sums then cost more traffic than the weight.  Here the tile is 128 x 128 (a quarter of
// the splits for the same number of workgroups) and the DMA ring is four k-tiles deep, three of
// them in flight (48 KB of weight per compute unit), which is what covers the HBM latency.  Each
// wave owns 64 x 64.  The result always goes to fp32 partial rows; splitk_finish_kernel adds the
// splits, the LoRA expand and the rounding.
static constexpr int SK_A_BYTES = SK_BM * BK * 2;         // 16 KB
static constexpr int SK_B_BYTES = SK_BN * BK * 2;         // 16 KB
static constexpr int SK_X_BYTES = SK_BX * BK * 2;         // 4 KB: extended (shrink) columns
static constexpr int SK_SLOT = SK_A_BYTES + SK_B_BYTES + SK_X_BYTES;   // 36 KB
static constexpr int SK_SLOTS = 4;
static constexpr int SK_LDS = SK_SLOTS * SK_SLOT + SK_BM * 4;
#define SK_NI (8 + (EXT ? 1 : 0))   // DMA instructions per wave per k-tile

template <int FORM, bool EXT>
__global__ __launch_bounds__(256) void gemm_skinny_kernel(GemmArgs a) {
  extern __shared__ __attribute__((aligned(16))) char smem[];
  int32_t* tok_s = (int32_t*)(smem + SK_SLOTS * SK_SLOT);
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  int tm, tn, ks_idx;
  {
    // consecutive workgroups of one XCD: the row tiles of one column tile (they share the weight
    // tile through that XCD's L2), then its contraction splits, then the next column tile
    const int G = a.tiles_m * a.tiles_n * a.ksplit;
    const int b = blockIdx.x;
    const int xcd = b & 7, idx = b >> 3;
    const int q = G >> 3, rem = G & 7;
    const int bbs = xcd * q + (xcd < rem ? xcd : rem) + idx;
    tm = bbs % a.tiles_m;
    const int rest = bbs / a.tiles_m;
    ks_idx = rest % a.ksplit;
    tn = rest / a.ksplit;
  }
  const int64_t m0 = (int64_t)tm * SK_BM;
  const int64_t pn0 = (int64_t)tn * SK_BN;       // column of this tile in the partial sums
  // the projection this column tile belongs to (wave-uniform)
  const bf16_t* Bop = a.Bop;
  int64_t ldb = a.ldb, Nout = a.Nout, n0 = pn0;
  if (a.n_proj > 1) {
    int p = 0;
    for (int q = 1; q < a.n_proj; ++q) if (tn >= a.proj[q].tile0) p = q;
    const ProjEntry pe = a.proj[p];
    Bop = (const bf16_t*)pe.W; ldb = pe.ldw; Nout = pe.Nout;
    n0 = (int64_t)(tn - pe.tile0) * SK_BN;
  }
  const int64_t kbeg = (int64_t)ks_idx * a.kchunk;
  const int64_t kend = (kbeg + a.kchunk) < a.Kc ? (kbeg + a.kchunk) : a.Kc;
  const int64_t ntile = (kend - kbeg) / BK;
  // (two dependent table loads: requested first, needed last)
  // extended columns: one DMA instruction per wave per k-tile
  const bf16_t* x_src = nullptr;
  int64_t x_step = 0;
  if (EXT) {
    if (FORM == FORM_NT) {           // tile [32 e][64 k]: row = extended column, factor stored [r][Kc]
      const int row = wave * 8 + (lane >> 3);
      const int unit = (lane & 7) ^ ((row >> 1) & 7);
      const ExtCol c = a.ext_cols[ext_column(a, tm, tn * SK_BX + row, 1)];
      x_src = (const bf16_t*)(a.which ? c.A : c.B) + (int64_t)c.q * a.Kc + kbeg + unit * 8;
      x_step = BK;
    } else {                         // tile [64 k][32 e], 64-byte rows: factor stored [Kc][r], r % 8 == 0
      const int k = wave * 16 + (lane >> 2);
      const ExtCol c = a.ext_cols[ext_column(a, tm, tn * SK_BX + (lane & 3) * 8, 8)];
      const AdapterEntry en = a.table[c.t - a.ext_t0];     // (this storage form needs the rank)
      x_src = (const bf16_t*)(a.which ? en.A : en.B) + (kbeg + k) * en.rank + c.q;
      x_step = (int64_t)BK * en.rank;
    }
  }

  // DMA sources: 4 instructions (1 KB each) per wave per operand per k-tile.  The weight requests
  // do not depend on the token indices, so the first three k-tiles of the weight go out before
  // the indices are even loaded (three k-tiles stay in flight throughout).
  const bf16_t* a_src[4];
  const bf16_t* b_src[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (FORM == FORM_NT) {           // B tile [128 n][64 k], 128-byte rows
      const int row = (wave * 4 + j) * 8 + (lane >> 3);
      const int unit = (lane & 7) ^ ((row >> 1) & 7);
      int64_t n = n0 + row;
      if (n >= Nout) n = Nout - 1;
      b_src[j] = Bop + n * ldb + kbeg + unit * 8;
    } else {                         // B tile [64 k][128 n], 256-byte rows
      const int k = (wave * 4 + j) * 4 + (lane >> 4);
      int64_t n = n0 + (((lane & 15) ^ ((k & 3) << 2)) << 3);
      if (n >= Nout) n = Nout - 8;
      b_src[j] = Bop + (kbeg + k) * ldb + n;
    }
  }
  const int64_t b_step = FORM == FORM_NT ? (int64_t)BK : (int64_t)BK * ldb;
#pragma unroll
  for (int s3 = 0; s3 < 3; ++s3)
    if (s3 < ntile) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        __builtin_amdgcn_global_load_lds((gptr_t)b_src[j], (lptr_t)(smem + s3 * SK_SLOT + SK_A_BYTES + wave * 4096 + j * 1024), 16, 0, 0);
        b_src[j] += b_step;
      }
    }

  if (tid < SK_BM) {
    const int64_t m = m0 + tid;
    tok_s[tid] = m < a.T ? (a.perm ? a.perm[m] : (int32_t)m) : -1;
  }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int row = (wave * 4 + j) * 8 + (lane >> 3);
    const int unit = (lane & 7) ^ ((row >> 1) & 7);
    const int32_t tok = tok_s[row];
    a_src[j] = a.Aop + (int64_t)(tok < 0 ? tok_s[0] : tok) * a.lda + kbeg + unit * 8;
  }
#pragma unroll
  for (int s3 = 0; s3 < 3; ++s3)
    if (s3 < ntile) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        __builtin_amdgcn_global_load_lds((gptr_t)a_src[j], (lptr_t)(smem + s3 * SK_SLOT + wave * 4096 + j * 1024), 16, 0, 0);
        a_src[j] += BK;
      }
    }
  const int frow = lane & 31, fk = lane >> 5;
  const int a_row = wm * 64 + frow, b_row = wn * 64 + frow;
  const int a_off = a_row * 128, a_swz = (a_row >> 1) & 7;
  const int b_off = b_row * 128, b_swz = (b_row >> 1) & 7;
  int btr[2];
  {
    const int g16 = lane >> 4, i16 = lane & 15;
    const int kb = (g16 >> 1) * 8 + (i16 >> 2);
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
      const int ncol = wn * 64 + nt * 32 + (g16 & 1) * 16 + 4 * (i16 & 3);
      btr[nt] = kb * 256 + (((ncol >> 3) ^ ((kb & 3) << 2)) << 4) + (ncol & 7) * 2;
    }
  }

  const int x_off = frow * 128, x_swz = (frow >> 1) & 7;        // NT fragment of the extended tile
  int xtr = 0;                                                   // NN: transposing read offset
  {
    const int g16 = lane >> 4, i16 = lane & 15;
    const int kb = (g16 >> 1) * 8 + (i16 >> 2);
    xtr = kb * 64 + ((g16 & 1) * 16 + 4 * (i16 & 3)) * 2;
  }
  f32x16 acc_x;
#pragma unroll
  for (int v = 0; v < 16; ++v) acc_x[v] = 0.f;
  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

#define SK_DMA_X(slot_)                                                                                   \
  do {                                                                                                    \
    if (EXT) {                                                                                            \
      __builtin_amdgcn_global_load_lds((gptr_t)x_src,                                                     \
          (lptr_t)(smem + (slot_) * SK_SLOT + SK_A_BYTES + SK_B_BYTES + wave * 1024), 16, 0, 0);           \
      x_src += x_step;                                                                                    \
    }                                                                                                     \
  } while (0)

  auto kstep = [&](const char* as, const char* bs, int ks) {
    bf16x8 af[2], bfr[2];
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
      af[mt] = *(const bf16x8*)(as + a_off + mt * (32 * 128) + (((ks * 2 + fk) ^ a_swz) << 4));
#pragma unroll
    for (int nt = 0; nt < 2; ++nt) {
      if (FORM == FORM_NT) {
        bfr[nt] = *(const bf16x8*)(bs + b_off + nt * (32 * 128) + (((ks * 2 + fk) ^ b_swz) << 4));
      } else {
        const char* p = bs + btr[nt] + ks * (16 * 256);   // k & 3 is unchanged by steps of 4
        bfr[nt] = lds_read_frag_tr(p, p + 4 * 256);
      }
    }
#pragma unroll
    for (int mt = 0; mt < 2; ++mt)
#pragma unroll
      for (int nt = 0; nt < 2; ++nt)
        acc[mt][nt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[mt], bfr[nt], acc[mt][nt], 0, 0, 0);
    if (EXT) {
      const char* xs = bs + SK_B_BYTES;
      bf16x8 xf;
      if (FORM == FORM_NT) {
        xf = *(const bf16x8*)(xs + x_off + (((ks * 2 + fk) ^ x_swz) << 4));
      } else {
        const char* px = xs + xtr + ks * (16 * 64);
        xf = lds_read_frag_tr(px, px + 4 * 64);
      }
      acc_x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wn ? af[1] : af[0], xf, acc_x, 0, 0, 0);
    }
  };

  // One wave per SIMD: nothing but the instruction order hides LDS and DMA latency, so the loop
  // is software-pipelined by hand (sched_barrier pins the order).  Fragments of k-step s + 1 are
  // read while the MFMAs of k-step s run; the wait + barrier for the next k-tile sits before the
  // last k-step, whose MFMAs cover the first fragment reads of the next tile and the DMA issue.
#define SK_READ(base_, ks_, af_, bf_)                                                                     \
  do {                                                                                                    \
    const char* _as = (base_);                                                                            \
    const char* _bs = _as + SK_A_BYTES;                                                                   \
    af_[0] = *(const bf16x8*)(_as + a_off + ((((ks_) * 2 + fk) ^ a_swz) << 4));                           \
    af_[1] = *(const bf16x8*)(_as + a_off + 32 * 128 + ((((ks_) * 2 + fk) ^ a_swz) << 4));                \
    if (FORM == FORM_NT) {                                                                                \
      bf_[0] = *(const bf16x8*)(_bs + b_off + ((((ks_) * 2 + fk) ^ b_swz) << 4));                         \
      bf_[1] = *(const bf16x8*)(_bs + b_off + 32 * 128 + ((((ks_) * 2 + fk) ^ b_swz) << 4));              \
    } else {                                                                                              \
      const char* _p0 = _bs + btr[0] + (ks_) * (16 * 256);                                                \
      const char* _p1 = _bs + btr[1] + (ks_) * (16 * 256);                                                \
      bf_[0] = lds_read_frag_tr(_p0, _p0 + 4 * 256);                                                      \
      bf_[1] = lds_read_frag_tr(_p1, _p1 + 4 * 256);                                                      \
    }                                                                                                     \
    if (EXT) {                                                                                            \
      const char* _xs = _bs + SK_B_BYTES;                                                                 \
      if (FORM == FORM_NT) {                                                                              \
        bf_[2] = *(const bf16x8*)(_xs + x_off + ((((ks_) * 2 + fk) ^ x_swz) << 4));                       \
      } else {                                                                                            \
        const char* _px = _xs + xtr + (ks_) * (16 * 64);                                                  \
        bf_[2] = lds_read_frag_tr(_px, _px + 4 * 64);                                                     \
      }                                                                                                   \
    }                                                                                                     \
    __builtin_amdgcn_sched_barrier(0);                                                                    \
  } while (0)
#define SK_MMAX(af_, bf_)                                                                                 \
  do {                                                                                                    \
    if (EXT) {                                                                                            \
      acc_x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wn ? af_[1] : af_[0], bf_[2], acc_x, 0, 0, 0);                   \
      __builtin_amdgcn_sched_barrier(0);                                                                  \
    }                                                                                                     \
  } while (0)
#define SK_MMA1(af_, bf_, mt_, nt_)                                                                       \
  do {                                                                                                    \
    acc[mt_][nt_] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af_[mt_], bf_[nt_], acc[mt_][nt_], 0, 0, 0);  \
    __builtin_amdgcn_sched_barrier(0);                                                                    \
  } while (0)
#define SK_DMA_B(sb_, j_)                                                                                 \
  do {                                                                                                    \
    __builtin_amdgcn_global_load_lds((gptr_t)b_src[j_], (lptr_t)((sb_) + SK_A_BYTES + (j_) * 1024), 16, 0, 0); \
    b_src[j_] += b_step;                                                                                \
  } while (0)
#define SK_DMA_A(sb_, j_)                                                                                 \
  do {                                                                                                    \
    __builtin_amdgcn_global_load_lds((gptr_t)a_src[j_], (lptr_t)((sb_) + (j_) * 1024), 16, 0, 0);         \
    a_src[j_] += BK;                                                                                      \
  } while (0)

  // (three k-tiles of A and B are in flight already;) the extended columns' source addresses
  // arrive last (two dependent table loads), so their requests go last
  if (ntile > 0) SK_DMA_X(0);
  if (ntile > 1) SK_DMA_X(1);
  if (ntile > 2) SK_DMA_X(2);
  if constexpr (FORM == FORM_NT) {
    // The compiler drains the whole LDS queue before the first use of any LDS result, which with
    // one wave per SIMD exposes the LDS latency at every k-step.  Here the fragment reads are
    // inline assembly (the compiler does not see them as pending), issued two k-steps ahead into
    // four fragment sets, and the waits are written by hand: LDS results return in order, so
    // "at most 2 x NR reads outstanding" means the set issued two steps ago is complete.
    constexpr int NR = EXT ? 5 : 4;                 // reads per k-step
    const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)smem;
    uint32_t ra[4], rb[4], rx[4];                   // this lane's fragment addresses in slot 0, per k-step
#pragma unroll
    for (int ks = 0; ks < 4; ++ks) {
      ra[ks] = lds0 + a_off + (((ks * 2 + fk) ^ a_swz) << 4);
      rb[ks] = lds0 + SK_A_BYTES + b_off + (((ks * 2 + fk) ^ b_swz) << 4);
      rx[ks] = lds0 + SK_A_BYTES + SK_B_BYTES + x_off + (((ks * 2 + fk) ^ x_swz) << 4);
    }
    bf16x8 f0[5], f1[5], f2[5], f3[5];              // a0 a1 b0 b1 x
#define SKP_READ(so_, ks_, f_)                                                                            \
  do {                                                                                                    \
    const uint32_t _a = ra[ks_] + (so_), _b = rb[ks_] + (so_);                                            \
    asm volatile("ds_read_b128 %0, %1" : "=v"(f_[0]) : "v"(_a));                                          \
    asm volatile("ds_read_b128 %0, %1 offset:4096" : "=v"(f_[1]) : "v"(_a));                              \
    asm volatile("ds_read_b128 %0, %1" : "=v"(f_[2]) : "v"(_b));                                          \
    asm volatile("ds_read_b128 %0, %1 offset:4096" : "=v"(f_[3]) : "v"(_b));                              \
    if (EXT) { const uint32_t _x = rx[ks_] + (so_); asm volatile("ds_read_b128 %0, %1" : "=v"(f_[4]) : "v"(_x)); } \
    __builtin_amdgcn_sched_barrier(0);                                                                    \
  } while (0)
#define SKP_WAIT(n_) do { asm volatile("s_waitcnt lgkmcnt(%0)" :: "n"(n_) : "memory"); __builtin_amdgcn_sched_barrier(0); } while (0)
#define SKP_MMA1(f_, mt_, nt_)                                                                            \
  do {                                                                                                    \
    acc[mt_][nt_] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(f_[mt_], f_[2 + nt_], acc[mt_][nt_], 0, 0, 0); \
    __builtin_amdgcn_sched_barrier(0);                                                                    \
  } while (0)
#define SKP_MMAX(f_)                                                                                      \
  do {                                                                                                    \
    if (EXT) {                                                                                            \
      acc_x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wn ? f_[1] : f_[0], f_[4], acc_x, 0, 0, 0);          \
      __builtin_amdgcn_sched_barrier(0);                                                                  \
    }                                                                                                     \
  } while (0)
#define SKP_MMA(f_) do { SKP_MMA1(f_, 0, 0); SKP_MMA1(f_, 0, 1); SKP_MMA1(f_, 1, 1); SKP_MMA1(f_, 1, 0); SKP_MMAX(f_); } while (0)
    if (ntile > 0) {
      // (all three tiles: the per-tile counting of the loop needs each tile's requests adjacent)
      __builtin_amdgcn_s_waitcnt(VMCNT(0));
      asm volatile("s_barrier" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      SKP_READ(0u, 0, f0);
      SKP_READ(0u, 1, f1);
    }
    int64_t kt = 0;
    // steady state: tile kt + 3 is requested during tile kt
    for (; kt + 3 < ntile; ++kt) {
      const uint32_t so = (uint32_t)(kt & (SK_SLOTS - 1)) * SK_SLOT;
      const uint32_t sn = (uint32_t)((kt + 1) & (SK_SLOTS - 1)) * SK_SLOT;
      SKP_READ(so, 2, f2); SKP_WAIT(2 * NR); SKP_MMA(f0);
      SKP_READ(so, 3, f3); SKP_WAIT(2 * NR); SKP_MMA(f1);
      // this wave's part of tile kt + 1 has landed (tile kt + 2 may still be in flight); after the
      // barrier everyone's has, and nobody still reads tile kt - 1, whose slot is filled next
      // (every read of it was waited for before its MFMAs, a tile ago)
      __builtin_amdgcn_s_waitcnt(VMCNT(SK_NI));
      asm volatile("s_barrier" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      SKP_READ(sn, 0, f0); SKP_WAIT(2 * NR);
      char* sb = smem + (int)((kt + 3) & (SK_SLOTS - 1)) * SK_SLOT + wave * 4096;
      SKP_MMA1(f2, 0, 0);
      SK_DMA_B(sb, 0); SK_DMA_B(sb, 1); SK_DMA_B(sb, 2);
      SKP_MMA1(f2, 0, 1);
      SK_DMA_B(sb, 3); SK_DMA_A(sb, 0); SK_DMA_A(sb, 1);
      SKP_MMA1(f2, 1, 1);
      SK_DMA_A(sb, 2); SK_DMA_A(sb, 3);
      SK_DMA_X((int)((kt + 3) & (SK_SLOTS - 1)));
      SKP_MMA1(f2, 1, 0);
      SKP_MMAX(f2);
      SKP_READ(sn, 1, f1); SKP_WAIT(2 * NR); SKP_MMA(f3);
    }
    // the last three tiles are already requested
    for (; kt + 1 < ntile; ++kt) {
      const uint32_t so = (uint32_t)(kt & (SK_SLOTS - 1)) * SK_SLOT;
      const uint32_t sn = (uint32_t)((kt + 1) & (SK_SLOTS - 1)) * SK_SLOT;
      SKP_READ(so, 2, f2); SKP_WAIT(2 * NR); SKP_MMA(f0);
      SKP_READ(so, 3, f3); SKP_WAIT(2 * NR); SKP_MMA(f1);
      __builtin_amdgcn_s_waitcnt(VMCNT(0));
      asm volatile("s_barrier" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      SKP_READ(sn, 0, f0); SKP_WAIT(2 * NR); SKP_MMA(f2);
      SKP_READ(sn, 1, f1); SKP_WAIT(2 * NR); SKP_MMA(f3);
    }
    // last tile: nothing follows
    if (kt < ntile) {
      const uint32_t so = (uint32_t)(kt & (SK_SLOTS - 1)) * SK_SLOT;
      SKP_READ(so, 2, f2); SKP_WAIT(2 * NR); SKP_MMA(f0);
      SKP_READ(so, 3, f3); SKP_WAIT(2 * NR); SKP_MMA(f1);
      SKP_WAIT(0);
      SKP_MMA(f2);
      SKP_MMA(f3);
    }
  } else {
    bf16x8 fa0[2], fb0[3], fa1[2], fb1[3];
    if (ntile > 0) {
      // (all three: the per-tile counting of the loop needs each tile's requests to be adjacent)
      __builtin_amdgcn_s_waitcnt(VMCNT(0));
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      SK_READ(smem, 0, fa0, fb0);
    }
    // One k-step: the first MFMA (the compiler's wait for this step's fragments sits before it and
    // drains the LDS queue, so no younger read may be outstanding here), then the reads of the next
    // step into the other fragment set, then the remaining three MFMAs.
#define SK_STEP(ua_, ub_, base_, ks_, la_, lb_)                                                           \
    do {                                                                                                    \
      SK_MMA1(ua_, ub_, 0, 0);                                                                              \
      SK_READ(base_, ks_, la_, lb_);                                                                        \
      SK_MMA1(ua_, ub_, 0, 1); SK_MMA1(ua_, ub_, 1, 1); SK_MMA1(ua_, ub_, 1, 0); SK_MMAX(ua_, ub_);         \
    } while (0)
    // steady state: tile kt + 3 is requested during tile kt
    int64_t kt = 0;
    for (; kt + 3 < ntile; ++kt) {
      const char* cur = smem + (int)(kt & (SK_SLOTS - 1)) * SK_SLOT;
      SK_STEP(fa0, fb0, cur, 1, fa1, fb1);
      SK_STEP(fa1, fb1, cur, 2, fa0, fb0);
      SK_STEP(fa0, fb0, cur, 3, fa1, fb1);
      // this wave's part of tile kt + 1 has landed (tile kt + 2 may still be in flight) ...
      __builtin_amdgcn_s_waitcnt(VMCNT(SK_NI));
      // ... everyone's has, and nobody still reads tile kt - 1, whose slot is filled next
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      char* sb = smem + (int)((kt + 3) & (SK_SLOTS - 1)) * SK_SLOT + wave * 4096;
      SK_MMA1(fa1, fb1, 0, 0);
      SK_READ(smem + (int)((kt + 1) & (SK_SLOTS - 1)) * SK_SLOT, 0, fa0, fb0);
      SK_DMA_B(sb, 0); SK_DMA_B(sb, 1); SK_DMA_B(sb, 2);
      SK_MMA1(fa1, fb1, 0, 1);
      SK_DMA_B(sb, 3);
      SK_DMA_A(sb, 0); SK_DMA_A(sb, 1);
      SK_MMA1(fa1, fb1, 1, 1);
      SK_DMA_A(sb, 2); SK_DMA_A(sb, 3);
      SK_MMA1(fa1, fb1, 1, 0);
      SK_DMA_X((int)((kt + 3) & (SK_SLOTS - 1)));
      SK_MMAX(fa1, fb1);
    }
    // drain: the last three tiles are already requested
    for (; kt < ntile; ++kt) {
      const char* cur = smem + (int)(kt & (SK_SLOTS - 1)) * SK_SLOT;
      SK_STEP(fa0, fb0, cur, 1, fa1, fb1);
      SK_STEP(fa1, fb1, cur, 2, fa0, fb0);
      SK_STEP(fa0, fb0, cur, 3, fa1, fb1);
      __builtin_amdgcn_s_waitcnt(VMCNT(0));
      asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
      // (after the last tile this reads a stale slot; those fragments are not used)
      SK_STEP(fa1, fb1, smem + (int)((kt + 1) & (SK_SLOTS - 1)) * SK_SLOT, 0, fa0, fb0);
    }
  }
  __syncthreads();
  // k tail of the last split: one masked tile through registers into slot 0
  if (kbeg + ntile * BK < kend) {
    const int64_t k0 = kbeg + ntile * BK;
    const uint4 zero4 = make_uint4(0, 0, 0, 0);
    char* as = smem;
    char* bs = smem + SK_A_BYTES;
    {
      const int lc = tid & 7, lr = tid >> 3;
      const bool ka = (k0 + lc * 8) < kend;
      for (int i = 0; i < 4; ++i) {
        const int row = lr + 32 * i;
        const int32_t tok = tok_s[row];
        uint4 v = zero4;
        if (ka && tok >= 0) v = *(const uint4*)(a.Aop + (int64_t)tok * a.lda + k0 + lc * 8);
        *(uint4*)(as + swz_rowk(row, lc)) = v;
        if (FORM == FORM_NT) {
          uint4 w = zero4;
          if (ka && (n0 + row) < Nout) w = *(const uint4*)(Bop + (n0 + row) * ldb + k0 + lc * 8);
          *(uint4*)(bs + swz_rowk(row, lc)) = w;
        }
      }
    }
    if (FORM == FORM_NN) {
      const int lc = tid & 15, lr = tid >> 4;
      for (int i = 0; i < 4; ++i) {
        const int k = lr + 16 * i;
        uint4 w = zero4;
        if ((k0 + k) < kend && (n0 + lc * 8) < Nout) w = *(const uint4*)(Bop + (k0 + k) * ldb + n0 + lc * 8);
        *(uint4*)(bs + k * 256 + ((lc ^ ((k & 3) << 2)) << 4)) = w;
      }
    }
    if (EXT) {
      char* xs = bs + SK_B_BYTES;
      if (FORM == FORM_NT) {
        const int lc = tid & 7, row = tid >> 3;             // 32 rows x 8 units
        const ExtCol c = a.ext_cols[ext_column(a, tm, tn * SK_BX + row, 1)];
        uint4 w = zero4;
        if ((k0 + lc * 8) < kend) w = *(const uint4*)((const bf16_t*)(a.which ? c.A : c.B) + (int64_t)c.q * a.Kc + k0 + lc * 8);
        *(uint4*)(xs + swz_rowk(row, lc)) = w;
      } else {
        const int lc = tid & 3, k = tid >> 2;               // 64 k-rows x 4 units
        const ExtCol c = a.ext_cols[ext_column(a, tm, tn * SK_BX + lc * 8, 8)];
        uint4 w = zero4;
        const AdapterEntry en = a.table[c.t - a.ext_t0];
        if ((k0 + k) < kend) w = *(const uint4*)((const bf16_t*)(a.which ? en.A : en.B) + (k0 + k) * en.rank + c.q);
        *(uint4*)(xs + k * 64 + lc * 16) = w;
      }
    }
    __syncthreads();
    const int ksteps = (int)((kend - k0 + 15) / 16);
    for (int ks = 0; ks < ksteps; ++ks) kstep(as, bs, ks);
  }
  float* part = a.partials + ((int64_t)ks_idx * a.pm + m0 + wm * 64) * a.ldp + pn0 + wn * 64 + (lane & 31);
#pragma unroll
  for (int mt = 0; mt < 2; ++mt)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int row = mt * 32 + 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
#pragma unroll
      for (int nt = 0; nt < 2; ++nt) part[(int64_t)row * a.ldp + nt * 32] = acc[mt][nt][v];
    }
  if (EXT) {
    // this wave's 32 rows (row block 2 wm + wn of the tile) x the tile's 32 extended columns
    float* up = a.u_part + ((int64_t)ks_idx * a.pm + m0 + wm * 64 + wn * 32) * a.ldu + tn * SK_BX + (lane & 31);
#pragma unroll
    for (int v = 0; v < 16; ++v) up[(int64_t)(8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * a.ldu] = acc_x[v];
  }
}

// Second step of the split-K path: add the partial sums in split order, add the LoRA expand in
// fp32 (u is fp32, so no two-term split is needed here) and scatter the rows.  A block owns one
// row chunk (up to 8 consecutive grouped rows of one adapter) x 512 columns, 2 per thread, so the
// adapter's factor is read once per chunk and every load of a block is issued up front.  With a
// column-chunk count that is a multiple of 8, column chunk c of every row chunk runs on XCD
// c mod 8, whose L2 then holds that slice of each factor.
static constexpr int FIN_THREADS = 256;
static constexpr int FIN_COLS = 2 * FIN_THREADS;

template <int FORM, bool OUT_F32>
__global__ __launch_bounds__(FIN_THREADS) void splitk_finish_kernel(GemmArgs a) {
  constexpr int R = ROW_CHUNK;
  constexpr int UPT = R * 128 / FIN_THREADS;        // u values staged per thread
  __shared__ float u_s[R][128];
  const int tid = threadIdx.x;
  const int ncol = a.fin_cols;
  int col = blockIdx.x % ncol;
  const RowChunk ch = a.chunks[blockIdx.x / ncol];
  // the projection this column chunk belongs to (block-uniform)
  int64_t Nout = a.Nout, ldo = a.ldo, pcol0 = 0;
  void* outp = a.out;
  int tab0 = 0, p = 0;
  if (a.n_proj > 1) {
    for (int q = 1; q < a.n_proj; ++q) if (col >= a.proj[q].fin0) p = q;
    const ProjEntry pe = a.proj[p];
    Nout = pe.Nout; ldo = pe.ldo; outp = pe.out; tab0 = pe.tab0;
    pcol0 = (int64_t)pe.tile0 * SK_BN;
    col -= pe.fin0;
  }
  const int64_t n = (int64_t)col * FIN_COLS + 2 * tid;
  const bool active = n < Nout;                     // Nout is a multiple of 8
  const int64_t kstride = a.pm * a.ldp;
  const bool lora_on = ch.t >= 0 && (a.U != nullptr || a.n_ext > 0);
  // A block's run time is a few dependent memory round trips plus the partial-sum traffic, so
  // the loads are requested in the order of their dependence depth: adapter entry, then u and
  // the factor (ranks up to 32 are prefetched into registers), then the partial sums.
  AdapterEntry e;
  e.A = nullptr; e.B = nullptr; e.rank = 0; e.scale = 0.f;
  float ureg[UPT];
  uint4 wa[4], wb[4];          // FORM_NT prefetch: rows n and n + 1 of the factor, 8 ranks per entry
  uint32_t wn[32];             // FORM_NN prefetch: columns n, n + 1 of factor row q
  const bf16_t* L = nullptr;
  bool pref = false;
  if (lora_on) {
    e = a.table[tab0 + ch.t];
    L = (const bf16_t*)(a.which ? e.B : e.A);
    const int r = e.rank;
    if (a.n_ext > 0) {
      // fused shrink: u = scale * (sum over the splits of this adapter's extended columns)
      const int roff = a.ext_roff[tab0 + ch.t];
      const int64_t ustride = a.pm * a.ldu;
#pragma unroll
      for (int i = 0; i < UPT; ++i) {
        const int j = (tid >> 7) + i * (FIN_THREADS >> 7), q = tid & 127;
        float sum = 0.f;
        if (j < ch.nrows && q < r) {
          const float* up = a.u_part + (int64_t)(ch.row0 + j) * a.ldu + ext_local(a, (ch.row0 + j) / SK_BM, p, roff) + q;
          for (int ks0 = 0; ks0 < a.ksplit; ks0 += 4) {
            float pu[4];
#pragma unroll
            for (int ii = 0; ii < 4; ++ii) pu[ii] = up[(ks0 + ii < a.ksplit ? ks0 + ii : a.ksplit - 1) * ustride];
#pragma unroll
            for (int ii = 0; ii < 4; ++ii) if (ks0 + ii < a.ksplit) sum += pu[ii];
          }
          sum *= e.scale;
        }
        // (ranks r .. r_stride - 1 are padding of the row: zeros, as the shrink kernels write them)
        if (col == 0 && a.u_out && j < ch.nrows && q < a.r_stride) a.u_out[(int64_t)(ch.row0 + j) * a.r_stride + q] = sum;
        ureg[i] = sum;
      }
    } else {
#pragma unroll
      for (int i = 0; i < UPT; ++i) {
        const int j = (tid >> 7) + i * (FIN_THREADS >> 7), q = tid & 127;
        ureg[i] = (j < ch.nrows && q < r) ? a.U[(int64_t)(ch.row0 + j) * a.r_stride + q] : 0.f;
      }
    }
    pref = r <= 32 && (FORM == FORM_NN || (r & 7) == 0);
    if (pref && active) {
      if (FORM == FORM_NT) {               // L[n * r + q]
#pragma unroll
        for (int qt = 0; qt < 4; ++qt)
          if (qt * 8 < r) {
            wa[qt] = *(const uint4*)(L + n * r + qt * 8);
            wb[qt] = *(const uint4*)(L + (n + 1) * r + qt * 8);
          }
      } else {                             // L[q * Nout + n]
#pragma unroll
        for (int q = 0; q < 32; ++q)
          if (q < r) wn[q] = *(const uint32_t*)(L + (int64_t)q * Nout + n);
      }
    }
  }
  // partial sums of every row of the chunk, in split order; four splits (32 loads) at a time
  float y0[R], y1[R];
  {
    const float* part = a.partials + (int64_t)ch.row0 * a.ldp + pcol0 + (active ? n : 0);
#pragma unroll
    for (int j = 0; j < R; ++j) { y0[j] = 0.f; y1[j] = 0.f; }
    for (int ks0 = 0; ks0 < a.ksplit; ks0 += 4) {
      float2 p[4][R];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int ks = ks0 + i < a.ksplit ? ks0 + i : a.ksplit - 1;
        const float* pk = part + ks * kstride;
#pragma unroll
        for (int j = 0; j < R; ++j) p[i][j] = *(const float2*)(pk + (j < ch.nrows ? j : 0) * a.ldp);
      }
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool on = ks0 + i < a.ksplit;
#pragma unroll
        for (int j = 0; j < R; ++j) {
          if (on && j < ch.nrows) { y0[j] += p[i][j].x; y1[j] += p[i][j].y; }
        }
      }
    }
  }
  if (lora_on) {
    const int r = e.rank;
#pragma unroll
    for (int i = 0; i < UPT; ++i) u_s[(tid >> 7) + i * (FIN_THREADS >> 7)][tid & 127] = ureg[i];
    __syncthreads();
    if (active) {
      if (pref && FORM == FORM_NT) {
#pragma unroll
        for (int qt = 0; qt < 4; ++qt)
          if (qt * 8 < r) {
            const uint32_t aw[4] = {wa[qt].x, wa[qt].y, wa[qt].z, wa[qt].w}, bw[4] = {wb[qt].x, wb[qt].y, wb[qt].z, wb[qt].w};
            float fa[8], fb[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
              fa[i] = __uint_as_float((aw[i >> 1] >> ((i & 1) * 16)) << 16);
              fb[i] = __uint_as_float((bw[i >> 1] >> ((i & 1) * 16)) << 16);
            }
#pragma unroll
            for (int j = 0; j < R; ++j) {
              float sa = 0.f, sb = 0.f;
#pragma unroll
              for (int i = 0; i < 8; ++i) {
                const float uq = u_s[j][qt * 8 + i];
                sa = fmaf(uq, fa[i], sa); sb = fmaf(uq, fb[i], sb);
              }
              y0[j] += sa; y1[j] += sb;
            }
          }
      } else if (pref) {
#pragma unroll
        for (int q = 0; q < 32; ++q)
          if (q < r) {
            const float fa = __uint_as_float(wn[q] << 16), fb = __uint_as_float(wn[q] & 0xffff0000u);
#pragma unroll
            for (int j = 0; j < R; ++j) { y0[j] = fmaf(u_s[j][q], fa, y0[j]); y1[j] = fmaf(u_s[j][q], fb, y1[j]); }
          }
      } else if (FORM == FORM_NT) {        // any rank: stream the factor
        for (int q = 0; q < r; ++q) {
          const float fa = bf16_bits_to_float(L[n * r + q]), fb = bf16_bits_to_float(L[(n + 1) * r + q]);
#pragma unroll
          for (int j = 0; j < R; ++j) { y0[j] = fmaf(u_s[j][q], fa, y0[j]); y1[j] = fmaf(u_s[j][q], fb, y1[j]); }
        }
      } else {
        for (int q = 0; q < r; ++q) {
          const uint32_t w = *(const uint32_t*)(L + (int64_t)q * Nout + n);
          const float fa = __uint_as_float(w << 16), fb = __uint_as_float(w & 0xffff0000u);
#pragma unroll
          for (int j = 0; j < R; ++j) { y0[j] = fmaf(u_s[j][q], fa, y0[j]); y1[j] = fmaf(u_s[j][q], fb, y1[j]); }
        }
      }
    }
  }
  if (!active) return;
#pragma unroll
  for (int j = 0; j < R; ++j) {
    if (j < ch.nrows) {
      const int64_t m = ch.row0 + j;
      const int64_t tok = a.perm ? a.perm[m] : m;
      if (OUT_F32) *(float2*)((float*)outp + tok * ldo + n) = make_float2(y0[j], y1[j]);
      else *(uint32_t*)((bf16_t*)outp + tok * ldo + n) = float_to_bf16_bits(y0[j]) | ((uint32_t)float_to_bf16_bits(y1[j]) << 16);
    }
  }
}

// dst[c][r] = src[r][c] for a bf16 matrix of R rows and C columns (both multiples of 8), 64 x 64
// tiles.  Used to give a large-batch GEMM whose weight is stored output-contiguous the
// contraction-contiguous form, whose LDS fragment reads are plain 16-byte reads.
__global__ __launch_bounds__(256) void transpose_bf16_kernel(const bf16_t* __restrict__ src, int64_t lds_,
                                                             bf16_t* __restrict__ dst, int64_t ldd, int64_t R, int64_t C) {
  __shared__ __attribute__((aligned(16))) bf16_t s[64][72];   // s[c][r]
  const int tid = threadIdx.x, tx = tid & 7, ty = tid >> 3;
  const int64_t r0 = (int64_t)blockIdx.y * 64, c0 = (int64_t)blockIdx.x * 64;
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int r = ty + 32 * i;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (r0 + r < R && c0 + tx * 8 < C) v = *(const uint4*)(src + (r0 + r) * lds_ + c0 + tx * 8);
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int j = 0; j < 8; ++j) s[tx * 8 + j][r] = (bf16_t)(w[j >> 1] >> ((j & 1) * 16));
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int c = ty + 32 * i;
    if (c0 + c < C && r0 + tx * 8 < R) *(uint4*)(dst + (c0 + c) * ldd + r0 + tx * 8) = *(const uint4*)&s[c][tx * 8];
  }
}

hipError_t launch_transpose_bf16(const bf16_t* src, int64_t lds, bf16_t* dst, int64_t ldd, int64_t R, int64_t C, hipStream_t stream) {
  if (R <= 0 || C <= 0) return hipSuccess;
  hipLaunchKernelGGL(transpose_bf16_kernel, dim3((unsigned)((C + 63) / 64), (unsigned)((R + 63) / 64)), dim3(256), 0, stream, src, lds, dst,
                     ldd, R, C);
  return hipGetLastError();
}

// rows of a batch from which transposing the weight into scratch pays for itself
static constexpr int64_t WT_MIN_ROWS = 4096;

// Raise a kernel's dynamic LDS limit once per device (done: bit i set = device i has it).
static hipError_t allow_lds(const void* kernel, int bytes, std::atomic<uint64_t>& done) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = 1ull << (dev & 63);
  if (done.load(std::memory_order_acquire) & bit) return hipSuccess;
  e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
  if (e == hipSuccess) done.fetch_or(bit, std::memory_order_release);
  return e;
}

// The small-batch kernels: products, then the finish.
template <int FORM, bool OUT_F32>
static hipError_t launch_small(const GemmArgs& a, bool packed, hipStream_t stream) {
  static std::atomic<uint64_t> done_sk{0}, done_skx{0};
  const int G = a.tiles_m * a.tiles_n;
  if (packed) {
    // packed weight: its fragments go straight into registers (gemm_decode.hip)
    hipError_t ed = launch_gemm_decode(a, stream);
    if (ed != hipSuccess || a.fin_in_kernel) return ed;
  } else {
    hipError_t e0 = a.n_ext > 0 ? allow_lds((const void*)gemm_skinny_kernel<FORM, true>, SK_LDS, done_skx)
                                : allow_lds((const void*)gemm_skinny_kernel<FORM, false>, SK_LDS, done_sk);
    if (e0 != hipSuccess) return e0;
    if (a.n_ext > 0) hipLaunchKernelGGL((gemm_skinny_kernel<FORM, true>), dim3(G * a.ksplit), dim3(256), SK_LDS, stream, a);
    else hipLaunchKernelGGL((gemm_skinny_kernel<FORM, false>), dim3(G * a.ksplit), dim3(256), SK_LDS, stream, a);
    e0 = hipGetLastError();
    if (e0 != hipSuccess) return e0;
  }
  const int64_t fin_blocks = (int64_t)a.fin_cols * a.n_chunks;
  hipLaunchKernelGGL((splitk_finish_kernel<FORM, OUT_F32>), dim3((unsigned)fin_blocks), dim3(FIN_THREADS), 0, stream, a);
  return hipGetLastError();
}

// How a call is tiled.  wide: the large-batch kernel (gemm_wide.hip); otherwise 128 x 128 tiles with
// the contraction split (small batches), which can also carry the shrink as 32 extended columns per
// column tile.
struct GemmPlan {
  bool wide = true;
  WidePlan w;
  int tiles_m = 0, tiles_n = 0, ksplit = 1;
  int64_t kchunk = 0, ldp = 0, pm = 0, ldu = 0;
  size_t bytes = 0, u_bytes = 0;       // partial sums (either kernel), of the extended columns
};

static constexpr int CUS = 256;        // compute units; every GEMM kernel here runs one workgroup on each

// The small-batch plan for a requested number of contraction splits.
static GemmPlan small_plan(int64_t s, int64_t T, int64_t Kc, int64_t Nout, int n_ext) {
  GemmPlan p;
  p.wide = false;
  p.tiles_m = (int)((T + SK_BM - 1) / SK_BM);
  p.tiles_n = (int)((Nout + SK_BN - 1) / SK_BN);
  int64_t kc = (Kc + s - 1) / s;
  kc = (kc + BK - 1) / BK * BK;
  p.kchunk = kc;
  p.ksplit = (int)((Kc + kc - 1) / kc);
  p.ldp = (int64_t)p.tiles_n * SK_BN;
  p.pm = (int64_t)p.tiles_m * SK_BM;
  p.bytes = (size_t)p.ksplit * p.pm * p.ldp * sizeof(float);
  if (n_ext > 0 && n_ext <= SK_BX * p.tiles_n) {
    p.ldu = (int64_t)p.tiles_n * SK_BX;
    p.u_bytes = (size_t)p.ksplit * p.pm * p.ldu * sizeof(float);
  }
  return p;
}

// Estimated run time of a small-batch plan in microseconds, from rates measured with one workgroup
// per compute unit: time per 64-deep k-tile (bound by the fill rate, less so when fewer than 256
// workgroups share it; the packed weight skips LDS), a fixed cost per round of workgroups, a separate
// shrink launch where the GEMM does not carry it, and the partial sums written once and read once.
// Only the ordering of the candidates matters.
static double small_cost(const GemmPlan& p, int n_ext, bool packed) {
  const int64_t wgs = (int64_t)p.tiles_m * p.tiles_n * p.ksplit;
  const int64_t rounds = (wgs + CUS - 1) / CUS;
  const int64_t ktiles = (p.kchunk + BK - 1) / BK;
  const double busy = wgs < CUS ? (double)wgs / CUS : 1.0;
  const double shrink = n_ext > 0 && p.u_bytes == 0 ? 15.0 : 0.0;
  if (!packed) return rounds * (ktiles * 0.9 * (0.75 + 0.25 * busy) + 4.5) + shrink + 3.5 + 2.0 * (double)(p.bytes + p.u_bytes) / 5.0e6;
  // (an unsplit contraction is finished in the kernel)
  const double finish = p.ksplit == 1 ? (n_ext > 0 ? 8.0 : 0.0) : 6.0 + 2.0 * (double)(p.bytes + p.u_bytes) / 8.0e6;
  return rounds * (ktiles * (0.45 + 0.22 * busy) + 9.0) + shrink + finish;
}

// The same for the large-batch kernel with adapters: the shrink and the row tiles' lists as launches,
// and per tile its extra contraction tiles (need: ranks of the adapters of a row tile, or of all).
static double wide_cost(const WidePlan& w, int64_t T, int need) {
  if (need <= 0) return w.us;
  const double share = T > 32 * w.mt ? (double)(32 * w.mt) / T : 1.0;
  const double extra = 1.0 + 2.0 * need / 64.0 * share;
  return w.us + 16.0 + (w.rounds + (w.tail_tiles ? 1 : 0)) * 1.4 * extra;
}

// The best small-batch plan for these sizes (us: its estimated time; left alone when none qualifies).
static bool best_small(int64_t T, int64_t Kc, int64_t Nout, int need, bool packed, size_t max_bytes, double* us, GemmPlan* best) {
  bool found = false;
  int64_t max_s = Kc / 256;                         // contraction values per split, at least
  if (max_s > 32) max_s = 32;
  if (max_s < 1) max_s = 1;
  int last = 0;
  for (int64_t s = 1; s <= max_s; ++s) {
    const GemmPlan p = small_plan(s, T, Kc, Nout, need);
    if (p.ksplit == last) continue;                 // rounding the chunk to whole k-tiles gave the same split
    last = p.ksplit;
    if ((int64_t)p.tiles_m * p.tiles_n * p.ksplit > 4 * CUS || p.bytes + p.u_bytes > max_bytes) break;
    const double c = small_cost(p, need, packed);
    if (c < *us) { *us = c; *best = p; found = true; }
  }
  return found;
}

// need: extended columns of the fullest row tile; packed: the weight has a packed copy; max_bytes: room
// for partial sums (the best plan that fits; the large-batch kernel unsplit needs none).
// small_only: only the 128 x 128 kernels are candidates (the several-projections pass exists for
// them alone); the large-batch plan is returned when none of them qualifies.
static GemmPlan gemm_plan(int64_t T, int64_t Kc, int64_t Nout, int need, bool packed, size_t max_bytes, bool small_only = false) {
  GemmPlan best;
  best.w = wide_plan(T, Kc, Nout, max_bytes);
  best.bytes = best.w.part_bytes;
  // at least half a round of 256 x 256 tiles: the large-batch kernel
  const int64_t G = ((T + 255) / 256) * ((Nout + 255) / 256);
  if (T <= 0 || Nout <= 0 || G > CUS / 2) return best;
  double us = small_only ? 1e30 : wide_cost(best.w, T, need);
  best_small(T, Kc, Nout, need, packed, max_bytes, &us, &best);
  return best;
}

// The plan of a call (the 128 x 128 kernels need the map's row chunks).
static GemmPlan call_plan(int64_t T, int64_t Kc, int64_t Nout, int need, bool packed, size_t max_bytes, bool has_chunks) {
  GemmPlan p = gemm_plan(T, Kc, Nout, need, packed, max_bytes);
  if (!p.wide && !has_chunks) {
    p.wide = true;
    p.w = wide_plan(T, Kc, Nout, max_bytes);
  }
  return p;
}

int gemm_tile_rows(int64_t T, int64_t Kc, int64_t Nout, int need, bool packed, size_t partial_bytes, bool has_chunks) {
  if (T <= 0 || Nout <= 0) return 0;
  const GemmPlan p = call_plan(T, Kc, Nout, need, packed, partial_bytes, has_chunks);
  return p.wide ? 32 * p.w.mt : 0;
}

int gemm_ext_room(int64_t Nout) { return (int)((Nout + SK_BN - 1) / SK_BN) * SK_BX; }

static int ext_carried_at_most(int64_t Nout, int n_ext) { return n_ext < gemm_ext_room(Nout) ? n_ext : gemm_ext_room(Nout); }

// (room for whichever kernel a call takes: a descriptor's packed weight and, where the map object is
// reused, the grouping are not known here)
size_t gemm_splitk_bytes(int64_t T, int64_t Kc, int64_t Nout, int n_ext) {
  if (T <= 0 || Nout <= 0) return 0;
  size_t bytes = wide_plan(T, Kc, Nout, SIZE_MAX).part_bytes;
  const int64_t G = ((T + 255) / 256) * ((Nout + 255) / 256);
  for (int packed = 0; packed < 2 && G <= CUS / 2; ++packed) {
    GemmPlan q;
    double us = 1e30;
    if (best_small(T, Kc, Nout, ext_carried_at_most(Nout, n_ext), packed != 0, SIZE_MAX, &us, &q) && q.bytes + q.u_bytes > bytes) bytes = q.bytes + q.u_bytes;
  }
  return bytes;
}

// A deep contraction whose 256 x 256 tiles leave more than half of the chip idle has to be split: the sums
// of the plan that needs the least room for them.  Elsewhere a pass does without where room is short: the
// large-batch kernel runs its last round unsplit.
size_t gemm_splitk_min_bytes(int64_t T, int64_t Kc, int64_t Nout, int n_ext) {
  if (T <= 0 || Nout <= 0 || Kc < 2048) return 0;
  const int64_t G = ((T + 255) / 256) * ((Nout + 255) / 256);
  if (G > CUS / 2) return 0;
  const GemmPlan p = small_plan(1, T, Kc, Nout, ext_carried_at_most(Nout, n_ext));
  const size_t small = p.bytes + p.u_bytes, wide = 2 * (size_t)G * 256 * 256 * sizeof(float);
  return small < wide ? small : wide;
}

size_t gemm_wt_bytes(int form, int64_t T, int64_t Kc, int64_t Nout) {
  if (form != FORM_NN || T < WT_MIN_ROWS || Kc <= 0 || Nout <= 0 || Kc > 65535 * 64) return 0;
  if (!gemm_plan(T, Kc, Nout, 0, false, SIZE_MAX).wide) return 0;
  return (size_t)Kc * Nout * sizeof(bf16_t);
}

bool gemm_can_fuse_shrink(int form, int64_t T, int64_t Kc, int64_t Nout, int need, bool ranks_mult8, bool packed,
                          size_t partial_bytes) {
  if (T <= 0 || Nout <= 0 || need <= 0) return false;
  if (form == FORM_NN && !ranks_mult8) return false;     // 16-byte DMA units must not straddle adapters
  const GemmPlan p = gemm_plan(T, Kc, Nout, need, packed, partial_bytes);
  return !p.wide && p.u_bytes > 0;
}

// Way the decode kernel's call is finished: the one asked for where its conditions hold, else the
// next best.  Both ways other than the generic finish kernel need the splits to divide a tile's
// 32 units and u of a tile's rows to fit in LDS.  The in-kernel way also needs its counters; with
// several splits it is only taken when every workgroup of the launch fits on the chip at once, so
// that the splits of a tile normally run at the same time (a split that does not see the others
// in time leaves its share to the last one: correct either way).  DECODE_FINISH_AUTO: in the
// kernel when there is one split and u is not waited for in vain (`ext` extended columns; the sums never
// leave the registers, only u crosses workgroups), a launch of its own otherwise
// (measured: the counters' round trips cost more than the second launch once 16 MB of partial
// sums have to cross anyway; 412 rows of q/k/v of 9912 + 2944 + 2944 columns, contraction 8440, 20 adapters of rank 8,
// waited 201 ms for workgroups that had no unit, 217 us with the second launch).
static int decode_finish_mode(const DecodeSync* sync, int n_adapters, int r_stride, int tiles_m, int tiles_n, int ksplit, int ext) {
  if (!sync || sync->mode == DECODE_FINISH_GENERIC || (n_adapters > 0 && !sync->grp_ids)) return DECODE_FINISH_GENERIC;
  if (n_adapters > 0 && r_stride > 128) return DECODE_FINISH_GENERIC;
  if (ksplit != 1 && ksplit != 2 && ksplit != 4 && ksplit != 8) return DECODE_FINISH_GENERIC;
  int want = sync->mode;
  if (want == DECODE_FINISH_AUTO) want = ksplit == 1 && decode_u_comes_first(tiles_m, tiles_n, ext, sync->cu_count) ? DECODE_FINISH_IN_KERNEL : DECODE_FINISH_LAUNCH;
  if (want == DECODE_FINISH_LAUNCH) return DECODE_FINISH_LAUNCH;
  const int64_t tiles = (int64_t)tiles_m * tiles_n;
  if (sync->counters && 2 * tiles + 2 * tiles_m <= DECODE_SYNC_INTS && (ksplit == 1 || tiles * ksplit <= sync->cu_count))
    return DECODE_FINISH_IN_KERNEL;
  return DECODE_FINISH_LAUNCH;
}

hipError_t launch_gemm_bf16(const bf16_t* Aop, int64_t lda, const bf16_t* Bop, int64_t ldb,
                            int form, int64_t T, int64_t Kc, int64_t Nout, const int32_t* perm,
                            const int32_t* seg_off, int n_adapters, const AdapterEntry* table,
                            int which, const float* U, int r_stride, void* out, int64_t ldo,
                            int out_is_f32, float* partials, size_t partial_bytes, const RowChunk* chunks,
                            int n_chunks, const GemmFuse* fuse, int need_unfused, bf16_t* wt_scratch, size_t wt_bytes, const bf16_t* Bt_kept, const LoraDma* dma,
                            const bf16_t* Bpacked, bool use_packed, const DecodeSync* sync, hipStream_t stream) {
  if (T <= 0 || Nout <= 0) return hipSuccess;
  if (ldb > (1 << 22)) return hipErrorInvalidValue;      // 32-bit byte offsets inside a weight tile
  const bool packed = Bpacked != nullptr && use_packed;
  if (partials == nullptr) partial_bytes = 0;
  GemmPlan p = call_plan(T, Kc, Nout, fuse ? fuse->need : n_adapters > 0 ? need_unfused : 0, packed, partial_bytes, chunks != nullptr);
  // the caller skipped the shrink: the conditions of gemm_can_fuse_shrink() must hold
  if (fuse && (!gemm_can_fuse_shrink(form, T, Kc, Nout, fuse->need, fuse->ranks_mult8, packed, partial_bytes) || chunks == nullptr))
    return hipErrorInvalidValue;
  if (p.wide) {
    WideArgs w;
    w.A = Aop; w.lda = lda; w.B = Bop; w.ldb = ldb; w.T = T; w.Kc = Kc; w.Nout = Nout;
    w.perm = perm; w.seg_off = seg_off; w.n_adapters = n_adapters; w.table = table; w.which = which;
    w.U = U; w.r_stride = r_stride; w.U2 = nullptr; w.lora_tiles = nullptr; w.zero_line = dma->zero_line;
    w.out = out; w.ldo = ldo; w.partials = partials;
    // the expand's operands by DMA when the shrink's launch left u as a bf16 split and the lists
    w.lora = n_adapters > 0 && U != nullptr ? WIDE_LORA_STAGED : WIDE_LORA_NONE;
    if (w.lora && dma->u2 && dma->tiles && dma->list_rows == 32 * p.w.mt) {
      w.U2 = dma->u2; w.lora_tiles = (const LoraTile*)dma->tiles; w.lora = WIDE_LORA_LISTS;
    }
    int wform = form;
    if (form == FORM_NN && Bt_kept != nullptr) {
      // weight stored [Kc][Nout], and the caller keeps a transposed copy of it
      w.B = Bt_kept; w.ldb = Kc; wform = FORM_NT;
    } else if (form == FORM_NN && wt_scratch != nullptr && wt_bytes >= gemm_wt_bytes(form, T, Kc, Nout) && gemm_wt_bytes(form, T, Kc, Nout) > 0) {
      // weight stored [Kc][Nout]: transpose it into scratch ([Nout][Kc]) and run the
      // contraction-contiguous kernel; the adapters' factors keep their storage
      hipError_t e = launch_transpose_bf16(Bop, ldb, wt_scratch, Kc, Kc, Nout, stream);
      if (e != hipSuccess) return e;
      w.B = wt_scratch; w.ldb = Kc; wform = FORM_NT;
    }
    return launch_gemm_wide(w, p.w, wform, form, out_is_f32, stream);
  }
  GemmArgs a;
  a.Aop = Aop; a.lda = lda; a.Bop = Bop; a.ldb = ldb; a.T = T; a.Kc = Kc; a.Nout = Nout;
  a.perm = perm; a.seg_off = seg_off; a.n_adapters = n_adapters; a.table = table; a.which = which;
  a.U = U; a.r_stride = r_stride; a.out = out; a.ldo = ldo;
  a.ext_cols = nullptr; a.ext_roff = nullptr; a.n_ext = 0; a.u_part = nullptr; a.ldu = 0; a.u_out = nullptr;
  a.ext_t0 = 0; a.ext_base = 0;
  memset(a.proj, 0, sizeof a.proj);
  a.n_proj = 1; a.fin_cols = (int)((Nout + FIN_COLS - 1) / FIN_COLS);
  a.fin_in_kernel = 0; a.out_is_f32 = out_is_f32; a.lform = form; a.spin_limit = 0;
  a.sync = nullptr; a.grp_ids = nullptr;
  if (fuse) {
    a.ext_cols = fuse->cols; a.ext_roff = fuse->roff; a.n_ext = fuse->n_ext;
    a.ext_t0 = fuse->t0; a.ext_base = fuse->ext_base; a.ext = fuse->rows;
    a.u_part = partials + p.bytes / sizeof(float); a.ldu = p.ldu; a.u_out = fuse->u_out;
    a.U = nullptr;
  }
  a.tiles_m = p.tiles_m; a.tiles_n = p.tiles_n; a.ksplit = p.ksplit; a.kchunk = p.kchunk;
  a.ldp = p.ldp; a.pm = p.pm; a.partials = partials; a.chunks = chunks; a.n_chunks = n_chunks;
  // a packed copy of the weight: the decode kernel reads it instead of Bop
  if (packed) {
    a.Bop = Bpacked; a.ldb = packed_weight_ksteps(Kc);
    a.fin_in_kernel = decode_finish_mode(sync, n_adapters, r_stride, p.tiles_m, p.tiles_n, p.ksplit, fuse ? fuse->need : 0);
    if (a.fin_in_kernel) { a.sync = sync->counters; a.grp_ids = sync->grp_ids; a.spin_limit = sync->spin_limit; }
  }
  if (form == FORM_NT)
    return out_is_f32 ? launch_small<FORM_NT, true>(a, packed, stream) : launch_small<FORM_NT, false>(a, packed, stream);
  return out_is_f32 ? launch_small<FORM_NN, true>(a, packed, stream) : launch_small<FORM_NN, false>(a, packed, stream);
}

// ---- few rows
bool gemm_thin_ok(int form, int64_t T, bool lora, int r_stride, const DecodeSync* sync) {
  return T > 0 && T <= THIN_ROWS && sync && (!lora || (sync->counters && form == FORM_NT && sync->grp_ids && r_stride <= 128)) &&
         (sync->mode == DECODE_FINISH_AUTO || sync->mode == DECODE_FINISH_IN_KERNEL);
}

hipError_t launch_gemm_bf16_thin(const bf16_t* Aop, int64_t lda, int form, int64_t T, int64_t Kc, const int32_t* perm, int n_adapters,
                                 const AdapterEntry* table, int which, const ProjEntry* proj_host, int n_proj, int out_is_f32,
                                 float* u, int r_stride, int max_tiles, const DecodeSync* sync, hipStream_t stream) {
  if (n_proj < 1 || n_proj > MAX_PROJ) return hipErrorInvalidValue;
  GemmArgs a;
  memset(&a, 0, sizeof a);
  a.Aop = Aop; a.lda = lda; a.T = T; a.Kc = Kc; a.perm = perm; a.n_adapters = n_adapters; a.table = table; a.which = which;
  a.u_out = u; a.r_stride = r_stride; a.out_is_f32 = out_is_f32; a.lform = form;
  a.sync = sync->counters; a.grp_ids = sync->grp_ids; a.spin_limit = sync->spin_limit < MID_POLLS ? sync->spin_limit : MID_POLLS;
  if (sync->counters) a.thin_u = (float*)(sync->counters + DECODE_SYNC_INTS);
  a.n_proj = n_proj; a.n_prod = n_adapters > 0 ? n_proj * max_tiles : 0;
  for (int q = 0; q < n_proj; ++q) a.proj[q] = proj_host[q];
  return launch_gemm_thin(a, stream);
}

// ---- some more rows
MidPlan gemm_mid_plan(int form, int64_t T, int64_t lda, int64_t Kc, const ProjEntry* proj_host, int n_proj, const MidLora& lora, int ext, size_t room,
                      const DecodeSync* sync) {
  if (T <= 16 || T > MID_ROWS || lda > (1 << 20) || n_proj < 1 || n_proj > MAX_PROJ || !sync || (lora.n > 0 && (!sync->counters || form != FORM_NT || !sync->grp_ids || lora.r_stride > 128)) ||
      (sync->mode != DECODE_FINISH_AUTO && sync->mode != DECODE_FINISH_IN_KERNEL))
    return MidPlan();
  int64_t cols = 0;
  for (int q = 0; q < n_proj; ++q) cols += proj_host[q].Nout;
  auto wide_us = [&]() {                                         // (it takes the projections one after the other)
    double us = 0.0;
    for (int q = 0; q < n_proj; ++q) us += wide_plan(T, Kc, proj_host[q].Nout, room).us;
    return us;
  };
  const MidPlan small = mid_plan(T, Kc, proj_host, n_proj, lora, sync->counters ? 4 : 1);     // (splits exchange sums)
  const MidPlan p = mid_taller(small, T, Kc, proj_host, n_proj, lora, mid_limit(T, Kc, cols, ext, wide_us));
  for (int q = 0; q < n_proj && p.rb; ++q)
    if ((proj_host[q].Nout + 32 * p.wn - 1) / (32 * p.wn) * p.ksplit > MID_CONSUMERS) return MidPlan();
  return p;
}

hipError_t launch_gemm_bf16_mid(const bf16_t* Aop, int64_t lda, int form, int64_t T, int64_t Kc, const int32_t* perm, const int32_t* seg_off, int n_adapters,
                                const AdapterEntry* table, int which, const ProjEntry* proj_host, int n_proj, int out_is_f32,
                                float* u, int r_stride, const MidPlan& plan, int proj_jobs, const bf16_t* zero_line, const DecodeSync* sync,
                                hipStream_t stream) {
  if (n_proj < 1 || n_proj > MAX_PROJ || plan.rb == 0) return hipErrorInvalidValue;
  GemmArgs a;
  memset(&a, 0, sizeof a);
  a.Aop = Aop; a.lda = lda; a.T = T; a.Kc = Kc; a.perm = perm; a.seg_off = seg_off; a.n_adapters = n_adapters; a.table = table; a.which = which;
  a.u_out = u; a.r_stride = r_stride; a.out_is_f32 = out_is_f32; a.lform = form;
  a.grp_ids = sync->grp_ids; a.spin_limit = sync->spin_limit < MID_POLLS ? sync->spin_limit : MID_POLLS; a.zero_line = zero_line;
  if (sync->counters) {
    a.turns = sync->counters + DECODE_SYNC_INTS + THIN_U_FLOATS;
    a.mid_u = (float*)(a.turns + TURN_INTS);
    a.partials = (float*)(sync->counters + (SYNC_INTS - MID_PART_FLOATS));
  }
  a.n_proj = n_proj;
  for (int q = 0; q < n_proj; ++q) a.proj[q] = proj_host[q];
  a.proj_jobs = n_adapters > 0 ? proj_jobs : 0;
  return launch_gemm_mid(a, plan, sync->cu_count, stream);
}

// ---- several projections in one pass
static int64_t multi_tiles(const ProjEntry* proj, int n_proj) {
  int64_t tiles = 0;
  for (int p = 0; p < n_proj; ++p) tiles += (proj[p].Nout + SK_BN - 1) / SK_BN;
  return tiles;
}

int gemm_multi_ext_room(const ProjEntry* proj_host, int n_proj) { return (int)multi_tiles(proj_host, n_proj) * SK_BX; }

size_t gemm_multi_bytes(int64_t T, int64_t Kc, const ProjEntry* proj_host, int n_proj, int n_ext) {
  if (T <= 0 || n_proj <= 0) return 0;
  const int room = gemm_multi_ext_room(proj_host, n_proj), need = n_ext < room ? n_ext : room;
  size_t bytes = 0;
  for (int packed = 0; packed < 2; ++packed) {
    const GemmPlan p = gemm_plan(T, Kc, multi_tiles(proj_host, n_proj) * SK_BN, need, packed != 0, SIZE_MAX, true);
    if (!p.wide && p.bytes + p.u_bytes > bytes) bytes = p.bytes + p.u_bytes;
  }
  return bytes;
}

bool gemm_multi_ok(int form, int64_t T, int64_t Kc, const ProjEntry* proj_host, int n_proj, int need,
                   bool ranks_mult8, bool packed, size_t partial_bytes) {
  if (T <= 0 || n_proj < 2 || need < 0) return false;
  if (need > 0 && form == FORM_NN && !ranks_mult8) return false;
  const int64_t tiles = multi_tiles(proj_host, n_proj);
  if (tiles * SK_BN > (1 << 24)) return false;
  const GemmPlan p = gemm_plan(T, Kc, tiles * SK_BN, need, packed, partial_bytes, true);
  return !p.wide && (need == 0 || p.u_bytes > 0);
}

hipError_t launch_gemm_bf16_multi(const bf16_t* Aop, int64_t lda, int form, int64_t T, int64_t Kc,
                                  const int32_t* perm, const int32_t* seg_off, int n_adapters,
                                  const AdapterEntry* table, const ProjEntry* proj_host,
                                  int n_proj, int out_is_f32, float* partials,
                                  size_t partial_bytes, const RowChunk* chunks, int n_chunks,
                                  const GemmFuse* fuse, int packed, const DecodeSync* sync, int r_stride,
                                  hipStream_t stream) {
  const int need = fuse ? fuse->need : 0;
  if (!gemm_multi_ok(form, T, Kc, proj_host, n_proj, need, fuse ? fuse->ranks_mult8 : true, packed != 0,
                     partials ? partial_bytes : 0) || chunks == nullptr || n_proj > MAX_PROJ)
    return hipErrorInvalidValue;
  const int64_t tiles = multi_tiles(proj_host, n_proj);
  const GemmPlan p = gemm_plan(T, Kc, tiles * SK_BN, need, packed != 0, partials ? partial_bytes : 0, true);
  GemmArgs a;
  a.Aop = Aop; a.lda = lda; a.Bop = (const bf16_t*)proj_host[0].W; a.ldb = proj_host[0].ldw;
  a.T = T; a.Kc = Kc; a.Nout = proj_host[0].Nout;
  a.perm = perm; a.seg_off = seg_off; a.n_adapters = n_adapters; a.table = table; a.which = 1;
  a.U = nullptr; a.r_stride = 0; a.out = proj_host[0].out; a.ldo = proj_host[0].ldo;
  a.tiles_m = p.tiles_m; a.tiles_n = p.tiles_n; a.ksplit = p.ksplit; a.kchunk = p.kchunk;
  a.partials = partials; a.ldp = p.ldp; a.pm = p.pm; a.chunks = chunks; a.n_chunks = n_chunks;
  a.ext_cols = nullptr; a.ext_roff = nullptr; a.n_ext = 0; a.u_part = nullptr; a.ldu = 0; a.u_out = nullptr;
  a.ext_t0 = 0; a.ext_base = 0;
  if (fuse) {
    a.ext_cols = fuse->cols; a.ext_roff = fuse->roff; a.n_ext = fuse->n_ext;
    a.ext_t0 = fuse->t0; a.ext_base = fuse->ext_base; a.ext = fuse->rows;
    a.u_part = partials + p.bytes / sizeof(float); a.ldu = p.ldu;
  }
  memset(a.proj, 0, sizeof a.proj);
  for (int q = 0; q < n_proj; ++q) a.proj[q] = proj_host[q];
  a.n_proj = n_proj;
  int fin_cols = 0;
  for (int q = 0; q < n_proj; ++q) fin_cols += (int)((proj_host[q].Nout + FIN_COLS - 1) / FIN_COLS);
  a.fin_cols = fin_cols;
  // (packed: every ProjEntry::W is a packed copy and ProjEntry::ldw its k-steps per column block)
  const bool pk = packed != 0 && (fuse == nullptr || form == FORM_NT);
  if (packed != 0 && !pk) return hipErrorInvalidValue;
  a.fin_in_kernel = 0; a.out_is_f32 = out_is_f32; a.lform = form; a.spin_limit = 0;
  a.sync = nullptr; a.grp_ids = nullptr;
  if (pk) a.fin_in_kernel = decode_finish_mode(sync, n_adapters, r_stride, p.tiles_m, p.tiles_n, p.ksplit, need);
  if (a.fin_in_kernel) {
    a.sync = sync->counters; a.grp_ids = sync->grp_ids; a.spin_limit = sync->spin_limit;
    a.r_stride = r_stride;
  }
  if (form == FORM_NT)
    return out_is_f32 ? launch_small<FORM_NT, true>(a, pk, stream) : launch_small<FORM_NT, false>(a, pk, stream);
  return out_is_f32 ? launch_small<FORM_NN, true>(a, pk, stream) : launch_small<FORM_NN, false>(a, pk, stream);
}

}  // namespace marlaas
