// Base GEMM of large batches on the bf16 matrix cores with the LoRA expand fused in:
//
//   out[tok(m), :] = A[tok(m), :] * B  +  u(m) * L_t          (m in the segment of adapter t)
//
// m runs over tokens grouped by adapter (tok = perm), B is the shared frozen base weight (paper
// Sec. 1 principle (1)), u = s_t * (x A_t) is the shrink's result, and L_t is the adapter's
// output-side factor (B_t in forward, A_t in backward).
//
// Tile: 32 MT rows x 256 columns per workgroup of 4 waves (2 x 2), each wave 16 MT x 128 as MT x 8
// MFMA 16x16x32 accumulators.  The contraction runs in k-tiles of 64 that go from global memory
// straight into LDS (16 bytes per lane, no register staging; every row segment is one whole
// 128-byte line) through two slots.  16-byte units are XOR-swizzled so that DMA writes and fragment
// reads are bank-conflict free.
//
// One workgroup per compute unit walks a list of work items (WidePlan): whole tiles, then at most
// one piece of a tile whose contraction is split, where the tiles of the last round would leave
// compute units idle.  The next item's first two k-tiles are requested before the results of the
// current one are stored, so neither the token gather nor the first memory latency nor the burst of
// stores stands between two tiles.  Measured (16384 x 16384 outputs, K = 2048 / 4096 / 8192): as one
// workgroup per tile each tile paid 12 us besides its k-tiles of 1.36 us.
// What bounds a k-tile: 2048 cycles of matrix instructions a wave, with one wave per SIMD, so every instruction that does not
// fit an MFMA's shadow is added to them (stamps, 40960 rows, 4096 x 14336: 2342 cycles with requests in one piece, 2200
// with one instruction a shadow; the clock falls as the power limit has it, 3.50 -> 3.41 ms with the expand, 2.6 %).
#include "gemm_args.h"

#include <atomic>


namespace marlaas {

static constexpr int WK = 64;                               // k-tile
static constexpr int WN = 256;                              // columns of a tile
static constexpr int W_THREADS = 256;
static constexpr int W_B_BYTES = WN * WK * 2;               // 32 KB: the weight part of a slot
static constexpr int W_NT = 8;                              // 16-column blocks per wave
static constexpr int W_LT_BYTES = (LT_MAX + 1) * (int)sizeof(LoraTile);   // an item's list of extra contraction tiles
static_assert(W_LT_BYTES == 4096, "the list is fetched with one DMA instruction per wave");
template <int MT> static constexpr int wide_lds() { return 2 * (32 * MT * WK * 2 + W_B_BYTES) + W_LT_BYTES + 3 * 32 * MT * 4; }

// Swizzle of 16-byte unit `unit` (of 32) of k-row `k` in a [64][256] bf16 tile.
__device__ __forceinline__ int kn_swz(int k) { return ((k & 3) << 2) | (((k >> 3) & 1) << 1); }
__device__ __forceinline__ int swz_kn(int k, int unit) { return k * 512 + ((unit ^ kn_swz(k)) << 4); }

__device__ __forceinline__ uint4 pack8(const bf16_t* o) {
  uint4 pk;
  pk.x = o[0] | ((uint32_t)o[1] << 16); pk.y = o[2] | ((uint32_t)o[3] << 16);
  pk.z = o[4] | ((uint32_t)o[5] << 16); pk.w = o[6] | ((uint32_t)o[7] << 16);
  return pk;
}
// Two 16 x 16 accumulator blocks side by side (lane: row lane % 16, columns 4 (lane / 16) .. + 3 of
// each) as eight consecutive bf16 columns per lane: odd lane groups take the right-hand block.
// Lane group lg ends up with columns 16 (lg & 1) + 8 (lg / 2) .. + 7 of the 32.
__device__ __forceinline__ uint4 pair_rows(const f32x4& l, const f32x4& r) {
  const auto a = __builtin_amdgcn_permlane16_swap(pack2(l[0], l[1]), pack2(r[0], r[1]), false, false);
  const auto b = __builtin_amdgcn_permlane16_swap(pack2(l[2], l[3]), pack2(r[2], r[3]), false, false);
  return make_uint4(a[0], b[0], a[1], b[1]);
}

// 16 bytes of results, not kept in L2: the 32 MB of a round of tiles would push out the panels that the
// next tiles share (zero operands, K = 4096: 1.26 -> 1.17 ms for 16384 x 16384 outputs).
__device__ __forceinline__ void store_out(void* p, uint4 v) {
  typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
  __builtin_nontemporal_store(u32x4{v.x, v.y, v.z, v.w}, (u32x4*)p);
}
__device__ __forceinline__ void store_out(void* p, const f32x4& v) { __builtin_nontemporal_store(v, (f32x4*)p); }

// c += a b on an accumulator that stays where it is: left to choose, the compiler moves accumulators between the two register
// files, with waits, in every k-tile but the steady ones, and spills (16384 rows, 14336 x 4096, a task's forward and backward
// 2960 us, 2910 so).  It knows nothing of the instruction: whoever reads accumulators otherwise calls acc_settle first, and no
// vector arithmetic writes an operand right before; where fragments are put together from transposing reads it does (MOVED: two
// wait states in front of every product; 3000 rows of 8 adapters, 4096 x 4096, math layout without a transposed copy, with the loop as it is now 160 -> 111 us all the
// same, 2500 rows, 8192 x 2048, 193 -> 120, forward and backward of 3500 rows, 2048 x 8192, 356 -> 282).
// tests/test_generated_code.py reads the code for both.
template <bool MOVED>
__device__ __forceinline__ void mma(f32x4& c, bf16x8 a, bf16x8 b) {
  if (MOVED) asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
  else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b));
}
template <bool MOVED>
__device__ __forceinline__ void mma_first(f32x4& c, bf16x8 a, bf16x8 b) {     // c = a b
  if (MOVED) asm volatile("s_nop 1\n\tv_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(c) : "v"(a), "v"(b));
  else asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, 0" : "=a"(c) : "v"(a), "v"(b));
}
__device__ __forceinline__ void acc_settle() { asm volatile("s_nop 15\n\ts_nop 15" ::: "memory"); }
// An accumulator's values as arithmetic sees them, read here and not earlier: left to the compiler all
// of them are copied out ahead of the stores, into registers that are not there.
__device__ __forceinline__ f32x4 acc_read(f32x4 c) { asm volatile("" : "+v"(c)); return c; }
// The value, recomputed from here on: what is derived from it is not kept in registers across the
// item loop (the accumulators leave few, and a reload from scratch would wait for every request).
__device__ __forceinline__ int fresh(int v) { asm volatile("" : "+v"(v)); return v; }

// all but the VM youngest vector-memory requests and the LG youngest LDS reads of this wave are complete, everywhere
template <int VM, int LG>
__device__ __forceinline__ void wide_meet() {
  asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(%1)\n\ts_barrier" :: "n"(VM > 63 ? 63 : VM), "n"(LG) : "memory");
}

// a pointer that is the same in all lanes, in scalar registers
__device__ __forceinline__ const char* uniform(const char* p) {
  const uint64_t v = (uint64_t)(uintptr_t)p;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((int)v), hi = __builtin_amdgcn_readfirstlane((int)(v >> 32));
  return (const char*)(uintptr_t)((uint64_t)hi << 32 | lo);
}

// every vector-memory request of this wave is complete
__device__ __forceinline__ void wide_drain() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// The MFMAs take the weight fragment as their first operand, so a block of the accumulators is the
// transpose of the output block: in a 16 x 16 block lane l holds output row (token) l % 16 and the
// four consecutive output columns 4 (l / 16) .. + 3.
// FORM: storage of the weight operand; LFORM: storage of the adapters' expand factors (they
// differ when a transposed copy of the weight is read).
template <int MT, int FORM, bool OUT_F32, int LFORM>
__global__ __launch_bounds__(W_THREADS) void gemm_wide_kernel(WideArgs a) {
  constexpr int HB = MT / 2;                                // row blocks of a phase
  constexpr int ROWS = 32 * MT, A_BYTES = ROWS * WK * 2, SLOT = A_BYTES + W_B_BYTES;
  constexpr int C1 = (10 + HB) / 3, C2 = (9 + HB) / 3, C3 = (8 + HB) / 3;   // the 8 + HB first requests over three phases
  static_assert(C1 + C2 + C3 == 8 + HB, "");
  constexpr int NST = (OUT_F32 ? 8 : 4) * MT;               // stores per wave of a whole tile
  extern __shared__ __attribute__((aligned(128))) char smem[];
  char* lt_s = smem + 2 * SLOT;
  int32_t* tok3 = (int32_t*)(lt_s + W_LT_BYTES);            // [3][ROWS] tokens of items i - 1, i, i + 1

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int frow = lane & 15, fg = lane >> 4;               // MFMA operand: row, 8-wide quarter of the 32-wide k step

  // ---- work items.  Workgroup b runs on XCD b mod 8, each with its own L2: an XCD walks a compact
  // run of tiles, groups of row tiles sharing their column tiles.
  const int xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
  const int tail_items = a.tail_tiles * a.tail_split;
  const int tq = tail_items >> 3, tr = tail_items & 7;
  const int n_items = a.rounds + (idx < tq + (xcd < tr ? 1 : 0) ? 1 : 0);
  if (n_items == 0) return;
  int64_t m0 = 0, n0 = 0, kbeg = 0, kend = 0;
  int tm = 0, split = 0, ptile = -1;                        // ptile: tile among the split ones, -1: whole tile
#define W_ITEM(i_)                                                                                        \
  do {                                                                                                    \
    int _t;                                                                                               \
    kbeg = 0; kend = a.Kc; split = 0; ptile = -1;                                                         \
    if ((i_) < a.rounds) {                                                                                \
      /* (turned by one per round: else a workgroup keeps its row tile, and the one whose row tile has */  \
      /* the most adapters is late in every round)                                                      */  \
      _t = (xcd * a.rounds + (i_)) * 32 + ((idx + (i_)) & 31);                                            \
    } else {                                                                                              \
      const int _j = xcd * tq + (xcd < tr ? xcd : tr) + idx;                                              \
      split = _j / a.tail_tiles;                                                                          \
      const int _p = _j - split * a.tail_tiles;                                                           \
      _t = a.rounds * 256 + _p;                                                                           \
      if (a.tail_split > 1) {                                                                             \
        ptile = _p;                                                                                       \
        kbeg = split * a.tail_kchunk;                                                                     \
        if (split + 1 < a.tail_split) kend = kbeg + a.tail_kchunk;                                        \
      }                                                                                                   \
    }                                                                                                     \
    const int _tn = wide_tile(_t, MT, a.tiles_m, a.tiles_n, &tm);                                         \
    m0 = (int64_t)tm * ROWS; n0 = (int64_t)_tn * WN;                                                      \
  } while (0)

  // tokens of item i_ -> tok3[i_ % 3] (rows past the end repeat the last token)
#define W_TOKENS(i_)                                                                                      \
  do {                                                                                                    \
    const int64_t _m0 = m0, _n0 = n0, _kb = kbeg, _ke = kend;                                             \
    const int _tm = tm, _sp = split, _pt = ptile;                                                         \
    W_ITEM(i_);                                                                                           \
    int64_t _m = m0 + wave * 64 + lane;                                                                   \
    m0 = _m0; n0 = _n0; kbeg = _kb; kend = _ke; tm = _tm; split = _sp; ptile = _pt;                       \
    if (_m >= a.T) _m = a.T - 1;                                                                          \
    if (wave * 64 < ROWS) {                                                                               \
      int32_t* _d = tok3 + ((i_) % 3) * ROWS + wave * 64;                                                 \
      if (a.perm) __builtin_amdgcn_global_load_lds((gptr_t)(a.perm + _m), (lptr_t)_d, 4, 0, 0);           \
      else _d[lane] = (int32_t)_m;                                                                        \
    }                                                                                                     \
  } while (0)

  // ---- DMA geometry.  One wave instruction moves 64 x 16 B = 1 KB into consecutive LDS bytes.
  // Row-k tiles (128 B per row): 8 rows per instruction, lane l writes unit (l & 7) of row (l >> 3)
  // and so fetches the global unit (l & 7) ^ swizzle(row).  k-n tiles (512 B per k-row): 2 k-rows
  // per instruction.  Per k-tile a wave issues MT instructions for A and 8 for B.  B's addresses
  // are one wave-uniform base, advanced per k-tile with scalar arithmetic, plus a constant 32-bit
  // byte offset per lane and instruction (a weight tile spans less than 4 GB: leading dimensions
  // are at most 2^22 elements); gathered rows need full 64-bit addresses.
  const bf16_t* a_src[MT];
  const char* b_base = nullptr;      // wave-uniform
  uint32_t b_off[8];
  const int64_t b_step = FORM == FORM_NT ? WK * 2 : (int64_t)WK * a.ldb * 2;
  int ntile = 0, tail_k = WK;        // k-tiles of the item; contraction values of its last one
  int nfast = 0;                     // k-tiles that are whole
  const int a_dma = wave * MT * 1024, b_dma = A_BYTES + wave * 8 * 1024;
  const uint32_t lds0 = (uint32_t)(uintptr_t)(lptr_t)smem;
  const uint32_t a_to = lds0 + ((wave >> 1) * (16 * MT) + (wave & 1) * (8 * HB)) * 128, b_to = lds0 + b_dma;   // of request 0, slot 0
  // Instruction j < HB of a wave moves 8 of the rows that phases 0 and 1 multiply (the first half of
  // each wave row's row blocks), instruction j >= HB rows of the other half.
#define W_AROW(j_) (((j_) >= HB ? 8 * MT : 0) + (wave * HB + (j_) % HB) / (2 * HB) * (16 * MT) + (wave * HB + (j_) % HB) % (2 * HB) * 8)
#define W_SETUP(i_)                                                                                       \
  do {                                                                                                    \
    const int _ln = fresh(lane);                                                                          \
    ntile = (int)((kend - kbeg + WK - 1) / WK);                                                           \
    tail_k = (int)(kend - kbeg) - (ntile - 1) * WK;                                                       \
    nfast = tail_k < WK ? ntile - 1 : ntile;                                                              \
    const int32_t* _tok = tok3 + ((i_) % 3) * ROWS;                                                       \
    _Pragma("unroll") for (int j = 0; j < MT; ++j) {                                                      \
      const int _row = W_AROW(j) + (_ln >> 3);                                                 \
      const int _unit = (_ln & 7) ^ ((_row >> 1) & 7);                                                   \
      a_src[j] = a.A + (int64_t)_tok[_row] * a.lda + kbeg + _unit * 8;                                    \
    }                                                                                                     \
    _Pragma("unroll") for (int j = 0; j < 8; ++j) {                                                       \
      if (FORM == FORM_NT) {                                                                              \
        const int _row = (wave * 8 + j) * 8 + (_ln >> 3);                                                \
        const int _unit = (_ln & 7) ^ ((_row >> 1) & 7);                                                 \
        int64_t _n = n0 + _row;                                                                           \
        if (_n >= a.Nout) _n = a.Nout - 1;           /* clamped columns are never stored */               \
        b_off[j] = (uint32_t)(((_n - n0) * a.ldb + _unit * 8) * 2);                                       \
      } else {                                                                                            \
        const int _k = (wave * 8 + j) * 2 + (_ln >> 5);                                                  \
        int64_t _n = n0 + ((_ln & 31) ^ kn_swz(_k)) * 8;                                                 \
        if (_n >= a.Nout) _n = a.Nout - 8;                                                                \
        b_off[j] = (uint32_t)((_k * a.ldb + (_n - n0)) * 2);                                              \
      }                                                                                                   \
    }                                                                                                     \
    b_base = uniform((const char*)(FORM == FORM_NT ? a.B + n0 * a.ldb + kbeg : a.B + kbeg * a.ldb + n0)); \
  } while (0)
  // the last k-tile of a contraction that is no multiple of 64 fetches zeros beyond the end
#define W_DMA_A(slot_, j_, tail_)                                                                              \
  do {                                                                                                    \
    const bf16_t* _src = a_src[j_];                                                                       \
    if (tail_) {                                                                                          \
      const int _ln = fresh(lane);                                                                        \
      const int _unit = (_ln & 7) ^ (((W_AROW(j_) + (_ln >> 3)) >> 1) & 7);                               \
      if (_unit * 8 >= (tail_)) _src = a.zero_line;                                                       \
    }                                                                                                     \
    __builtin_amdgcn_global_load_lds((gptr_t)_src, (lptr_t)(smem + (slot_) * SLOT + W_AROW(j_) * 128), 16, 0, 0); \
    a_src[j_] += WK;                                                                                      \
  } while (0)
#define W_DMA_B(slot_, j_, tail_)                                                                              \
  do {                                                                                                    \
    char* _sb = smem + (slot_) * SLOT + b_dma + (j_) * 1024;                                              \
    if (tail_) {                                                                                          \
      const int _k = FORM == FORM_NT ? ((fresh(lane) & 7) ^ ((((wave * 8 + (j_)) * 8 + (fresh(lane) >> 3)) >> 1) & 7)) * 8 \
                                     : (wave * 8 + (j_)) * 2 + (fresh(lane) >> 5);                               \
      const char* _src = _k < (tail_) ? b_base + b_off[j_] : (const char*)a.zero_line;                     \
      __builtin_amdgcn_global_load_lds((gptr_t)_src, (lptr_t)_sb, 16, 0, 0);                              \
    } else {                                                                                              \
      /* scalar base + 32-bit lane offset: the builtin only emits the 64-bit-address form, which */       \
      /* costs a 64-bit vector add per request (m0 = LDS byte address of lane 0's 16 bytes)       */      \
      const uint32_t _lds = (uint32_t)(uintptr_t)(lptr_t)_sb;                                             \
      asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1"                        \
                   :: "v"(b_off[j_]), "s"(b_base), "s"(_lds) : "memory", "m0");                           \
    }                                                                                                     \
    if ((j_) == 7) b_base += b_step;                                                                              \
  } while (0)
  // Request q_ of the part of a k-tile that is needed first: its weights (8) and the first half's rows (HB)
#define W_DMA_FIRST(slot_, q_, tail_)                                                                          \
  do { if ((q_) < 8) W_DMA_B(slot_, (q_) & 7, tail_); else W_DMA_A(slot_, ((q_) - 8) % HB, tail_); } while (0)
  // The same of a whole k-tile in three parts, each one instruction in the shadow of an MFMA of its own (W_PHASE): m0 = LDS
  // byte address of lane 0's 16 bytes, the request, the address's advance.  Nothing else between the first two parts writes m0.
#define W_PART_A(part_, to_, j_)                                                                          \
  do {                                                                                                    \
    if ((part_) == 0) asm volatile("s_add_u32 m0, %0, %1" :: "s"((to_) + a_to), "n"(((j_) >= HB ? 8 * MT * 128 : 0) + (j_) % HB * 1024) : "memory", "m0", "scc"); \
    if ((part_) == 1) asm volatile("global_load_lds_dwordx4 %0, off" :: "v"(a_src[j_]) : "memory");       \
    if ((part_) == 2) a_src[j_] += WK;                                                                    \
  } while (0)
#define W_PART_B(part_, to_, j_)                                                                          \
  do {                                                                                                    \
    if ((part_) == 0) asm volatile("s_add_u32 m0, %0, %1" :: "s"((to_) + b_to), "n"((j_) * 1024) : "memory", "m0", "scc"); \
    if ((part_) == 1) asm volatile("global_load_lds_dwordx4 %0, %1" :: "v"(b_off[j_]), "s"(b_base) : "memory"); \
    if ((part_) == 2 && (j_) == 7) b_base += b_step;                                                      \
  } while (0)
#define W_PART_FIRST(part_, to_, q_)                                                                      \
  do { if ((q_) < 8) W_PART_B(part_, to_, (q_) & 7); else W_PART_A(part_, to_, ((q_) - 8) % HB); } while (0)
  // contraction values of k-tile kt_
#define W_KLEN(kt_) ((kt_) == ntile - 1 ? tail_k : WK)
  // an item's first requests, oldest first: the tokens of the item after it, its list of extra
  // contraction tiles, its first k-tile and the part of the second that is needed first
#define W_REQUEST(i_)                                                                                     \
  do {                                                                                                    \
    if ((i_) + 1 < n_items) W_TOKENS((i_) + 1);                                                           \
    if (a.lora == WIDE_LORA_LISTS && split == 0)                                                          \
      __builtin_amdgcn_global_load_lds((gptr_t)((const char*)(a.lora_tiles + (int64_t)tm * (LT_MAX + 1)) + wave * 1024 + lane * 16), \
                                       (lptr_t)(lt_s + wave * 1024), 16, 0, 0);                           \
    const int _k0 = W_KLEN(0), _k1 = W_KLEN(1);                                                           \
    if (_k0 == WK) { _Pragma("unroll") for (int _q = 0; _q < 8 + HB; ++_q) W_DMA_FIRST(0, _q, 0); }  \
    else { _Pragma("unroll") for (int _q = 0; _q < 8 + HB; ++_q) W_DMA_FIRST(0, _q, _k0); }         \
    _Pragma("unroll") for (int _j = HB; _j < MT; ++_j) W_DMA_A(0, _j, _k0);                         \
    if (ntile > 1) {                                                                                      \
      if (_k1 == WK) { _Pragma("unroll") for (int _q = 0; _q < 8 + HB; ++_q) W_DMA_FIRST(1, _q, 0); } \
      else { _Pragma("unroll") for (int _q = 0; _q < 8 + HB; ++_q) W_DMA_FIRST(1, _q, _k1); }       \
    }                                                                                                     \
  } while (0)

  // ---- fragment geometry: 16 rows x 32 contraction values per MFMA operand, lane l supplies row
  // l % 16, values 8 (l / 16) .. + 7
  const int a_off_row = (wm * (MT * 16) + frow) * 128, b_off_row = (wn * 128 + frow) * 128;
  const int f_swz = (frow >> 1) & 7;                 // (rows 16 apart share the swizzle)
  int btr[W_NT];
  {
    // transposing reads of a [k][n] tile: the 16 lanes of group fg fetch the 4 x 16 block of rows
    // 8 fg .. + 3 (lane i: row i / 4, columns 4 (i % 4) .. + 3) and each receives its own column
    const int kb = fg * 8 + (frow >> 2);
    for (int nt = 0; nt < W_NT; ++nt) {
      const int ncol = wn * 128 + nt * 16 + 4 * (frow & 3);
      btr[nt] = swz_kn(kb, ncol >> 3) + (ncol & 7) * 2;
    }
  }
#define W_READ_X(slot_, ks_, mt_, dst_)                                                                   \
  dst_ = *(const bf16x8*)(smem + (slot_) * SLOT + a_off_row + (mt_) * 2048 + ((((ks_) * 4 + fg) ^ f_swz) << 4))
  // The main loop's reads: byte addresses of the wave's rows of x and of the weight in k-step 0 and 1, each moved to
  // the other slot (toggle) behind its last use in a k-tile.
  typedef const bf16x8 __attribute__((address_space(3)))* lds_x8;
  uint32_t x_at[2] = {0, 0}, w_at[2] = {0, 0};
#define W_TOGGLE(r_) asm volatile("v_add_u32 %0, %1, %0" : "+v"(r_) : "s"(_nto - _to))
#define W_NEXT_X(ks_, mt_, dst_) dst_ = *(lds_x8)(x_at[ks_] + (mt_) * 2048)
#define W_NEXT_W(slot_, ks_, nt_, dst_)                                                                   \
  do {                                                                                                    \
    if (FORM == FORM_NT) dst_ = *(lds_x8)(w_at[ks_] + (nt_) * 2048);                                      \
    else W_READ_W(FORM, slot_, ks_, nt_, dst_);                                                           \
  } while (0)
#define W_READ_W(form_, slot_, ks_, nt_, dst_)                                                            \
  do {                                                                                                    \
    const char* _bs = smem + (slot_) * SLOT + A_BYTES;                                                    \
    if ((form_) == FORM_NT) {                                                                             \
      dst_ = *(const bf16x8*)(_bs + b_off_row + (nt_) * 2048 + ((((ks_) * 4 + fg) ^ f_swz) << 4));        \
    } else {                                                                                              \
      const char* _p = _bs + btr[nt_] + (ks_) * (32 * 512);                                               \
      dst_ = lds_read_frag_tr(_p, _p + 4 * 512);                                                          \
    }                                                                                                     \
  } while (0)

  f32x4 acc[MT][W_NT];

  // One phase: the MFMAs of HB row blocks (x fragments ux_) against all eight column blocks (weight
  // fragments uw_).  In their shadow, spread over its first three quarters, the LDS reads for the
  // next phase: HB x fragments of k-step xks_, row half xh_ and, rd_w_, the eight weight fragments of
  // k-step wks_; and, spread evenly, cnt_ DMA instructions (dma_(p_, r_): part p_ of the r_-th).  sched_barrier pins
  // the order: with one wave per SIMD nothing else hides the issue of LDS and DMA instructions, and an MFMA's shadow hides
  // three instructions, so that a request's parts go into three of them.
#define W_PHASE(z_, h_, ux_, uw_, rd_, xslot_, xks_, xh_, lx_, rd_w_, wks_, lw_, cnt_, dma_, end_)            \
  do {                                                                                                    \
    _Pragma("unroll") for (int _i = 0; _i < 8 * HB; ++_i) {                                               \
      if (z_) mma_first<FORM == FORM_NN>(acc[HB * (h_) + (_i >> 3)][_i & 7], uw_[_i & 7], ux_[_i >> 3]);                   \
      else mma<FORM == FORM_NN>(acc[HB * (h_) + (_i >> 3)][_i & 7], uw_[_i & 7], ux_[_i >> 3]);                            \
      __builtin_amdgcn_sched_barrier(0);                                                                  \
      constexpr int _nr = HB + ((rd_w_) ? 8 : 0), _at = 8 * HB * 3 / 4;                                   \
      if (rd_) {                                                                                          \
        _Pragma("unroll") for (int _r = 0; _r < _nr; ++_r)                                                \
          if (_r * _at / _nr == _i) {                                                                     \
            if ((rd_w_) && _r < 8) W_NEXT_W(xslot_, wks_, _r & 7, lw_[_r & 7]);                           \
            else W_NEXT_X(xks_, HB * (xh_) + (_r - ((rd_w_) ? 8 : 0)) % HB, lx_[(_r - ((rd_w_) ? 8 : 0)) % HB]); \
          }                                                                                               \
      }                                                                                                   \
      _Pragma("unroll") for (int _r = 0; _r < (cnt_); ++_r)                                               \
        _Pragma("unroll") for (int _p = 0; _p < 3; ++_p)                                                  \
          if ((2 * _r + 1) * 8 * HB / (2 * ((cnt_) > 0 ? (cnt_) : 1)) - 1 + _p == _i) dma_(_p, _r);       \
      if (_i == 8 * HB - 2) { end_; }                                                                     \
      __builtin_amdgcn_sched_barrier(0);                                                                  \
    }                                                                                                     \
  } while (0)

  // One k-tile kt_ (slot kt_ & 1) in four phases: (row half, k-step) = (0, 0), (0, 1), (1, 0), (1, 1).
  // After phase 0 every weight fragment and the first half's x fragments are in registers: the waves
  // meet, and that part of tile kt + 2 goes into this slot over phases 1 to 3; after phase 2 the rest
  // is, and follows in the next tile's phase 0.  So the requests are spread evenly over the k-tile
  // (64 KB per tile and compute unit are close to what L2 and the fabric deliver on average: measured
  // on zero operands, where power sets no limit, 1.17 us per k-tile with the requests bunched into two
  // phases, 0.91 without any) and each has three phases or more to arrive.  At each meeting everything
  // but the youngest requests has arrived (x1_, f2_: the part of tile kt + 1 / kt + 2 is requested in
  // this tile, 1 whole, 2 perhaps partial; st_: the stores of the item before are younger than tile 1).
#define W_X1(p_, r_, k_) do { if ((k_) == 1) W_PART_A(p_, _nto, HB + (r_)); else if ((p_) == 1) W_DMA_A(_slot ^ 1, HB + (r_), _l1); } while (0)
#define W_FQ(p_, q_, k_) do { if ((k_) == 1) W_PART_FIRST(p_, _to, q_); else if ((p_) == 1) W_DMA_FIRST(_slot, q_, _l2); } while (0)
#define W_X1_1(p_, r_) W_X1(p_, r_, 1)
#define W_X1_2(p_, r_) W_X1(p_, r_, 2)
#define W_F1_1(p_, r_) W_FQ(p_, r_, 1)
#define W_F1_2(p_, r_) W_FQ(p_, r_, 2)
#define W_F2_1(p_, r_) W_FQ(p_, C1 + (r_), 1)
#define W_F2_2(p_, r_) W_FQ(p_, C1 + (r_), 2)
#define W_F3_1(p_, r_) W_FQ(p_, C1 + C2 + (r_), 1)
#define W_F3_2(p_, r_) W_FQ(p_, C1 + C2 + (r_), 2)
#define W_X1_0 W_X1_1
#define W_F1_0 W_F1_1
#define W_F2_0 W_F2_1
#define W_F3_0 W_F3_1
#define W_TILE(kt_, x1_, f2_, st_)                                                                        \
  do {                                                                                                    \
    const int _slot = (kt_) & 1, _to = _slot * SLOT, _nto = SLOT - _to;                                   \
    const int _l1 = (x1_) == 2 ? W_KLEN((kt_) + 1) : 0, _l2 = (f2_) == 2 ? W_KLEN((kt_) + 2) : 0;         \
    W_PHASE((st_) > 0, 0, xa0, wb0, 1, _slot, 1, 0, xa1, 1, 1, wb1, (x1_) ? HB : 0, W_X1_##x1_, );                   \
    if (x1_) wide_meet<8 + 2 * HB + (st_), 0>();                                                          \
    else if (lt_cnt > 0) wide_meet<8 + MT, 0>();                                                          \
    else wide_meet<0, 0>();                                                                               \
    W_PHASE(0, 0, xa1, wb1, 1, _slot, 0, 1, xa0, 0, 0, wb0, (f2_) ? C1 : 0, W_F1_##f2_, W_TOGGLE(w_at[1]));  \
    W_PHASE((st_) > 0, 1, xa0, wb0, 1, _slot, 1, 1, xa1, 0, 0, wb0, (f2_) ? C2 : 0, W_F2_##f2_, W_TOGGLE(x_at[0]); W_TOGGLE(w_at[0])); \
    if (x1_) wide_meet<HB + ((f2_) ? C1 + C2 : 0) + (st_), 0>();                                          \
    W_PHASE(0, 1, xa1, wb1, x1_, _slot ^ 1, 0, 0, xa0, 1, 0, wb0, (f2_) ? C3 : 0, W_F3_##f2_, W_TOGGLE(x_at[1])); \
  } while (0)

  // One extra contraction tile of the LoRA expand (entry i_ of the row tile's list) into slot slot_:
  // the x side from the two-term bf16 split of u (rows outside the segment fetch zeros), the weight
  // side from the adapter's factor (both halves of the contraction read the same ranks).
#define W_LORA_DMA(i_, slot_)                                                                             \
  do { const int _ln = fresh(lane);                                                                                                    \
    const LoraTile _e = ((const LoraTile*)lt_s)[(i_) + 1];                                                \
    const int _rp = (_e.rank + 15) & ~15, _kext = 2 * _rp;                                                \
    const bf16_t* _L = (const bf16_t*)(uintptr_t)_e.L;                                                    \
    _Pragma("unroll") for (int _j = 0; _j < MT; ++_j) {                                                   \
      const int _row = (wave * MT + _j) * 8 + (_ln >> 3);                                                \
      const int _kk = _e.kc + (((_ln & 7) ^ ((_row >> 1) & 7)) << 3);                                    \
      const int64_t _m = m0 + _row;                                                                       \
      const bf16_t* _src = a.zero_line;                                                                   \
      if (_m >= _e.lo && _m < _e.hi && _kk < _kext) _src = a.U2 + _m * (2 * a.r_stride) + _kk;            \
      __builtin_amdgcn_global_load_lds((gptr_t)_src, (lptr_t)(smem + (slot_) * SLOT + a_dma + _j * 1024), 16, 0, 0); \
      __builtin_amdgcn_sched_barrier(0); \
    }                                                                                                     \
    _Pragma("unroll") for (int _j = 0; _j < 8; ++_j) {                                                    \
      const bf16_t* _src = a.zero_line;                                                                   \
      if (LFORM == FORM_NT) {          /* L_t[n * r + q]: row-k tile */                                   \
        const int _row = (wave * 8 + _j) * 8 + (_ln >> 3);                                               \
        const int _kk = _e.kc + (((_ln & 7) ^ ((_row >> 1) & 7)) << 3);                                  \
        const int _q = _kk >= _rp ? _kk - _rp : _kk;                                                      \
        const int64_t _n = n0 + _row;                                                                     \
        if (_kk < _kext && _q < _e.rank && _n < a.Nout) _src = _L + _n * _e.rank + _q;                    \
      } else {                         /* L_t[q * Nout + n]: k-n tile */                                  \
        const int _k = (wave * 8 + _j) * 2 + (_ln >> 5);                                                 \
        const int _kk = _e.kc + _k;                                                                       \
        const int _q = _kk >= _rp ? _kk - _rp : _kk;                                                      \
        const int64_t _n = n0 + (((_ln & 31) ^ kn_swz(_k)) << 3);                                        \
        if (_kk < _kext && _q < _e.rank && _n < a.Nout) _src = _L + (int64_t)_q * a.Nout + _n;            \
      }                                                                                                   \
      __builtin_amdgcn_global_load_lds((gptr_t)_src, (lptr_t)(smem + (slot_) * SLOT + b_dma + _j * 1024), 16, 0, 0); \
      __builtin_amdgcn_sched_barrier(0); \
    }                                                                                                     \
  } while (0)
  // One 32-wide contraction step out of slot_ for the wave's row blocks that have rows in [lo_, hi_).
#define W_LORA_MMA(slot_, ks_, lo_, hi_)                                                                  \
  do {                                                                                                    \
    bf16x8 _wf[W_NT], _xf[MT];                                                                            \
    _Pragma("unroll") for (int _n = 0; _n < W_NT; ++_n) W_READ_W(LFORM, slot_, ks_, _n, _wf[_n]);         \
    _Pragma("unroll") for (int _mt = 0; _mt < MT; ++_mt) W_READ_X(slot_, ks_, _mt, _xf[_mt]);             \
    _Pragma("unroll") for (int _mt = 0; _mt < MT; ++_mt) {                                                \
      const int64_t _r0 = m0 + wm * (16 * MT) + _mt * 16;                                                 \
      if (_r0 + 16 > (lo_) && _r0 < (hi_)) {                                                              \
        _Pragma("unroll") for (int _n = 0; _n < W_NT; ++_n) mma<LFORM == FORM_NN>(acc[_mt][_n], _wf[_n], _xf[_mt]);         \
        shared_rows |= __builtin_amdgcn_readfirstlane(_r0 < (lo_) || _r0 + 16 > (hi_)) << _mt;            \
      }                                                                                                   \
    }                                                                                                     \
  } while (0)

  W_ITEM(0);
  W_TOKENS(0);
  wide_meet<0, 0>();
  W_SETUP(0);
  W_REQUEST(0);
  bool stores = false;               // the previous item's NST stores are younger than this item's first requests

  for (int item = 0; item < n_items; ++item) {
    // (a tile behind stores starts its sums with its first products)
    if (!stores || nfast <= 2) {
      bf16x8 z = {};
      asm volatile("" : "+v"(z));
#pragma unroll
      for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < W_NT; ++j) mma_first<true>(acc[i][j], z, z);
    }
    // the first part of k-tile 0 (and everything older) has landed
    if (ntile > 1) {
      if (stores) wide_meet<8 + 2 * HB + NST, 0>(); else wide_meet<8 + 2 * HB, 0>();
    } else {
      wide_meet<0, 0>();
    }
    int shared_rows = 0;             // row blocks of this wave that hold rows of several adapters
    int lt_cnt = 0;
    if (a.lora == WIDE_LORA_LISTS && split == 0) lt_cnt = __builtin_amdgcn_readfirstlane(((const LoraTile*)lt_s)->lo);
    int lslot = 0;                   // slot of the first extra contraction tile
    {
      bf16x8 xa0[HB], xa1[HB], wb0[W_NT], wb1[W_NT];
      {
        const int _ln = fresh(lane), _row = _ln & 15, _g = (_ln >> 4) ^ ((_row >> 1) & 7);
        x_at[0] = lds0 + (wm * (MT * 16) + _row) * 128 + (_g << 4);
        w_at[0] = lds0 + A_BYTES + (wn * 128 + _row) * 128 + (_g << 4);
        x_at[1] = x_at[0] ^ 64; w_at[1] = w_at[0] ^ 64;      // (k-step 1: unit ^ 4)
      }
#pragma unroll
      for (int i = 0; i < HB; ++i) W_READ_X(0, 0, i, xa0[i]);
#pragma unroll
      for (int i = 0; i < W_NT; ++i) W_READ_W(FORM, 0, 0, i, wb0[i]);
      int kt = 0;
      if (stores && kt + 2 < nfast) { W_TILE(kt, 1, 1, NST); ++kt; }
      for (; kt + 2 < nfast; ++kt) W_TILE(kt, 1, 1, 0);
      if (kt + 2 < ntile) { W_TILE(kt, 2, 2, 0); ++kt; }
      if (kt + 1 < ntile) { W_TILE(kt, 2, 0, 0); ++kt; }
      if (lt_cnt > 0) {
        // the slot the last k-tile does not use is free
        lslot = (kt + 1) & 1;
        W_LORA_DMA(0, lslot);
      }
      W_TILE(kt, 0, 0, 0);
    }
    // ---- LoRA expand by DMA: extra contraction tiles, tile i + 1 in flight while tile i is multiplied
    for (int i = 0; i < lt_cnt; ++i) {
      wide_meet<0, 0>();             // tile i has landed everywhere, nobody still reads tile i - 1
      const int s = (lslot + i) & 1;
      if (i + 1 < lt_cnt) W_LORA_DMA(i + 1, s ^ 1);
      const LoraTile e = ((const LoraTile*)lt_s)[i + 1];
      const int lo = __builtin_amdgcn_readfirstlane(e.lo), hi = __builtin_amdgcn_readfirstlane(e.hi);
      const int left = 2 * ((__builtin_amdgcn_readfirstlane(e.rank) + 15) & ~15) - __builtin_amdgcn_readfirstlane(e.kc);
      W_LORA_MMA(s, 0, lo, hi);
      if (left >= WK) W_LORA_MMA(s, 1, lo, hi);      // (2 r_pad is a multiple of 32)
    }
    wide_meet<0, 0>();               // nobody reads the slots any more
    // ---- LoRA expand staged through registers: ranks that are no multiples of 8, or no split of u
    // (also a row tile with more extra contraction tiles than a list holds)
    if (split == 0 && (a.lora == WIDE_LORA_STAGED || lt_cnt < 0)) {
      char* La = smem;
      char* Lb = smem + A_BYTES;
      const int lc = tid & 7, lr = tid >> 3;         // 16-byte unit along k, row (32 per pass) of row-k tiles
      const int ncu = tid & 31, nkr = tid >> 5;      // 16-byte unit along n, k-row (8 per pass) of k-n tiles
      const int64_t T_lora = a.seg_off[a.n_adapters];
      const int64_t m_end = (m0 + ROWS) < T_lora ? (m0 + ROWS) : T_lora;
      int t = m0 < m_end ? segment_of(a.seg_off, a.n_adapters, (int)m0) : a.n_adapters;
      for (; t < a.n_adapters && (int64_t)a.seg_off[t] < m_end; ++t) {
        const int64_t lo = a.seg_off[t] > m0 ? (int64_t)a.seg_off[t] : m0;
        const int64_t hi = (int64_t)a.seg_off[t + 1] < m_end ? (int64_t)a.seg_off[t + 1] : m_end;
        if (hi <= lo) continue;
        const AdapterEntry e = a.table[t];
        const bf16_t* L = (const bf16_t*)(a.which ? e.B : e.A);
        const int r = e.rank, r_pad = (r + 15) & ~15, kext = 2 * r_pad;
        for (int kc = 0; kc < kext; kc += WK) {
          const int kk0 = kc + lc * 8;
          const bool second = kk0 >= r_pad;
          const int q0 = kk0 - (second ? r_pad : 0);
#pragma unroll 2
          for (int i = 0; i < MT; ++i) {             // u of the rows of this segment, zeros elsewhere, as [u_hi | u_lo]
            const int64_t m = m0 + lr + 32 * i;
            float4 f0 = make_float4(0.f, 0.f, 0.f, 0.f), f1 = f0;
            if (kk0 < kext && m >= lo && m < hi) {
              const float4* up = (const float4*)(a.U + m * a.r_stride + q0);
              f0 = up[0]; f1 = up[1];
            }
            const float f[8] = {f0.x, f0.y, f0.z, f0.w, f1.x, f1.y, f1.z, f1.w};
            bf16_t o[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              const bf16_t h = float_to_bf16_bits(f[j]);
              o[j] = second ? float_to_bf16_bits(f[j] - bf16_bits_to_float(h)) : h;
            }
            *(uint4*)(La + swz_rowk(lr + 32 * i, lc)) = pack8(o);
          }
#pragma unroll 2
          for (int i = 0; i < 8; ++i) {              // L_t stacked twice along the contraction
            uint4 w = make_uint4(0, 0, 0, 0);
            if (LFORM == FORM_NT) {
              const int64_t n = n0 + lr + 32 * i;
              if (kk0 < kext && n < a.Nout && q0 < r) {
                const bf16_t* lp = L + n * r + q0;
                if ((r & 7) == 0) {
                  w = *(const uint4*)lp;
                } else {
                  bf16_t o[8];
                  for (int j = 0; j < 8; ++j) o[j] = (q0 + j < r) ? lp[j] : (bf16_t)0;
                  w = pack8(o);
                }
              }
              *(uint4*)(Lb + swz_rowk(lr + 32 * i, lc)) = w;
            } else {
              const int kk = kc + nkr + 8 * i;
              const int q = kk - (kk >= r_pad ? r_pad : 0);
              if (kk < kext && q < r && (n0 + ncu * 8) < a.Nout) w = *(const uint4*)(L + (int64_t)q * a.Nout + n0 + ncu * 8);
              *(uint4*)(Lb + swz_kn(nkr + 8 * i, ncu)) = w;
            }
          }
          __syncthreads();
          W_LORA_MMA(0, 0, lo, hi);
          if (kext - kc >= WK) W_LORA_MMA(0, 1, lo, hi);
          __syncthreads();
        }
      }
    }
    // In a block of rows of several adapters the others' u is 0, and 0 times a factor that is infinite or
    // not a number is not 0: such sums are computed again behind the stores.  (The test reads the shared
    // blocks' accumulators; 40960 rows of 32 adapters, 4096 x 14336: 3.58 ms without it, 3.56 with.)
    bool again = false;
    acc_settle();
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
      if (shared_rows >> mt & 1) {
        float z = 0.f;
#pragma unroll
        for (int nt = 0; nt < W_NT; ++nt) {
          const f32x4 c = acc_read(acc[mt][nt]);
          z = fmaf(c[0], 0.f, fmaf(c[1], 0.f, fmaf(c[2], 0.f, fmaf(c[3], 0.f, z))));
        }
        again |= z != 0.f;
      }
    again = __ballot(again) != 0;
    // ---- the next item's first requests, then this item's results
    const int64_t em0 = m0, en0 = n0;
    const int eptile = ptile, esplit = split;
    if (item + 1 < n_items) {
      W_ITEM(item + 1);
      W_SETUP(item + 1);
      W_REQUEST(item + 1);
    }
    asm volatile("" ::: "memory");   // (the stores stay behind the requests: wide_meet counts them)
    const int el = fresh(lane), erow = el & 15, eg = el >> 4;
    stores = eptile < 0 && em0 + ROWS <= a.T && en0 + WN <= a.Nout;
    if (eptile >= 0) {
      // a piece of a split tile: sums in accumulator order, [split][tile][wave][row block][column block][lane] x 4
      f32x4* part = (f32x4*)a.partials + ((int64_t)(esplit * a.tail_tiles + eptile) * 4 + wave) * (MT * W_NT * 64) + el;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < W_NT; ++nt) part[(mt * W_NT + nt) * 64] = acc[mt][nt];
    } else if (!OUT_F32 && stores) {
      // a whole tile
      const int32_t* tok = tok3 + (item % 3) * ROWS + wm * (16 * MT) + erow;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        bf16_t* o = (bf16_t*)a.out + (int64_t)tok[mt * 16] * a.ldo + en0 + wn * 128 + (eg & 1) * 16 + (eg >> 1) * 8;
#pragma unroll
        for (int np = 0; np < W_NT / 2; ++np) {
          __builtin_amdgcn_sched_barrier(0);
          store_out(o + np * 32, pair_rows(acc_read(acc[mt][2 * np]), acc_read(acc[mt][2 * np + 1])));
        }
      }
    } else {
      const int32_t* tok = tok3 + (item % 3) * ROWS + wm * (16 * MT) + erow;
      const int64_t mrow = em0 + wm * (16 * MT) + erow;
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) {
        const bool row_ok = mrow + mt * 16 < a.T;
        const int64_t base = (int64_t)tok[mt * 16] * a.ldo;
        if (OUT_F32) {
          const int64_t col = en0 + wn * 128 + 4 * eg;
          float* o = (float*)a.out + base + col;
#pragma unroll
          for (int nt = 0; nt < W_NT; ++nt)
            if (row_ok && col + nt * 16 < a.Nout) store_out(o + nt * 16, acc[mt][nt]);
        } else {
          const int64_t col = en0 + wn * 128 + (eg & 1) * 16 + (eg >> 1) * 8;
          bf16_t* o = (bf16_t*)a.out + base + col;
#pragma unroll
          for (int np = 0; np < W_NT / 2; ++np) {
            __builtin_amdgcn_sched_barrier(0);
            const uint4 v = pair_rows(acc_read(acc[mt][2 * np]), acc_read(acc[mt][2 * np + 1]));
            if (row_ok && col + np * 32 < a.Nout) store_out(o + np * 32, v);
          }
        }
      }
    }
    asm volatile("" ::: "memory");
    if (again) {
      // (a broken adapter) the wave's row blocks of several adapters in plain fp32, a row's own adapter only
      const int64_t k0 = eptile >= 0 ? esplit * a.tail_kchunk : 0, k1 = eptile >= 0 && esplit + 1 < a.tail_split ? k0 + a.tail_kchunk : a.Kc;
      wide_drain();                  // (the stores above)
#pragma unroll 1
      for (int mt = 0; mt < MT; ++mt) {
        const int row = wm * (16 * MT) + mt * 16 + erow;
        const int64_t m = em0 + row;
        if (!(shared_rows >> mt & 1) || m >= a.T) continue;
        const int64_t tok = tok3[(item % 3) * ROWS + row];
        const int t = m < a.seg_off[a.n_adapters] ? segment_of(a.seg_off, a.n_adapters, (int)m) : -1;
#pragma unroll 1
        for (int c = 0; c < W_NT * 4; ++c) {
          const int64_t n = en0 + wn * 128 + (c >> 2) * 16 + 4 * eg + (c & 3);
          if (n >= a.Nout) continue;
          float sum = 0.f;
          for (int64_t k = k0; k < k1; k += 8) {       // (contraction lengths are multiples of 8)
            union { uint4 u; bf16_t h[8]; } x, w;
            x.u = *(const uint4*)(a.A + tok * a.lda + k);
            if (FORM == FORM_NT) w.u = *(const uint4*)(a.B + n * a.ldb + k);
            else for (int i = 0; i < 8; ++i) w.h[i] = a.B[(k + i) * a.ldb + n];
#pragma unroll
            for (int i = 0; i < 8; ++i) sum = fmaf(bf16_bits_to_float(x.h[i]), bf16_bits_to_float(w.h[i]), sum);
          }
          if (t >= 0 && esplit == 0) {
            const AdapterEntry e = a.table[t];
            const bf16_t* L = (const bf16_t*)(a.which ? e.B : e.A);
            for (int q = 0; q < e.rank; ++q)
              sum = fmaf(a.U[m * a.r_stride + q], bf16_bits_to_float(LFORM == FORM_NT ? L[n * e.rank + q] : L[(int64_t)q * a.Nout + n]), sum);
          }
          if (eptile >= 0) a.partials[((((int64_t)(esplit * a.tail_tiles + eptile) * 4 + wave) * MT + mt) * W_NT + (c >> 2)) * 256 + el * 4 + (c & 3)] = sum;
          else if (OUT_F32) ((float*)a.out)[tok * a.ldo + n] = sum;
          else ((bf16_t*)a.out)[tok * a.ldo + n] = float_to_bf16_bits(sum);
        }
      }
      wide_drain();
    }
  }
}

// The split tiles' results: their pieces' sums added in split order, rounded, rows scattered.  Block =
// one row block of one wave's part of a tile (16 rows x 128 columns); bound by reading the sums once.
template <bool OUT_F32>
__global__ __launch_bounds__(W_THREADS) void wide_finish_kernel(WideArgs a, int mt_all) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, frow = lane & 15, fg = lane >> 4;
  const int mt = blockIdx.x % mt_all, rest = blockIdx.x / mt_all;
  const int part = rest & 3, ptile = rest >> 2;            // wave part (2 x 2) of the tile
  int tm;
  const int tn = wide_tile(a.rounds * 256 + ptile, mt_all, a.tiles_m, a.tiles_n, &tm);
  const int64_t m = (int64_t)tm * (32 * mt_all) + (part >> 1) * (16 * mt_all) + mt * 16 + frow;
  const int64_t n0 = (int64_t)tn * WN + (part & 1) * 128 + wave * 32;   // this wave's two column blocks
  const int64_t stride = (int64_t)a.tail_tiles * 4 * mt_all * (W_NT * 64);
  const f32x4* p = (const f32x4*)a.partials + (((int64_t)ptile * 4 + part) * mt_all + mt) * (W_NT * 64) + wave * 128 + lane;
  f32x4 s0 = p[0], s1 = p[64];
  for (int k = 1; k < a.tail_split; ++k) {
    const f32x4 q0 = p[k * stride], q1 = p[k * stride + 64];
    s0[0] += q0[0]; s0[1] += q0[1]; s0[2] += q0[2]; s0[3] += q0[3];
    s1[0] += q1[0]; s1[1] += q1[1]; s1[2] += q1[2]; s1[3] += q1[3];
  }
  const bool row_ok = m < a.T;
  const int64_t tok = !row_ok ? 0 : a.perm ? a.perm[m] : m;
  if (OUT_F32) {
    float* o = (float*)a.out + tok * a.ldo + n0 + 4 * fg;
    if (row_ok && n0 + 4 * fg < a.Nout) store_out(o, s0);
    if (row_ok && n0 + 4 * fg + 16 < a.Nout) store_out(o + 16, s1);
  } else {
    const int64_t col = n0 + (fg & 1) * 16 + (fg >> 1) * 8;
    const uint4 v = pair_rows(s0, s1);
    if (row_ok && col < a.Nout) store_out((bf16_t*)a.out + tok * a.ldo + col, v);
  }
}

// ---------------------------------------------------------------------------------------------
// Plan: the tile height and the split of the last round.  256 workgroups take the tiles in rounds;
// tiles that do not fill the last round are cut along the contraction into as many pieces as keep
// every compute unit busy, where the pieces' sums (written and read once, plus a launch) cost less
// than the time the shorter pieces save.  Rates fitted to a sweep of heights and splits at
// 512 .. 5000 rows and 4096 .. 14336 columns and contraction values: a k-tile takes longer the more
// compute units are busy (they share the fabric and the power budget), e.g. 4096 deep and 256 rows
// high: 66, 74, 81 and 96 us with 64, 128, 192 and 256 tiles in the round.
static double wide_ktile_us(int mt, int64_t busy) {
  const double b = busy < 256 ? (double)busy / 256 : 1.0;
  return mt == 8 ? 0.80 + 0.60 * b : mt == 6 ? 0.55 + 0.54 * b : 0.20 + 0.57 * b;
}
static constexpr double WIDE_ITEM_US = 6.0;                // store, first requests, expand: per tile

WidePlan wide_plan(int64_t T, int64_t Kc, int64_t Nout, size_t max_bytes) {
  WidePlan best;
  best.us = 1e30;
  const int64_t nk = (Kc + WK - 1) / WK;
  for (int mt = 8; mt >= 4; mt -= 2) {
    WidePlan p;
    p.mt = mt;
    const int64_t tm = (T + 32 * mt - 1) / (32 * mt), tn = (Nout + WN - 1) / WN;
    p.tiles_m = (int)tm; p.tiles_n = (int)tn;
    p.rounds = (int)(tm * tn / 256);
    p.tail_tiles = (int)(tm * tn - (int64_t)p.rounds * 256);
    const double whole = p.rounds * (nk * wide_ktile_us(mt, 256) + WIDE_ITEM_US);
    p.us = whole + (p.tail_tiles ? nk * wide_ktile_us(mt, p.tail_tiles) + WIDE_ITEM_US : 0.0);
    if (p.us < best.us) best = p;
    if (p.tail_tiles == 0) continue;
    for (int s = 2; s <= 256 / p.tail_tiles && s <= 32 && s * 4 <= nk; ++s) {
      WidePlan q = p;
      const int64_t chunk = (nk + s - 1) / s;
      q.tail_split = (int)((nk + chunk - 1) / chunk);
      q.tail_kchunk = chunk * WK;
      q.part_bytes = (size_t)q.tail_split * q.tail_tiles * (32 * mt) * WN * sizeof(float);
      if (q.part_bytes > max_bytes) continue;
      q.us = whole + chunk * wide_ktile_us(mt, q.tail_tiles * q.tail_split) + WIDE_ITEM_US + 5.0 + 2.0 * q.part_bytes / 15e6;
      if (q.us < best.us) best = q;
    }
  }
  return best;
}

size_t lora_tiles_bytes(int64_t T) {
  return T > 0 ? (size_t)((T + 127) / 128) * (LT_MAX + 1) * sizeof(LoraTile) : 0;
}

template <int MT, int FORM, bool OUT_F32, int LFORM>
static hipError_t launch_wide_mt(const WideArgs& a, hipStream_t stream) {
  static std::atomic<uint64_t> done{0};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = 1ull << (dev & 63);
  if (!(done.load(std::memory_order_acquire) & bit)) {
    e = hipFuncSetAttribute((const void*)gemm_wide_kernel<MT, FORM, OUT_F32, LFORM>, hipFuncAttributeMaxDynamicSharedMemorySize, wide_lds<MT>());
    if (e != hipSuccess) return e;
    done.fetch_or(bit, std::memory_order_release);
  }
  hipLaunchKernelGGL((gemm_wide_kernel<MT, FORM, OUT_F32, LFORM>), dim3(256), dim3(W_THREADS), wide_lds<MT>(), stream, a);
  return hipGetLastError();
}

hipError_t launch_gemm_wide(WideArgs a, const WidePlan& p, int form, int lform, int out_is_f32, hipStream_t stream) {
  a.tiles_m = p.tiles_m; a.tiles_n = p.tiles_n; a.rounds = p.rounds;
  a.tail_tiles = p.tail_tiles; a.tail_split = p.tail_split; a.tail_kchunk = p.tail_kchunk;
  hipError_t e;
#define W_PICK2(MT_, F_, L_) (out_is_f32 ? launch_wide_mt<MT_, F_, true, L_>(a, stream) : launch_wide_mt<MT_, F_, false, L_>(a, stream))
#define W_PICK(MT_) (form == FORM_NN ? W_PICK2(MT_, FORM_NN, FORM_NN) : lform == FORM_NN ? W_PICK2(MT_, FORM_NT, FORM_NN) : W_PICK2(MT_, FORM_NT, FORM_NT))
  e = p.mt == 8 ? W_PICK(8) : p.mt == 6 ? W_PICK(6) : W_PICK(4);
#undef W_PICK
#undef W_PICK2
  if (e != hipSuccess || p.tail_split <= 1) return e;
  const dim3 grid((unsigned)(p.tail_tiles * 4 * p.mt));
  if (out_is_f32) hipLaunchKernelGGL(wide_finish_kernel<true>, grid, dim3(W_THREADS), 0, stream, a, p.mt);
  else hipLaunchKernelGGL(wide_finish_kernel<false>, grid, dim3(W_THREADS), 0, stream, a, p.mt);
  return hipGetLastError();
}

}  // namespace marlaas
