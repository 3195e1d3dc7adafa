// Shared declarations of the HIP library (host + device side).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace marlaas {

typedef uint16_t bf16_t;  // raw bf16 bit pattern

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short short4v;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;

// One adapter as the kernels see it.  `lora_in` multiplies the layer input
// (A_t in forward, B_t in backward), `lora_out` produces the layer output
// (B_t in forward, A_t in backward); both are dense, orientation given by the
// kernel's template form.
struct AdapterEntry {
  const void* A;
  const void* B;
  int32_t rank;
  float scale;
};

struct GradEntry {
  float* dA;
  float* dB;
};

// Up to ROW_CHUNK consecutive rows of the grouped token order that belong to one adapter
// (t = -1: rows without an adapter).  The chunks of a segment map cover every row once.
static constexpr int ROW_CHUNK = 8;
struct RowChunk {
  int32_t row0, nrows, t, pad;
};

// Extended column e of the fused shrink: rank q of adapter entry t (e = rank offset of t + q), with
// that entry's factor pointers copied in, so that a kernel finds its source row with one load.
struct ExtCol {
  const void* A;
  const void* B;
  int32_t t, q;
  float scale;      // of entry t
  int32_t pad;
};

// One projection of a fused multi-projection forward (small batches): its weight, its output and
// where it sits in the concatenated column space (each projection padded to whole column tiles).
// The entries of a call travel inside the kernel arguments (no device copy).
struct ProjEntry {
  const void* W; int64_t ldw;     // weight operand, stored in the call's form
  int64_t Nout;                   // output columns of this projection
  void* out; int64_t ldo;
  int32_t tile0;                  // first column tile (128 wide) in the concatenated space
  int32_t fin0;                   // first column chunk (512 wide) of the finish kernel's grid
  int32_t tab0;                   // index of this projection's first adapter in the combined table
  int32_t pad;
};
static constexpr int MAX_PROJ = 8;

// Which extended columns the row tiles (128 rows) of a small batch carry.  Rows are grouped by adapter,
// so a row tile needs the factors of consecutive adapters only: columns base[tm][p] .. of projection p,
// laid out from column start[tm][p] of the tile on, count[tm] in all.  on = 0: every tile carries the
// call's columns 0 .. n_ext - 1, whatever the grouping.
static constexpr int EXT_ROW_TILES = 8;
struct ExtRows {
  int32_t on = 0;
  int32_t count[EXT_ROW_TILES] = {0};
  int32_t start[EXT_ROW_TILES][MAX_PROJ] = {{0}}, base[EXT_ROW_TILES][MAX_PROJ] = {{0}};
};

// The per-adapter tables of one call as the kernels read them, all in device memory.  They live
// either in an adapter table object (written when an adapter is registered or swapped) or in a
// slice of the caller's workspace (written at the start of the call); the passes only read them.
//   entries[i], grads[i] : i = projection * n_adapters + adapter
//   roff[i]              : sum of the ranks of entries 0 .. i - 1 (P + 1 values, P = entries)
//   cols[e]              : (factor pointers, entry, rank index) of extended column e, for e < min(roff[P], ext_cap)
struct DevTables {
  AdapterEntry* entries = nullptr;
  GradEntry* grads = nullptr;
  int32_t* roff = nullptr;
  ExtCol* cols = nullptr;
  int32_t ext_cap = 0;
};
// Bytes of one DevTables block for P entries and ext_cap extended columns, and its carving.
size_t dev_tables_bytes(int64_t P, int64_t ext_cap);
DevTables dev_tables_carve(void* base, int64_t P, int64_t ext_cap);
// Enqueue: entries[first .. first + count) = host values (by-value kernel arguments, no copy node).
hipError_t enqueue_write_entries(const DevTables& d, int64_t first, int64_t count, const AdapterEntry* host,
                                 hipStream_t stream);
hipError_t enqueue_write_grads(const DevTables& d, int64_t first, int64_t count, const GradEntry* host,
                               hipStream_t stream);
// Enqueue: roff and cols recomputed from entries[0 .. P) (after any change of a rank or a pointer).
hipError_t enqueue_derive(const DevTables& d, int64_t P, hipStream_t stream);

// How a [contraction, output] operand is stored.
//   FORM_NT: element (k, n) at ptr[n * ld + k]   (contraction index contiguous)
//   FORM_NN: element (k, n) at ptr[k * ld + n]   (output index contiguous)
enum { FORM_NT = 0, FORM_NN = 1 };

__device__ __forceinline__ float bf16_bits_to_float(bf16_t b) {
  return __uint_as_float(((uint32_t)b) << 16);
}
// round to nearest even (the hardware conversion of gfx950)
__device__ __forceinline__ bf16_t float_to_bf16_bits(float f) {
  const __bf16 h = (__bf16)f;
  return __builtin_bit_cast(bf16_t, h);
}
// two of them, the first one in the lower half: one instruction
__device__ __forceinline__ uint32_t pack2(float lo, float hi) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2{lo, hi}), bf16x2));
}

// A wave's 16 rows x 32 values, requested a row at a time (lane: row lane / 4, eight values lane % 4), as an operand of the
// matrix instructions (lane: row lane % 16, eight values lane / 16).  `stage`: 1 KB of LDS of this wave alone; a wave's LDS
// instructions are carried out in order, so the next call may follow at once.  What it is for: four neighbouring lanes in one
// line are one look-up of the unit's L1, and in operand order every lane is one: a kilobyte out of L2 keeps a unit busy for
// 27 ns, in rows for 8.3, in one piece for 7.0 (a prefill chunk's shrink, 2011 rows of 4096 values: 2.1 million look-ups, in rows 0.58).  The
// trip through LDS (0.1 us) goes into the chain of requests.
__device__ __forceinline__ uint4 rows_to_operand(char* stage, uint4 v, int lane) {
  const int li = lane & 15, lg = lane >> 4;
  *(uint4*)(stage + (lane >> 2) * 64 + (((lane & 3) ^ ((lane >> 3) & 3)) << 4)) = v;
  asm volatile("" ::: "memory");
  const uint4 o = *(const uint4*)(stage + li * 64 + ((lg ^ ((li >> 1) & 3)) << 4));
  asm volatile("" ::: "memory");
  return o;
}

// Segment t of the grouped token order is [seg_off[t], seg_off[t+1]).
// Largest t in [0, n] with seg_off[t] <= m (seg_off has n + 2 entries, last = T).
__device__ __forceinline__ int segment_of(const int32_t* __restrict__ seg_off, int n, int m) {
  int lo = 0, hi = n + 1;  // invariant: seg_off[lo] <= m < seg_off[hi]
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (seg_off[mid] <= m) lo = mid; else hi = mid;
  }
  return lo;
}

// The last index t of 0 .. n - 1 with le(t), for le true up to some index of 0 .. n - 1 and false behind it.
// All lanes of a wave call it: a ballot over 64 indices, and for n above 64 (up to 4096) one inside the piece found.
template <typename Le>
__device__ __forceinline__ int wave_last(int n, Le le) {
  const int lane = threadIdx.x & 63, step = (n + 63) >> 6;
  int t = (__popcll(__ballot(lane * step < n && le(lane * step))) - 1) * step;
  if (step > 1) t += __popcll(__ballot(lane < step && t + lane < n && le(t + lane))) - 1;
  return t;
}

// ---- launchers (implemented in the .hip files; all enqueue on `stream`) ----

struct SegmapDev {
  int32_t* perm;      // [T] or nullptr when the grouped order is the identity
  int32_t* seg_off;   // [n + 2]
};

// perm[m] = token of grouped row m, grp_ids[m] = its adapter (-1: none)
hipError_t launch_segmap(const int32_t* ids, int64_t T, int n, int32_t* perm, int32_t* grp_ids, int32_t* seg_off,
                         int32_t* block_hist, int32_t* flags, RowChunk* chunks, int32_t* order, int32_t* chunk_base,
                         hipStream_t stream);
// Token chunk of the weight-gradient reductions for batches whose segments are very unequal: a
// segment longer than this is cut into pieces of this many rows (twice the mean segment, at least
// 512, a multiple of 64), each piece a block of its own; chunk_base[t] (segment map) is the first
// partial-sum slot of adapter t's pieces, counting only adapters with more than one piece.
__host__ __device__ inline int reduce_ragged_chunk(int64_t T_lora, int n) {
  int64_t c = n > 0 ? 2 * T_lora / n : 0;
  if (c < 512) c = 512;
  return (int)((c + 63) / 64 * 64);
}
// Workgroups that such a cut takes per slab of columns: one for every slot, one for every adapter.  A chunk is at
// least twice the mean segment, so the slots are at most n / 2 whole chunks and n remainders: less than 3 n in all, and a
// grid's y holds 65535.
inline int reduce_ragged_rows(int n, int ragged_slots) { return ragged_slots + n; }
// The same in one launch (T <= 32768, n <= 800); host: pinned, receives seg_off[n + 2], the two
// flags and then `seq`, in this order (n + 5 values).
bool segmap_is_small(int64_t T, int n);
hipError_t launch_segmap_small(const int32_t* ids, int64_t T, int n, int32_t* perm, int32_t* grp_ids, int32_t* seg_off,
                               RowChunk* chunks, int32_t* order, int32_t* chunk_base, int32_t* host, int seq, hipStream_t stream);
int segmap_blocks(int64_t T);
// Row chunks of a grouped order with these segment offsets (n + 2 entries): how many there are.
int64_t segmap_chunk_count(const int32_t* seg_off, int n);
// Upper bound of that count for any map of T tokens and n adapters.
int64_t segmap_chunk_bound(int64_t T, int n);

// What a shrink's launch does besides, in workgroups behind its own: the row tiles' lists for the large-batch
// GEMM behind it, and the tables of a call that brings pointer lists of few adapters, which then travel in
// the kernel arguments (the shrink reads them there).  A launch of its own takes 5 us for either.
static constexpr int SIDE_INLINE = 16;
struct SideWork {
  int32_t* lists = nullptr; int list_rows = 0, list_tiles = 0;     // scratch (lora_tiles_bytes), rows of a tile, tiles
  int n_inl = 0;                                                   // entries below (0: none)
  AdapterEntry* entries_out = nullptr; GradEntry* grads_out = nullptr;   // where they go (grads_out may be null)
  AdapterEntry entry[SIDE_INLINE];
  GradEntry grad[SIDE_INLINE];
};

// u[m, 0..r_stride) = scale_t * sum_c X[perm[m], c] * L_t(c, q), grouped order m.
// which = 0 uses AdapterEntry::A as L_t, 1 uses ::B.  lora_form: FORM_NN when
// L_t is stored [C, r_t] (q contiguous), FORM_NT when stored [r_t, C].
hipError_t launch_shrink_bf16(const bf16_t* X, int64_t ldx, int64_t C, const int32_t* perm,
                              const int32_t* seg_off, int n_adapters, int max_seg,
                              const AdapterEntry* table, int which, int lora_form, float* u,
                              int r_stride, int64_t T_lora, float* partials, size_t partial_bytes,
                              bf16_t* u2, bool* wrote_u2, const bf16_t* zero_line, bool ranks_mult8, const SideWork& side, hipStream_t stream);
// scratch for the sums of a shrink whose contraction is split (0: it is not)
size_t shrink_partial_bytes(int64_t C, int64_t T_lora, int n_adapters, int r_stride);

// How the decode kernel's call gets finished (splits added, expand added, rows rounded and
// scattered), and what the ways other than the generic finish kernel need: the adapter of every
// grouped row; for the in-kernel way also zeroed device counters that stay zero between launches
// and the bounds of its one wait.
enum { DECODE_FINISH_GENERIC = 0,    // splitk_finish_kernel on fp32 rows (any split count)
       DECODE_FINISH_IN_KERNEL = 1,  // the decode kernel itself: one launch
       DECODE_FINISH_LAUNCH = 2,     // a second launch of the decode kernel's own finish
       DECODE_FINISH_AUTO = 3 };     // whichever of the two is faster for the split count
struct DecodeSync {
  int mode = DECODE_FINISH_GENERIC;  // the way asked for; the launcher falls back to the generic one
  int32_t* counters = nullptr;       // SYNC_INTS, all zero before the first launch; null: only kernels that exchange nothing
  const int32_t* grp_ids = nullptr;
  int spin_limit = 0;
  int cu_count = 0;
};
static constexpr int DECODE_SYNC_INTS = 4096;
static constexpr int THIN_ROWS = 32;                              // rows of the few-row kernel (gemm_thin.hip)
static constexpr int THIN_SPLITS = 4, THIN_U_FLOATS = MAX_PROJ * THIN_SPLITS * THIN_ROWS * 128;
// One launch for up to MID_ROWS rows (gemm_mid.hip): rows of a tile, columns of a tile / 32, contraction
// splits.  u travels in two areas ([projection][piece of the contraction][T][r_stride]) behind the few-row kernel's, the partial
// sums of at most MID_SPLIT_WGS workgroups behind those.
static constexpr int MID_ROWS = 1024, MID_SPLITS = 4, MID_SPLIT_WGS = 512;
static constexpr int MID_U_FLOATS = MAX_PROJ * 2 * MID_ROWS * 128;   // of u in one of its two areas: two pieces always fit
static constexpr int MID_TILE_FLOATS = 80 * 128, MID_PART_FLOATS = MID_SPLIT_WGS * MID_TILE_FLOATS;      // (of the largest tile whose contraction is split)
// Whose turn it is (agent_memory.h): lines of 32 ints; a line counts 2^TURN_SHIFT a launch, and a launch has fewer
// workgroups to a line than that.
static constexpr int TURN_LINES = 32, TURN_INTS = TURN_LINES * 32, TURN_SHIFT = 20;
// Column tiles of a projection, times splits: with all row tiles and projections, and a sixteenth as many producers, whose
// number is bounded by the rows, no more threads than the 2^32 of a launch.
static constexpr int64_t MID_WGS = (1ll << 32) / 512, MID_PRODUCERS = MID_WGS / 16;
static constexpr int MID_CONSUMERS = (int)((MID_WGS - MID_PRODUCERS) / (MAX_PROJ * (MID_ROWS / 64)));
// (16-rank tiles of adapters of rank 128: one a row, and again for every pair of row blocks)
static_assert((int64_t)MAX_PROJ * MID_SPLITS * 8 * (MID_ROWS + 3 * (MID_ROWS / 64)) <= MID_PRODUCERS && MID_WGS <= (int64_t)TURN_LINES << TURN_SHIFT, "");
static constexpr int SYNC_INTS = DECODE_SYNC_INTS + THIN_U_FLOATS + TURN_INTS + 2 * MID_U_FLOATS + MID_PART_FLOATS;
// Readings of a bounded wait, a round trip through the fabric each (1 to 1.5 us under load): what is waited for
// takes a tenth of it where its workgroups are on the chip, and doing without costs a few hundred microseconds.
static constexpr int MID_POLLS = 256;
// The adapters of a call as its plan takes them: how many (0: none), their ranks and 16-rank tiles in all (of a
// projection, the largest), the largest adapter's tiles, and the most that the adapters of T rows can have.
struct MidLora { int n = 0, ranks = 0, tiles = 0, tile_max = 0, tiles_max = 0, r_stride = 0; };
// The most shrink jobs of gemm_mid.hip (a projection's) that the adapters of T rows can have in tiles of 16 rb rows,
// however the rows are grouped: each adapter's 16-rank tiles once, and again for every pair of row blocks that
// begins inside an adapter's rows.
inline int mid_max_jobs(int64_t T, int rb, const MidLora& l) {
  const int64_t rows = 16 * rb, pairs = T / rows * ((rb + 1) / 2) + (T % rows + 31) / 32;
  return l.tiles_max + (int)(pairs - 1) * l.tile_max;
}
struct MidPlan { int rb = 0, wn = 2, ksplit = 1, tiles_m = 0; double us = 0.0; };     // rb = rows / 16; 0: none

// What lets the large-batch GEMM fetch the expand's operands by DMA: u (or v) as a two-term bf16
// split and the row tiles' lists of extra contraction tiles, both written by the shrink's launch
// (list_rows: rows of a tile, 0: no lists); zero_line: 16 zero bytes in device memory (always given).
struct LoraDma {
  const bf16_t* u2 = nullptr;
  const int32_t* tiles = nullptr; int list_rows = 0;
  const bf16_t* zero_line = nullptr;
};
size_t lora_tiles_bytes(int64_t T);
// Rows of the large-batch GEMM's tiles for a call that launch_gemm_bf16 gets with these sizes and no fused
// shrink; 0: another kernel runs.
int gemm_tile_rows(int64_t T, int64_t Kc, int64_t Nout, int need, bool packed, size_t partial_bytes, bool has_chunks);

struct GemmFuse {
  const ExtCol* cols;      // [n_ext] device
  const int32_t* roff;     // [n_adapters + 1] device: rank offsets
  int n_ext;               // sum of the ranks
  bool ranks_mult8;        // every rank is a multiple of 8
  float* u_out;            // [T][r_stride] device: receives scale_t * (X L_t) per grouped row
  // `cols` and `roff` may point into the tables of a larger adapter bank: ExtCol::t then counts
  // the bank's entries and t0 is the entry index of the call's table[0]; roff values are offsets
  // in the bank's extended-column space and ext_base is the call's first one (roff of table[0]).
  int t0 = 0, ext_base = 0;
  int need = 0;            // extended columns the fullest row tile carries (n_ext where `rows` is off)
  ExtRows rows;
};

// out[perm[m], :] = Aop[perm[m], :] * Bop + (m in segment t) U[m, :] * L_t
hipError_t launch_gemm_bf16(const bf16_t* Aop, int64_t lda, const bf16_t* Bop, int64_t ldb,
                            int form, int64_t T, int64_t Kc, int64_t Nout, const int32_t* perm,
                            const int32_t* seg_off, int n_adapters, const AdapterEntry* table,
                            int which, const float* U, int r_stride, void* out, int64_t ldo,
                            int out_is_f32, float* partials, size_t partial_bytes, const RowChunk* chunks,
                            int n_chunks, const GemmFuse* fuse, int need_unfused, bf16_t* wt_scratch, size_t wt_bytes, const bf16_t* Bt_kept, const LoraDma* dma,
                            const bf16_t* Bpacked, bool use_packed, const DecodeSync* sync, hipStream_t stream);
// (need_unfused: extended columns the row tiles would have needed, for the choice of kernel; use_packed: Bpacked may be read; Bpacked: optional packed copy of Bop for this contraction, used by small batches; with it the
// shrink is only fused when the adapters' factors are stored contraction-contiguous, which the
// caller says by passing fuse only then.)
// A call of few rows on packed weights (gemm_thin.hip): all of it, shrink included, in one launch.
// proj: the call's projections (W packed copies, ldw their k-steps), table: [projection][adapter], u
// (one projection; may be null): [T][r_stride] fp32, receives u; max_tiles: the most 16-rank tiles the adapters of T rows can
// have in any projection.
bool gemm_thin_ok(int form, int64_t T, bool lora, int r_stride, const DecodeSync* sync);
hipError_t launch_gemm_bf16_thin(const bf16_t* Aop, int64_t lda, int form, int64_t T, int64_t Kc, const int32_t* perm, int n_adapters,
                                 const AdapterEntry* table, int which, const ProjEntry* proj_host, int n_proj, int out_is_f32,
                                 float* u, int r_stride, int max_tiles, const DecodeSync* sync, hipStream_t stream);
// The same for more rows (gemm_mid.hip); the plan says whether it is the kernel for these sizes.  ext: ranks of
// all adapters in the batch (0: none); seg_off: rows of the adapters (device); proj_jobs: the most shrink jobs
// (16 ranks of an adapter x a pair of 16-row blocks of a row tile, 16 plan.rb rows) that any grouping of T rows
// has in any projection; room: bytes of partial sums that another kernel would have.
MidPlan gemm_mid_plan(int form, int64_t T, int64_t lda, int64_t Kc, const ProjEntry* proj_host, int n_proj, const MidLora& lora, int ext, size_t room,
                      const DecodeSync* sync);
hipError_t launch_gemm_bf16_mid(const bf16_t* Aop, int64_t lda, int form, int64_t T, int64_t Kc, const int32_t* perm, const int32_t* seg_off, int n_adapters,
                                const AdapterEntry* table, int which, const ProjEntry* proj_host, int n_proj, int out_is_f32,
                                float* u, int r_stride, const MidPlan& plan, int proj_jobs, const bf16_t* zero_line, const DecodeSync* sync,
                                hipStream_t stream);
// Several projections of the same input in one pass (small batches only: 128 x 128 tiles with
// the shrink carried as extended columns, or no adapters at all).  `proj_host` holds the n_proj
// entries (host memory); `table` is the combined adapter table ([projection][adapter]), `fuse` (null:
// no adapters) the combined extended-column tables, ExtCol::t indexing the combined table.  The
// projection entries travel in the kernel arguments.
// gemm_multi_ok tells whether the sizes qualify; otherwise the caller runs the projections one by one.
bool gemm_multi_ok(int form, int64_t T, int64_t Kc, const ProjEntry* proj_host, int n_proj, int need,
                   bool ranks_mult8, bool packed, size_t partial_bytes);
size_t gemm_multi_bytes(int64_t T, int64_t Kc, const ProjEntry* proj_host, int n_proj, int n_ext);
int gemm_multi_ext_room(const ProjEntry* proj_host, int n_proj);
hipError_t launch_gemm_bf16_multi(const bf16_t* Aop, int64_t lda, int form, int64_t T, int64_t Kc,
                                  const int32_t* perm, const int32_t* seg_off, int n_adapters,
                                  const AdapterEntry* table, const ProjEntry* proj_host,
                                  int n_proj, int out_is_f32, float* partials,
                                  size_t partial_bytes, const RowChunk* chunks, int n_chunks,
                                  const GemmFuse* fuse, int packed, const DecodeSync* sync, int r_stride,
                                  hipStream_t stream);
// Packed copy of a [contraction C, output O] operand for the decode kernel, in MFMA fragment order
// (16 output columns x 32 contraction values per kilobyte, zero beyond the matrix).  Element (c, o)
// of the source is at src[c * sc + o * so].
size_t packed_weight_bytes(int64_t C, int64_t O);
int64_t packed_weight_ksteps(int64_t C);
hipError_t launch_pack_weight(const bf16_t* src, int64_t sc, int64_t so, int64_t C, int64_t O, bf16_t* dst,
                              hipStream_t stream);
// Scratch for a transposed copy of the weight: a large batch whose weight is stored
// [contraction][output] runs faster on a [output][contraction] copy made per call (the copy
// costs two passes over the weight, the GEMM gains about a quarter).  0: not used for these sizes.
size_t gemm_wt_bytes(int form, int64_t T, int64_t Kc, int64_t Nout);
// dst[c][r] = src[r][c], bf16, R x C (both multiples of 8)
hipError_t launch_transpose_bf16(const bf16_t* src, int64_t lds, bf16_t* dst, int64_t ldd, int64_t R, int64_t C, hipStream_t stream);
// scratch for partial sums: what the fastest plan takes, and what a pass cannot run without; n_ext = sum of the
// adapter ranks (0: no adapters)
size_t gemm_splitk_bytes(int64_t T, int64_t Kc, int64_t Nout, int n_ext);
size_t gemm_splitk_min_bytes(int64_t T, int64_t Kc, int64_t Nout, int n_ext);
// Small batches: the GEMM can compute the shrink itself (as extra output columns over every
// adapter's factor; the finish kernel keeps each row's own adapter).  When this holds the caller
// skips the shrink launch and passes a GemmFuse; U is then ignored and u_out receives u.
// need: extended columns of the fullest row tile.
bool gemm_can_fuse_shrink(int form, int64_t T, int64_t Kc, int64_t Nout, int need, bool ranks_mult8, bool packed,
                          size_t partial_bytes);
// Extended columns that one row tile of these output columns can carry.
int gemm_ext_room(int64_t Nout);

// out_t(c, q) (+)= sum_{m in seg t} X[perm[m], c] * V[m, q]
// out_form FORM_NN: out_t[c * r_t + q]; FORM_NT: out_t[q * C + c].
// Optimizer step applied where a gradient element is completed (AdamW; see lora_small.hip):
// per adapter the fp32 master copy, the two moments and the bf16 output of the factor the
// reduction produces the gradient of.  on = 0: gradients are written as usual.
struct OptFactor { float* master; float* m; float* v; bf16_t* out; };
static constexpr int OPT_MAX_ADAPTERS = 8;
struct ReduceOpt {
  int on;
  float lr, beta1, beta2, eps, wd, inv_c1, inv_c2;   // inv_c: 1 / (1 - beta^step)
  OptFactor f[OPT_MAX_ADAPTERS];
};
// Both weight gradients of a backward; a job: X [T, C] and V [T, r_stride] of one of them.
struct ReduceJob {
  const bf16_t* X; int64_t ldx; int64_t C;
  const float* V;
  int which, form;          // 0: dA, 1: dB; storage of the gradient
  const ReduceOpt* opt;     // or null
};
hipError_t launch_reduce_bf16(const ReduceJob (&jobs)[2], const int32_t* perm, const int32_t* seg_off, int n_adapters, int64_t T_lora, int max_seg,
                              const AdapterEntry* table, const GradEntry* grads, int r_stride, int accumulate, float* partials, size_t partial_bytes,
                              const int32_t* order, const int32_t* chunk_base, int ragged_chunk, int ragged_slots, int ragged_adapters,
                              hipStream_t stream);
size_t reduce_partial_bytes(int64_t C, int n_adapters, int max_seg, int max_rank, bool always = false,
                            int ragged_chunk = 0, int ragged_slots = 0);

// fp32 path (fp32 matrix instructions, any shape).  The adapters of a call: device tables, or, for
// up to F32_INLINE adapters given as pointer lists, entries that travel in the kernel arguments
// (n_inl > 0), which saves the launch that writes them to device memory.
static constexpr int F32_INLINE = 16;
struct TablesF32 {
  const AdapterEntry* table; const GradEntry* grads;
  int n_inl;
  AdapterEntry entry[F32_INLINE];
  GradEntry grad[F32_INLINE];
};
// out[perm[m], :] = X[perm[m], :] * W + u(m) * L_t with u = scale_t X L'_t computed by the same
// launch (grp: adapter of every grouped row, null for none); u_out (nullable) receives u.  out = null: only u.
hipError_t launch_layer_f32(const float* X, int64_t ldx, const float* W, int64_t ldw, int form, int64_t T, int64_t Kc, int64_t Nout,
                            const int32_t* perm, const int32_t* grp, const TablesF32& tb, int which, float* u_out, int r_stride,
                            void* out, int64_t ldo, int out_is_f32, hipStream_t stream);
// One gradient: [C columns][ranks] (oform FORM_NN) or the other way round, of X's columns and the rows' V; which: dB (1) or dA.
struct ReduceF32Job { const float* X; int64_t ldx, C; const float* V; int which, oform; };
hipError_t launch_reduce_f32(const ReduceF32Job (&jobs)[2], const int32_t* perm, const int32_t* seg_off, int n_adapters, const TablesF32& tb,
                             int r_stride, int accumulate, hipStream_t stream);

}  // namespace marlaas
