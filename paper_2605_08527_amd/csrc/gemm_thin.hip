// Decode of few sequences (up to 32 rows) on the packed weight: the whole call in one launch.
//
//   out_p[tok(m), :] = x[tok(m), :] W_p  +  u_p(m) L_{t,p}        for every projection p of the call
//
// With few rows the weight is the traffic and the rest is latency: a 128-row tile (gemm_decode.hip)
// multiplies mostly padding, cuts the contraction over workgroups to occupy the chip and pays a second
// launch to add the pieces up (6 rows x 4096 x 4096: 17.9 + 6.9 us).  Here a workgroup owns all rows
// times 16 NC output columns and its eight waves split the contraction, so a weight fragment is read
// once, by the one wave that multiplies it, a wave requests 8 to 20 KB at a time (in two sets of registers, and what it waits
// for is all of both: requests stand behind branches, so nobody counts them), and the sums meet in LDS.  x comes straight from L2 (for the row counts of this kernel no more bytes than the weight), a row at
// a time where that pays (thin_rows).  Workgroups before the consumers ("producers") compute u: one per 16 ranks of an adapter
// that has rows, the same loop over the adapter's factor in place of the weight.  They are scheduled
// first and take little longer than a consumer's loop.  Every round trip through the fabric costs 1 to
// 1.5 us, so u carries its own flag: it travels through an area of the context that is all zero bits
// between launches, no value of u is stored as zero bits (+0 becomes -0), and a consumer reads its rows'
// u until nothing is zero bits any more.  The reading is bounded; a consumer that does not get a value in
// time computes u itself, in the same order of sums, so no workgroup depends on another one being scheduled
// and no bit on who was.  The workgroup that is last through with the area clears what was used of it.
#include "gemm_args.h"
#include "agent_memory.h"
#include "lora_expand.h"
#include "lora_shrink.h"

#include <atomic>

namespace marlaas {

static constexpr int TH_WAVES = 8, TH_THREADS = 64 * TH_WAVES;

// Registers are held to what lets two workgroups share a compute unit: with one each, a launch of one
// consumer per unit and a single producer took a second round of workgroups (1 row, 8 us against 15).
// R: 16-row blocks (T <= 16 R), NC: 16-column blocks per workgroup, ROWS: consumers request x a row at a time (rows_to_operand)
template <int R, int NC, bool ROWS>
__global__ __launch_bounds__(TH_THREADS, 4) void gemm_thin_kernel(GemmArgs a) {
  constexpr int U = R + NC <= 2 ? 4 : R + NC <= 3 ? 3 : R + NC <= 5 ? 2 : 1;   // k-steps requested together (twice: two sets of registers)
  constexpr int TILES = R * NC;
  extern __shared__ __attribute__((aligned(16))) char smem[];
  f32x4* red = (f32x4*)smem;                                    // [TH_WAVES][TILES][64]
  float* u_s = (float*)(smem + TH_WAVES * TILES * 1024);        // [16 R][r_stride + 4]: the rows' u
  const int us = a.r_stride + 4;
  const int oct_max = 2 * a.r_stride;                           // octets (8 ranks of one adapter) a 16-row block can have
  uint64_t* oct_L = (uint64_t*)(u_s + 16 * R * us);             // [R][oct_max]: address of the octet's ranks in row 0 of the factor
  uint32_t* oct_tq = (uint32_t*)(oct_L + R * oct_max);           // adapter << 8 | first rank
  int32_t* oct_r = (int32_t*)(oct_tq + R * oct_max);             // rank
  uint64_t* rL_s = (uint64_t*)(oct_r + R * oct_max);             // per row: expand factor,
  int32_t* tok_s = (int32_t*)(rL_s + 16 * R);                   // token (-1: past the end),
  int32_t* t_s = tok_s + 16 * R;                                // adapter (-1: none),
  int32_t* rank_s = t_s + 16 * R;                               // rank
  int32_t* cnt_s = rank_s + 16 * R;                             // [R] octets (-1: plain expand)
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lg = lane >> 4;
  const bool lora = a.n_adapters > 0 && a.table != nullptr;
  const int b = blockIdx.x;
  const bool producer = b < a.n_prod;
  // the projection of this workgroup, and its first column
  int p = 0;
  int64_t n0 = 0;
  if (producer) {
    p = b / (a.n_prod / a.n_proj);
  } else {
    const int c = b - a.n_prod;
    for (int q = 1; q < a.n_proj; ++q) if (c >= a.proj[q].tile0) p = q;
    n0 = (int64_t)(c - a.proj[p].tile0) * (16 * NC);
  }
  const int64_t Nout = a.proj[p].Nout, ldb = a.proj[p].ldw;
  const AdapterEntry* table = a.table + a.proj[p].tab0;
  // workgroups that are through with this projection's u, and its u: [split][T][r_stride], scaled; both
  // all zero bits between launches
  int32_t* done = a.sync + p;
  float* u_p = a.thin_u + p * (THIN_SPLITS * THIN_ROWS * 128);
  const int S = a.n_split, u_n = (int)a.T * a.r_stride;         // (u_n: floats of one split)
  const int prods = a.n_proj > 0 ? a.n_prod / a.n_proj : 0;
  const int everyone = prods + (p + 1 < a.n_proj ? a.proj[p + 1].tile0 : a.tiles_n) - a.proj[p].tile0;
  // (called by one whole wave whose requests are complete)
  auto leave = [&]() {
    int old = 0;
    if (lane == 0) old = __hip_atomic_fetch_add(done, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_amdgcn_readfirstlane(old) == everyone - 1) {
      for (int i = lane; i < S * (u_n >> 2); i += 64) store4_agent(u_p + i * 4, f32x4{0.f, 0.f, 0.f, 0.f});
      if (lane == 0) __hip_atomic_store(done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  };

  // this wave's part of the contraction, in 32-deep steps
  // (a producer's is cut over S workgroups first: its loads are row pieces from all over the factor, and
  // what it takes is their latency times the rounds of them)
  const int steps = (int)((a.Kc + 31) >> 5), per = (steps + TH_WAVES - 1) / TH_WAVES;
  const int s0 = wave * per, s1 = s0 + per < steps ? s0 + per : steps;

  const bool in_rows = ROWS && !producer;       // (producers do not: their chain is what u waits for)
  const int xr = in_rows ? lane >> 2 : li, xu = in_rows ? lane & 3 : lg;   // row, eight values that this lane requests
  // tokens of the rows this lane requests; adapter, and its entry, of row `lane`
  int32_t tokr[R];
#pragma unroll
  for (int i = 0; i < R; ++i) {
    const int64_t m = 16 * i + xr < a.T ? 16 * i + xr : a.T - 1;
    tokr[i] = a.perm ? a.perm[m] : (int32_t)m;
  }
  int g = -1, g_before = -1;
  if (lora && (producer || wave == 0) && lane < a.T && lane < 16 * R) {
    g = a.grp_ids[lane];
    if (lane > 0) g_before = a.grp_ids[lane - 1];
  }

#define TH_X(dst_, i_, ks_)                                                                               \
  do {                                                                                                    \
    const int64_t _k = (int64_t)(ks_) * 32 + 8 * xu;                                                      \
    dst_ = make_uint4(0, 0, 0, 0);                                                                        \
    if ((ks_) < s1 && _k < a.Kc) dst_ = *(const uint4*)(a.Aop + (int64_t)tokr[i_] * a.lda + _k);          \
  } while (0)
  union Frag { uint4 u; bf16x8 v; };

  if (producer) {
    AdapterEntry e;
    e.A = e.B = nullptr; e.rank = 0; e.scale = 0.f;
    if (g >= 0) e = table[g];
    // the 16-rank tiles of the adapters in row order: a lane per row, the first row of an adapter counts
    const int tiles = g >= 0 && g != g_before ? (e.rank + 15) >> 4 : 0;
    int inc = tiles;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) { const int v = __shfl_up(inc, d); if (lane >= d) inc += v; }
    const int j = (b - p * prods) / S;
    const uint64_t hit = __ballot(inc - tiles <= j && j < inc);
    if (hit == 0) {                                             // (the grid is sized for any grouping of T rows)
      if (wave == 0) leave();
      return;
    }
    const int row0 = __ffsll((unsigned long long)hit) - 1;
    const int t = __builtin_amdgcn_readlane(g, row0);
    const int q0 = (j - __builtin_amdgcn_readlane(inc - tiles, row0)) * 16;
    const int r = __builtin_amdgcn_readlane(e.rank, row0);
    const float scale = __shfl(e.scale, row0);
    const int row1 = row0 + __popcll(__ballot(g == t));         // rows [row0, row1) are this adapter's
    const uint64_t fp = (uint64_t)(uintptr_t)(a.which ? e.A : e.B);
    const bf16_t* L = (const bf16_t*)(((uint64_t)(uint32_t)__shfl((int)(fp >> 32), row0) << 32) | (uint32_t)__shfl((int)fp, row0));
    const int rb0 = row0 >> 4;
    int32_t tok0 = tokr[0];
#pragma unroll
    for (int i = 1; i < R; ++i) if (i == rb0) tok0 = tokr[i];
    const ShrinkJob job = {L, scale, r, q0, row0, row1, b % S};
    shrink_job<R == 1 ? 4 : 3, R>(job, a.Aop, a.lda, a.Kc, tok0, tokr[R - 1], S, red, [] {}, [&] { return u_p + b % S * u_n; }, a.r_stride, wave, lane);
    wait_vm<0>();                                                // (u is out)
    __syncthreads();
    if (wave == 0) leave();
    return;
  }

  // ---- consumers.  Column block c of this workgroup is block n0 / 16 + c of the packed weight
  // (blocks past the last one repeat it: those columns are never stored)
  char* const stage = smem + wave * (TILES * 1024);
  const bf16_t* wp[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) {
    const int64_t blocks = (Nout + 15) >> 4;
    int64_t nb = (n0 >> 4) + c;
    if (nb >= blocks) nb = blocks - 1;
    wp[c] = (const bf16_t*)a.proj[p].W + ((nb * ldb) << 9) + lane * 8;
  }
#define TH_LOAD(set_, s_)                                                                                 \
  do {                                                                                                    \
    _Pragma("unroll") for (int _u = 0; _u < U; ++_u) {                                                    \
      _Pragma("unroll") for (int _c = 0; _c < NC; ++_c) {                                                 \
        set_[_u][R + _c].u = make_uint4(0, 0, 0, 0);                                                      \
        if ((s_) + _u < s1) set_[_u][R + _c].u = *(const uint4*)(wp[_c] + (int64_t)((s_) + _u) * 512);    \
      }                                                                                                   \
      _Pragma("unroll") for (int _i = 0; _i < R; ++_i) TH_X(set_[_u][_i].u, _i, (s_) + _u);               \
    }                                                                                                     \
  } while (0)
#define TH_MMA(set_)                                                                                      \
  do {                                                                                                    \
    if (ROWS)                                                                                             \
      _Pragma("unroll") for (int _u = 0; _u < U; ++_u)                                                    \
        _Pragma("unroll") for (int _i = 0; _i < R; ++_i) set_[_u][_i].u = rows_to_operand(stage, set_[_u][_i].u, lane); \
    _Pragma("unroll") for (int _u = 0; _u < U; ++_u)                                                      \
      _Pragma("unroll") for (int _i = 0; _i < R; ++_i)                                                    \
        _Pragma("unroll") for (int _c = 0; _c < NC; ++_c)                                                 \
          acc[_i][_c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(set_[_u][R + _c].v, set_[_u][_i].v, acc[_i][_c], 0, 0, 0); \
  } while (0)
  f32x4 acc[R][NC];
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int c = 0; c < NC; ++c) acc[i][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  {
    Frag fa[U][R + NC], fb[U][R + NC];
    TH_LOAD(fa, s0);
    if (wave == 0) {
      // while those travel: the rows' tables, and per 16-row block the octets of its adapters (a lane
      // per row; the first row of an adapter in the block appends the adapter's octets)
      AdapterEntry e;
      e.A = e.B = nullptr; e.rank = 0; e.scale = 0.f;
      if (g >= 0) e = table[g];
      const bool first = g >= 0 && (g != g_before || li == 0);
      const int n_oct = first ? e.rank >> 3 : 0;
      int inc = n_oct, bad = g >= 0 && (e.rank & 7) ? 1 : 0;
#pragma unroll
      for (int d = 1; d < 16; d <<= 1) { const int v = __shfl_up(inc, d, 16), w = __shfl_up(bad, d, 16); if (li >= d) { inc += v; bad |= w; } }
      const uint64_t Lp = (uint64_t)(uintptr_t)(a.which ? e.B : e.A);
      if (lane < 16 * R) {
        tok_s[lane] = lane < a.T ? (a.perm ? a.perm[lane] : lane) : -1;
        t_s[lane] = g; rank_s[lane] = e.rank; rL_s[lane] = Lp;
        for (int q = 0, o = lg * oct_max + inc - n_oct; q < 8 * n_oct; q += 8, ++o) {
          oct_L[o] = Lp + (uint64_t)q * sizeof(bf16_t);
          oct_tq[o] = (uint32_t)g << 8 | q;
          oct_r[o] = e.rank;
        }
        if (li == 15) cnt_s[lg] = a.lform == FORM_NT && bad == 0 ? inc : -1;
      }
    }
    for (int s = s0; s < s1; s += 2 * U) {
      if (s + U < s1) TH_LOAD(fb, s + U);
      TH_MMA(fa);
      if (s + U < s1) {
        if (s + 2 * U < s1) TH_LOAD(fa, s + 2 * U);
        TH_MMA(fb);
      }
    }
  }
#pragma unroll
  for (int i = 0; i < R; ++i)
#pragma unroll
    for (int c = 0; c < NC; ++c) red[(wave * TILES + i * NC + c) * 64 + lane] = acc[i][c];
  __syncthreads();
  constexpr int MINE = (TILES + TH_WAVES - 1) / TH_WAVES;       // output tiles finished by a wave
  f32x4 y[MINE][1];
#pragma unroll
  for (int k = 0; k < MINE; ++k) {
    const int tile = wave + k * TH_WAVES;
    if (tile >= TILES) break;
    f32x4 s = red[tile * 64 + lane];
#pragma unroll
    for (int w = 1; w < TH_WAVES; ++w) {
      const f32x4 o = red[(w * TILES + tile) * 64 + lane];
      s[0] += o[0]; s[1] += o[1]; s[2] += o[2]; s[3] += o[3];
    }
    y[k][0] = s;
  }

  if (lora) {
    // the first octets' factor fragments depend on nothing that has to be waited for
    uint4 pre[MINE][1][1];
#pragma unroll
    for (int k = 0; k < MINE; ++k) {
      const int tile = wave + k * TH_WAVES, rb = tile / NC, c = tile - rb * NC;
      pre[k][0][0] = make_uint4(0, 0, 0, 0);
      if (tile < TILES && lg < cnt_s[rb]) {
        const int64_t n = n0 + c * 16 + li;
        const int o = rb * oct_max + lg;
        if (n < Nout) pre[k][0][0] = *(const uint4*)((const bf16_t*)(uintptr_t)oct_L[o] + n * oct_r[o]);
      }
    }
    for (int i = tid; i < 16 * R * (a.r_stride >> 2); i += TH_THREADS) {      // (whole waves)
      const int row = i / (a.r_stride >> 2), q = (i - row * (a.r_stride >> 2)) * 4;
      const int rank = t_s[row] >= 0 ? rank_s[row] : 0;
      f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
      bool ok = true;
      if (q < rank) ok = read_u(u_p + row * a.r_stride + q, u_n, S, a.spin_limit, v);
      if (__builtin_expect(__ballot(!ok) != 0, 0))               // (not reached in practice)
        u_again(table, a.which, a.Aop, a.lda, a.Kc, S, t_s, tok_s, row, q, !ok, lane, v);
#pragma unroll
      for (int j = 0; j < 4; ++j) if (q + j >= rank) v[j] = 0.f;
      *(f32x4*)(u_s + row * us + q) = v;
      if (a.u_out && b == a.n_prod && row < a.T && q < ((rank + 15) & ~15)) *(f32x4*)(a.u_out + (int64_t)row * a.r_stride + q) = v;
    }
    __syncthreads();
    if (wave == TH_WAVES - 1) leave();       // (it has few output tiles, or none)
#pragma unroll
    for (int k = 0; k < MINE; ++k) {
      const int tile = wave + k * TH_WAVES, rb = tile / NC, c = tile - rb * NC;
      if (tile >= TILES) break;
      const int row = rb * 16 + li, cnt = cnt_s[rb];
      if (cnt >= 0) {
        expand_octets(y[k], pre[k], cnt, lg, t_s[row],
                      [&](int q, bool mine, bf16x8& hi, bf16x8& lo) { split_u(u_s + row * us + q, mine, hi, lo); },
                      [&](int i) { return (int)oct_tq[rb * oct_max + i]; },
                      [&](int i, int) {
                        const int o = rb * oct_max + i;
                        const int64_t n = n0 + c * 16 + li;
                        return n < Nout ? *(const uint4*)((const bf16_t*)(uintptr_t)oct_L[o] + n * oct_r[o]) : make_uint4(0, 0, 0, 0);
                      });
      } else if (t_s[row] >= 0) {
        // ranks that are no multiples of 8, or factors stored rank-major: plain fp32 expand of this lane's row
        const int rank = rank_s[row];
        const bf16_t* L = (const bf16_t*)(uintptr_t)rL_s[row];
        const int64_t n = n0 + c * 16 + 4 * lg;
        if (n < Nout)
          for (int q = 0; q < rank; ++q) {
            const float uq = u_s[row * us + q];
#pragma unroll
            for (int v = 0; v < 4; ++v)
              y[k][0][v] = fmaf(uq, bf16_bits_to_float(a.lform == FORM_NT ? L[(n + v) * rank + q] : L[(int64_t)q * Nout + n + v]), y[k][0][v]);
          }
      }
    }
  }
#pragma unroll
  for (int k = 0; k < MINE; ++k) {
    const int tile = wave + k * TH_WAVES, rb = tile / NC, c = tile - rb * NC;
    if (tile >= TILES) break;
    const int32_t tok = tok_s[rb * 16 + li];
    const int64_t n = n0 + c * 16 + 4 * lg;
    if (tok < 0 || n >= Nout) continue;            // (Nout is a multiple of 8: four columns are in or out together)
    if (a.out_is_f32) {
      *(f32x4*)((float*)a.proj[p].out + (int64_t)tok * a.proj[p].ldo + n) = y[k][0];
    } else {
      uint2 o;
      o.x = float_to_bf16_bits(y[k][0][0]) | ((uint32_t)float_to_bf16_bits(y[k][0][1]) << 16);
      o.y = float_to_bf16_bits(y[k][0][2]) | ((uint32_t)float_to_bf16_bits(y[k][0][3]) << 16);
      *(uint2*)((bf16_t*)a.proj[p].out + (int64_t)tok * a.proj[p].ldo + n) = o;
    }
  }
}

template <int R, int NC, bool ROWS>
static hipError_t launch_thin(const GemmArgs& a, hipStream_t stream) {
  const size_t lds = (size_t)TH_WAVES * R * NC * 1024 + (size_t)16 * R * (a.r_stride + 4) * sizeof(float) +
                     (size_t)R * 2 * a.r_stride * 16 + (size_t)16 * R * 20 + R * 4 + 64;
  static std::atomic<uint64_t> done_dev{0};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  const uint64_t bit = 1ull << (dev & 63);
  if (!(done_dev.load(std::memory_order_acquire) & bit)) {
    e = hipFuncSetAttribute((const void*)gemm_thin_kernel<R, NC, ROWS>, hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
    if (e != hipSuccess) return e;
    done_dev.fetch_or(bit, std::memory_order_release);
  }
  hipLaunchKernelGGL((gemm_thin_kernel<R, NC, ROWS>), dim3(a.n_prod + a.tiles_n), dim3(TH_THREADS), lds, stream, a);
  return hipGetLastError();
}

// Column blocks per workgroup: as few as keep the consumers near 160 (4096 columns, rank-16 adapters, 1
// / 6 / 32 rows: 12.6 / 13.4 / 22.7 us with one block each, 10.3 / 11.8 / 16.4 with two: half as many
// workgroups read u and x).
hipError_t launch_gemm_thin(GemmArgs a, hipStream_t stream) {
  // splits of a producer's contraction: so that a wave of it has about eight steps, two rounds of loads
  const int64_t steps = ((a.Kc + 31) / 32 + TH_WAVES - 1) / TH_WAVES;
  a.n_split = (int)(steps <= 8 ? 1 : steps <= 16 ? 2 : THIN_SPLITS);
  a.n_prod *= a.n_split;
  const int R = a.T <= 16 ? 1 : 2;
  int64_t blocks = 0;
  for (int p = 0; p < a.n_proj; ++p) blocks += (a.proj[p].Nout + 15) / 16;
  const int nc = blocks <= 160 ? 1 : blocks <= 320 ? 2 : 4;
  a.tiles_n = 0;
  for (int p = 0; p < a.n_proj; ++p) {
    a.proj[p].tile0 = a.tiles_n;
    a.tiles_n += (int)((a.proj[p].Nout + 16 * nc - 1) / (16 * nc));
  }
  const bool rows = thin_rows(a.T, a.Kc, a.lda);
#define TH_PICK(R_, NC_) (rows ? launch_thin<R_, NC_, true>(a, stream) : launch_thin<R_, NC_, false>(a, stream))
  if (R == 1) return nc == 4 ? TH_PICK(1, 4) : nc == 2 ? TH_PICK(1, 2) : TH_PICK(1, 1);
  return nc == 4 ? TH_PICK(2, 4) : nc == 2 ? TH_PICK(2, 2) : TH_PICK(2, 1);
#undef TH_PICK
}

}  // namespace marlaas
