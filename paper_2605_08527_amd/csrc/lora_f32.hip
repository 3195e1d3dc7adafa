// fp32 path: the same layer in fp32 arithmetic for fp32 inputs (fp32 matrix instructions: full fp32
// products, fp32 accumulation, no rounding of inputs).  Sized for small problems, where the time is
// launches and memory latency; it exists so that fp32 data is never silently down-cast to bf16.
#include "common.h"

namespace marlaas {

static constexpr int F_WAVES = 8, F_THREADS = 64 * F_WAVES;
static constexpr int F_E = 2;          // 16-wide shrink tiles per pass over the contraction
static constexpr int F_U = 4;          // contraction steps whose operands are requested together

__device__ __forceinline__ const AdapterEntry& entry_of(const TablesF32& tb, int t) { return tb.n_inl ? tb.entry[t] : tb.table[t]; }

struct LayerF32Args {
  const float* X; int64_t ldx;
  const float* W; int64_t ldw;
  int64_t T, Kc, Nout;
  const int32_t* perm; const int32_t* grp;   // grp: adapter of every grouped row (null: no adapters)
  int which;                                 // 1: shrink by A, expand by B; 0: the other way round
  float* u_out; int r_stride;                // scaled shrink result, grouped order (may be null)
  void* out; int64_t ldo; int out_is_f32;
  int col_blocks;
  TablesF32 tb;
};

// One 16-row x 16 NC-column tile of the output per block, its eight waves splitting the contraction
// (partial tiles meet in LDS, added in wave order), the shrink of the rows' own adapters computed
// alongside as further 16-wide tiles (all column blocks of a row block repeat it: at most a few
// tiles, against a launch of its own), and the expand on the same matrix instructions.  NC = 0: the
// shrink alone.
//
// Bound: latency.  At 64 x 512 x 512 everything a wave needs (64 contraction values) is requested
// at once; the chain is index -> operands -> 16 MFMAs -> LDS -> expand -> store.  One thread per
// output and a shrink of its own, as this path was before, walked a serial chain of 512 dependent
// multiply-adds twice: 103 us per call, of which 5 us for a table upload that now travels in the
// arguments.
//
// A 16-deep step is four 16x16x4 MFMAs; lane (lg = lane / 16, li = lane % 16) supplies contraction
// values 4 lg .. + 3 of its row / column, one per MFMA (both operands use the same assignment).
template <int FORM, int NC>
__global__ __launch_bounds__(F_THREADS) void layer_f32_kernel(LayerF32Args a) {
  constexpr int U = NC == 4 || (FORM == FORM_NN && NC == 2) ? 2 : F_U;   // (registers)
  __shared__ f32x4 red[F_WAVES][NC + F_E][64];
  __shared__ __attribute__((aligned(16))) float u_s[F_E][16][20];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lg = lane >> 4;
  const int64_t rb = blockIdx.x / a.col_blocks, cbk = blockIdx.x - rb * a.col_blocks;
  const int64_t m0 = rb * 16, n0 = cbk * (16 * NC);
  const int64_t m = m0 + li < a.T ? m0 + li : a.T - 1;
  const int32_t tok = a.perm ? a.perm[m] : (int32_t)m;
  const int g = (a.grp && m0 + li < a.T) ? a.grp[m] : -1;   // adapter of row li (the same in all lane groups)
  const float* xr = a.X + (int64_t)tok * a.ldx;
  const int64_t kper = ((a.Kc + 16 * F_WAVES - 1) / (16 * F_WAVES)) * 16;
  const int64_t kb = wave * kper, ke = kb + kper < a.Kc ? kb + kper : a.Kc;

  // base-product columns of this lane (clamped columns are never stored)
  int64_t wcol[NC > 0 ? NC : 1];
#pragma unroll
  for (int c = 0; c < NC; ++c) { wcol[c] = n0 + 16 * c + li; if (wcol[c] >= a.Nout) wcol[c] = a.Nout - 1; }
  uint32_t woff[NC > 0 ? NC : 1];
#pragma unroll
  for (int c = 0; c < NC; ++c) woff[c] = (uint32_t)(4 * lg * a.ldw + wcol[c]);

  f32x4 y = f32x4{0.f, 0.f, 0.f, 0.f};        // wave c < NC: output tile c
  uint32_t todo = (uint32_t)(__ballot(g >= 0) & 0xffff);   // rows whose adapter has not been listed yet
  int t_cur = -1, q_cur = 0, r_cur = 0;
  for (int pass = 0;; ++pass) {
    // the next (at most F_E) shrink tiles: 16 ranks of one adapter each
    int et[F_E], eq[F_E], er[F_E];
    const float* ein[F_E];
    int n_e = 0;
#pragma unroll
    for (int e = 0; e < F_E; ++e) {
      et[e] = -1; eq[e] = 0; er[e] = 0; ein[e] = nullptr;
      if (t_cur < 0 && todo) {
        t_cur = __builtin_amdgcn_readlane(g, __ffs(todo) - 1);
        todo &= ~(uint32_t)(__ballot(g == t_cur) & 0xffff);
        r_cur = entry_of(a.tb, t_cur).rank;
        q_cur = 0;
      }
      if (t_cur >= 0) {
        const AdapterEntry& en = entry_of(a.tb, t_cur);
        et[e] = t_cur; eq[e] = q_cur; er[e] = r_cur; ein[e] = (const float*)(a.which ? en.A : en.B);
        n_e = e + 1;
        q_cur += 16;
        if (q_cur >= r_cur) t_cur = -1;
      }
    }
    if (pass > 0 && n_e == 0) break;
    if (pass == 0 && NC == 0 && n_e == 0) return;
    f32x4 acc[NC + F_E];
#pragma unroll
    for (int i = 0; i < NC + F_E; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int64_t k0 = kb; k0 < ke; k0 += 16 * U) {
      float4 xv[U], wv[NC + F_E][U];
#pragma unroll
      for (int s = 0; s < U; ++s) {
        const int64_t k = k0 + 16 * s + 4 * lg;
        const bool in = k < ke;                     // (Kc is a multiple of 8: four values are in or out together)
        xv[s] = make_float4(0.f, 0.f, 0.f, 0.f);
        if (in) xv[s] = *(const float4*)(xr + k);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
          float4 w = make_float4(0.f, 0.f, 0.f, 0.f);
          if (in && pass == 0) {
            if (FORM == FORM_NT) w = *(const float4*)(a.W + wcol[c] * a.ldw + k);
            else {                                  // (scalar row base, 32-bit lane offset: below 2^28 bytes)
              const float* p = a.W + (k0 + 16 * s) * a.ldw;
              w = make_float4(p[woff[c]], (p + a.ldw)[woff[c]], (p + 2 * a.ldw)[woff[c]], (p + 3 * a.ldw)[woff[c]]);
            }
          }
          wv[c][s] = w;
        }
#pragma unroll
        for (int e = 0; e < F_E; ++e) {
          float4 w = make_float4(0.f, 0.f, 0.f, 0.f);
          const int q = eq[e] + li;
          if (e < n_e && in && q < er[e]) {
            const int64_t r = er[e];
            if (FORM == FORM_NT) w = *(const float4*)(ein[e] + q * a.Kc + k);
            else {
              const float* p = ein[e] + (k0 + 16 * s) * r;
              const uint32_t o = 4 * lg * (uint32_t)r + q;
              w = make_float4(p[o], (p + r)[o], (p + 2 * r)[o], (p + 3 * r)[o]);
            }
          }
          wv[NC + e][s] = w;
        }
      }
#pragma unroll
      for (int s = 0; s < U; ++s)
#pragma unroll
        for (int i = 0; i < NC + F_E; ++i)
          if (i < NC ? pass == 0 : i - NC < n_e) {
            acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[s].x, wv[i][s].x, acc[i], 0, 0, 0);
            acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[s].y, wv[i][s].y, acc[i], 0, 0, 0);
            acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[s].z, wv[i][s].z, acc[i], 0, 0, 0);
            acc[i] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[s].w, wv[i][s].w, acc[i], 0, 0, 0);
          }
    }
#pragma unroll
    for (int i = 0; i < NC + F_E; ++i)
      if (i < NC ? pass == 0 : i - NC < n_e) red[wave][i][lane] = acc[i];
    __syncthreads();
    // wave i adds up tile i (accumulator layout: row 4 lg + v, column li)
    static_assert(NC + F_E <= F_WAVES, "one wave per tile");
    if (wave < NC ? pass == 0 : wave - NC < n_e) {
      f32x4 s = red[0][wave][lane];
#pragma unroll
      for (int w = 1; w < F_WAVES; ++w) {
        const f32x4 p = red[w][wave][lane];
        s[0] += p[0]; s[1] += p[1]; s[2] += p[2]; s[3] += p[3];
      }
      if (wave < NC) {
        y = s;
      } else {
        int t = -1, q0 = 0, r = 0;
#pragma unroll
        for (int e = 0; e < F_E; ++e) if (e == wave - NC) { t = et[e]; q0 = eq[e]; r = er[e]; }
        const float scale = entry_of(a.tb, t).scale;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          const int row = 4 * lg + v;
          const bool mine = __shfl(g, row) == t;
          const float val = mine && q0 + li < r ? scale * s[v] : 0.f;
          u_s[wave - NC][row][li] = val;
          if (mine && cbk == 0 && a.u_out) a.u_out[(m0 + row) * a.r_stride + q0 + li] = val;
        }
      }
    }
    __syncthreads();
    if (NC > 0 && wave < NC && n_e > 0) {
      int64_t col = n0 + 16 * wave + li;
      if (col >= a.Nout) col = a.Nout - 1;
      int gr[4];                                // adapters of this lane's four output rows
#pragma unroll
      for (int v = 0; v < 4; ++v) gr[v] = __shfl(g, 4 * lg + v);
#pragma unroll
      for (int e = 0; e < F_E; ++e)
        if (e < n_e) {
          // (only the adapter's own rows take the sum: the others' u is 0, and 0 times a factor that is
          // infinite or not a number is not 0)
          f32x4 z = y;
          const AdapterEntry& en = entry_of(a.tb, et[e]);
          const float* L = (const float*)(a.which ? en.B : en.A);
          const int r = er[e], q = eq[e] + 4 * lg;
          const f32x4 uv = *(const f32x4*)&u_s[e][li][4 * lg];
          float lv[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int j = 0; j < 4; ++j)
            if (q + j < r) lv[j] = FORM == FORM_NT ? L[col * r + q + j] : L[(int64_t)(q + j) * a.Nout + col];
#pragma unroll
          for (int j = 0; j < 4; ++j) z = __builtin_amdgcn_mfma_f32_16x16x4f32(uv[j], lv[j], z, 0, 0, 0);
#pragma unroll
          for (int v = 0; v < 4; ++v) y[v] = gr[v] == et[e] ? z[v] : y[v];
        }
    }
  }
  if (NC > 0 && wave < NC) {
    const int64_t col = n0 + 16 * wave + li;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const int64_t t = __shfl(tok, 4 * lg + v);
      if (m0 + 4 * lg + v < a.T && col < a.Nout) {
        if (a.out_is_f32) ((float*)a.out)[t * a.ldo + col] = y[v];
        else ((bf16_t*)a.out)[t * a.ldo + col] = float_to_bf16_bits(y[v]);
      }
    }
  }
}

// dA_t / dB_t: a 32-column x 16-rank tile of one adapter's gradient per block, its tokens dealt out
// to eight waves four at a time (contraction index of the MFMA), the waves' sums added in wave order.
// Bound by latency and by reading X once; the former one thread per gradient element walked the
// adapter's tokens as a serial chain.  Both gradients in one launch, as neither
// fills the chip (forward and backward of 20 rows of 304 x 920 22.7 -> 19.5 us, 23 of 696 x 776 30.3 -> 27.1, 70 of
// 328 x 488 22.7 -> 19.4).
static constexpr int G_CT = 2;
struct ReduceF32Args {
  ReduceF32Job job[2];
  int blocks0;                               // of the first one's columns
  const int32_t* perm; const int32_t* seg_off;
  int r_stride, accumulate;
  TablesF32 tb;
};
__global__ __launch_bounds__(F_THREADS) void reduce_f32_kernel(ReduceF32Args a) {
  __shared__ f32x4 red[F_WAVES][G_CT][64];
  const int t = blockIdx.y;
  const int r = entry_of(a.tb, t).rank;
  const int q0 = blockIdx.z * 16;
  if (q0 >= r) return;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, li = lane & 15, lg = lane >> 4;
  const int lo = a.seg_off[t], hi = a.seg_off[t + 1];
  const bool second = (int)blockIdx.x >= a.blocks0;
  const ReduceF32Job j = second ? a.job[1] : a.job[0];
  const int64_t c0 = (int64_t)(blockIdx.x - (second ? a.blocks0 : 0)) * (16 * G_CT);
  f32x4 acc[G_CT];
#pragma unroll
  for (int i = 0; i < G_CT; ++i) acc[i] = f32x4{0.f, 0.f, 0.f, 0.f};
  constexpr int STEP = 4 * F_WAVES;
  for (int s = lo + 4 * wave; s < hi; s += STEP * F_U) {
    int32_t tok[F_U];
    float vv[F_U], xv[G_CT][F_U];
#pragma unroll
    for (int i = 0; i < F_U; ++i) {
      const int m = s + i * STEP + lg;
      tok[i] = m < hi ? (a.perm ? a.perm[m] : m) : -1;
      vv[i] = (m < hi && q0 + li < r) ? j.V[(int64_t)m * a.r_stride + q0 + li] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < F_U; ++i)
#pragma unroll
      for (int c = 0; c < G_CT; ++c) {
        const int64_t col = c0 + 16 * c + li;
        xv[c][i] = (tok[i] >= 0 && col < j.C) ? j.X[(int64_t)tok[i] * j.ldx + col] : 0.f;
      }
#pragma unroll
    for (int i = 0; i < F_U; ++i)
#pragma unroll
      for (int c = 0; c < G_CT; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(xv[c][i], vv[i], acc[c], 0, 0, 0);
  }
#pragma unroll
  for (int c = 0; c < G_CT; ++c) red[wave][c][lane] = acc[c];
  __syncthreads();
  if (wave >= G_CT) return;
  f32x4 s = red[0][wave][lane];
#pragma unroll
  for (int w = 1; w < F_WAVES; ++w) {
    const f32x4 p = red[w][wave][lane];
    s[0] += p[0]; s[1] += p[1]; s[2] += p[2]; s[3] += p[3];
  }
  const GradEntry& ge = a.tb.n_inl ? a.tb.grad[t] : a.tb.grads[t];
  float* o = j.which ? ge.dB : ge.dA;
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int64_t c = c0 + 16 * wave + 4 * lg + v;
    const int q = q0 + li;
    if (c < j.C && q < r) {
      float* d = o + (j.oform == FORM_NN ? c * r + q : (int64_t)q * j.C + c);
      *d = a.accumulate ? *d + s[v] : s[v];
    }
  }
}

// Column tiles per block: four (the weight is then read with the fewest repeats of x and of the
// shrink) once that still gives every compute unit two blocks, else as few as one, because a small
// problem's time is the length of one wave's chain and not the traffic.
hipError_t launch_layer_f32(const float* X, int64_t ldx, const float* W, int64_t ldw, int form, int64_t T, int64_t Kc, int64_t Nout,
                            const int32_t* perm, const int32_t* grp, const TablesF32& tb, int which, float* u_out, int r_stride,
                            void* out, int64_t ldo, int out_is_f32, hipStream_t stream) {
  if (T <= 0 || Nout <= 0) return hipSuccess;
  LayerF32Args a;
  a.X = X; a.ldx = ldx; a.W = W; a.ldw = ldw; a.T = T; a.Kc = Kc; a.Nout = Nout; a.perm = perm; a.grp = grp;
  a.which = which; a.u_out = u_out; a.r_stride = r_stride; a.out = out; a.ldo = ldo; a.out_is_f32 = out_is_f32; a.tb = tb;
  const int64_t rows = (T + 15) / 16;
  int nc = 0;
  if (out) for (nc = 4; nc > 1 && rows * ((Nout + 16 * nc - 1) / (16 * nc)) < 512; nc >>= 1) {}
  const int64_t cols = nc ? (Nout + 16 * nc - 1) / (16 * nc) : 1;
  if (rows * cols > 0x7fffffff) return hipErrorInvalidValue;
  a.col_blocks = (int)cols;
  typedef void (*kern_t)(LayerF32Args);
#define F_PICK(F_) (nc == 4 ? layer_f32_kernel<F_, 4> : nc == 2 ? layer_f32_kernel<F_, 2> : nc == 1 ? layer_f32_kernel<F_, 1> : layer_f32_kernel<F_, 0>)
  const kern_t kern = form == FORM_NT ? F_PICK(FORM_NT) : F_PICK(FORM_NN);
#undef F_PICK
  hipLaunchKernelGGL(kern, dim3((unsigned)(rows * cols)), dim3(F_THREADS), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_reduce_f32(const ReduceF32Job (&jobs)[2], const int32_t* perm, const int32_t* seg_off, int n_adapters, const TablesF32& tb,
                             int r_stride, int accumulate, hipStream_t stream) {
  if (n_adapters <= 0) return hipSuccess;
  ReduceF32Args a;
  int64_t blocks[2];
  for (int i = 0; i < 2; ++i) { a.job[i] = jobs[i]; blocks[i] = (jobs[i].C + 16 * G_CT - 1) / (16 * G_CT); }
  if (blocks[0] + blocks[1] > 0x7fffffff) return hipErrorInvalidValue;
  a.blocks0 = (int)blocks[0];
  a.perm = perm; a.seg_off = seg_off; a.r_stride = r_stride; a.accumulate = accumulate; a.tb = tb;
  hipLaunchKernelGGL(reduce_f32_kernel, dim3((unsigned)(blocks[0] + blocks[1]), n_adapters, (r_stride + 15) / 16), dim3(F_THREADS), 0, stream, a);
  return hipGetLastError();
}

}  // namespace marlaas
