// Token grouping by adapter: a stable counting sort, one launch of one block for the batches of a
// serving step (segmap_small), several small kernels for very large ones.
// The mixed-tenant batch carries one adapter id per token (paper Sec. 4.5,
// cross-task batching of rollouts); every later kernel works on tokens grouped
// by adapter, so this map is built once per batch and reused by all layers.
#include "common.h"

namespace marlaas {

static constexpr int SEG_THREADS = 256;
static constexpr int SEG_CHUNK = 2048;  // tokens per block

int segmap_blocks(int64_t T) { return (int)((T + SEG_CHUNK - 1) / SEG_CHUNK); }

// bucket n collects tokens with id -1; flags[0] |= 1 on an id outside [-1, n),
// flags[1] |= 1 when the ids are not already grouped in bucket order.
__global__ __launch_bounds__(SEG_THREADS) void segmap_hist(const int32_t* __restrict__ ids,
                                                           int64_t T, int n,
                                                           int32_t* __restrict__ block_hist,
                                                           int32_t* __restrict__ flags) {
  extern __shared__ int32_t hist[];
  for (int b = threadIdx.x; b <= n; b += SEG_THREADS) hist[b] = 0;
  __syncthreads();
  int64_t base = (int64_t)blockIdx.x * SEG_CHUNK;
  bool bad = false, unsorted = false;
  for (int j = threadIdx.x; j < SEG_CHUNK; j += SEG_THREADS) {
    int64_t i = base + j;
    if (i >= T) break;
    int id = ids[i];
    if (id < -1 || id >= n) { bad = true; continue; }
    int b = id < 0 ? n : id;
    atomicAdd(&hist[b], 1);
    if (i + 1 < T) {
      int nx = ids[i + 1];
      int bn = nx < 0 ? n : nx;
      if (bn < b) unsorted = true;
    }
  }
  if (bad) atomicOr(&flags[0], 1);
  if (unsorted) atomicOr(&flags[1], 1);
  __syncthreads();
  for (int b = threadIdx.x; b <= n; b += SEG_THREADS)
    block_hist[(int64_t)blockIdx.x * (n + 1) + b] = hist[b];
}

// One block.  seg_off[b] = exclusive prefix of bucket totals (n + 2 entries);
// block_hist[blk][b] is replaced by the first output slot of block blk in bucket b.
__global__ __launch_bounds__(1024) void segmap_scan(int32_t* __restrict__ block_hist, int nblk,
                                                    int n, int32_t* __restrict__ seg_off) {
  extern __shared__ int32_t total[];
  for (int b = threadIdx.x; b <= n; b += blockDim.x) {
    int run = 0;
    for (int k = 0; k < nblk; ++k) {
      int c = block_hist[(int64_t)k * (n + 1) + b];
      block_hist[(int64_t)k * (n + 1) + b] = run;
      run += c;
    }
    total[b] = run;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int run = 0;
    for (int b = 0; b <= n; ++b) {
      int c = total[b];
      total[b] = run;
      seg_off[b] = run;
      run += c;
    }
    seg_off[n + 1] = run;
  }
  __syncthreads();
  for (int b = threadIdx.x; b <= n; b += blockDim.x) {
    int off = total[b];
    for (int k = 0; k < nblk; ++k) block_hist[(int64_t)k * (n + 1) + b] += off;
  }
}

// Stable scatter: tokens are taken 256 at a time in index order.  Inside a wave a token's rank
// among the earlier tokens of its bucket comes from ballots (one round per distinct bucket in
// the wave); the four waves of a group then take their slots from the bucket cursors one after
// the other, in wave order, so the order of equal ids is the order of their indices.
__global__ __launch_bounds__(SEG_THREADS) void segmap_scatter(const int32_t* __restrict__ ids,
                                                              int64_t T, int n,
                                                              const int32_t* __restrict__ block_base,
                                                              int32_t* __restrict__ perm,
                                                              int32_t* __restrict__ grp_ids) {
  extern __shared__ int32_t cursor[];  // [n + 1]
  for (int b = threadIdx.x; b <= n; b += SEG_THREADS)
    cursor[b] = block_base[(int64_t)blockIdx.x * (n + 1) + b];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));      // lanes before this one
  int64_t base = (int64_t)blockIdx.x * SEG_CHUNK;
  __syncthreads();
  for (int g = 0; g < SEG_CHUNK / SEG_THREADS; ++g) {
    int64_t i = base + (int64_t)g * SEG_THREADS + threadIdx.x;
    int b = -1;
    if (i < T) {
      int id = ids[i];
      if (id >= -1 && id < n) b = id < 0 ? n : id;
    }
    // rank inside the wave, and the number of the wave's tokens in the same bucket
    int rank = 0, cnt = 0;
    uint64_t todo = __ballot(b >= 0);
    while (todo) {
      const int leader = __ffsll((unsigned long long)todo) - 1;
      const int lb = __shfl(b, leader);
      const uint64_t same = __ballot(b == lb);
      if (b == lb) { rank = __popcll(same & below); cnt = __popcll(same); }
      todo &= ~same;
    }
    for (int w = 0; w < SEG_THREADS / 64; ++w) {
      if (wave == w && b >= 0) {
        const int slot = cursor[b] + rank;
        perm[slot] = (int32_t)i;
        grp_ids[slot] = b < n ? b : -1;                  // adapter of that grouped row
        if (rank == cnt - 1) cursor[b] += cnt;           // (the wave's reads of this cursor are behind it)
      }
      __syncthreads();
    }
  }
}

// Row chunks of the grouped order: segment t cut into pieces of ROW_CHUNK rows, the rows without
// an adapter (bucket n) last.  One block; thread b handles bucket b, the first chunk index of a
// bucket is the prefix sum of the buckets' chunk counts (serial over at most n + 1 values).
__global__ __launch_bounds__(1024) void segmap_chunks(const int32_t* __restrict__ seg_off, int n,
                                                      RowChunk* __restrict__ chunks) {
  extern __shared__ int32_t first[];   // [n + 2]
  if (threadIdx.x == 0) {
    int run = 0;
    for (int b = 0; b <= n; ++b) {
      first[b] = run;
      run += (seg_off[b + 1] - seg_off[b] + ROW_CHUNK - 1) / ROW_CHUNK;
    }
  }
  __syncthreads();
  for (int b = threadIdx.x; b <= n; b += blockDim.x) {
    const int32_t end = seg_off[b + 1];
    int c = first[b];
    for (int32_t row0 = seg_off[b]; row0 < end; row0 += ROW_CHUNK, ++c) {
      RowChunk ch;
      ch.row0 = row0; ch.nrows = end - row0 < ROW_CHUNK ? end - row0 : ROW_CHUNK; ch.t = b < n ? b : -1; ch.pad = 0;
      chunks[c] = ch;
    }
  }
}

// Adapters by falling segment length (ties: by index): order[k] = the adapter with the k-th longest
// segment.  Kernels whose blocks own whole segments take their adapter from it, so that the long
// segments start first and the short ones fill the end of the launch.  One block; every thread
// ranks its adapters by counting the ones that come before them (n <= 4096).
__global__ __launch_bounds__(1024) void segmap_order(const int32_t* __restrict__ seg_off, int n, int32_t* __restrict__ order,
                                                     int32_t* __restrict__ chunk_base) {
  extern __shared__ int32_t len[];     // [n]
  for (int t = threadIdx.x; t < n; t += blockDim.x) len[t] = seg_off[t + 1] - seg_off[t];
  __syncthreads();
  if (threadIdx.x == 0 && chunk_base != nullptr) {
    // first partial-sum slot of every adapter whose segment is cut into several token chunks
    const int tc = reduce_ragged_chunk(seg_off[n], n);
    int run = 0;
    for (int t = 0; t < n; ++t) {
      chunk_base[t] = run;
      const int nch = (len[t] + tc - 1) / tc;
      if (nch > 1) run += nch;
    }
    chunk_base[n] = run;
  }
  for (int t = threadIdx.x; t < n; t += blockDim.x) {
    const int mine = len[t];
    int before = 0;
    for (int s = 0; s < n; ++s) before += (len[s] > mine) || (len[s] == mine && s < t);
    order[before] = t;
  }
}

// ---- one launch for batches of up to SEG_SMALL_T tokens over up to SEG_SMALL_N adapters
static constexpr int SM_THREADS = 1024, SM_WAVES = SM_THREADS / 64;
static constexpr int64_t SEG_SMALL_T = 32768;
static constexpr int SEG_SMALL_N = 800;       // one bucket per thread in the scans, [waves][buckets] counters in LDS

// Exclusive prefix sums of two values per thread over the block's first `waves` waves (s_wave: 2 SM_WAVES ints of
// LDS that nobody else touches); every thread calls it, with 0 from the waves behind.
__device__ __forceinline__ int2 block_scan(int2 v, int waves, int32_t* s_wave, int2* total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int2 inc = v;
  if (wave < waves) {
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int x = __shfl_up(inc.x, d), y = __shfl_up(inc.y, d);
      if (lane >= d) { inc.x += x; inc.y += y; }
    }
    if (lane == 63) { s_wave[2 * wave] = inc.x; s_wave[2 * wave + 1] = inc.y; }
  }
  __syncthreads();
  int2 before = make_int2(0, 0), all = make_int2(0, 0);
  for (int w = 0; w < waves; ++w) {
    const int x = s_wave[2 * w], y = s_wave[2 * w + 1];
    if (w < wave) { before.x += x; before.y += y; }
    all.x += x; all.y += y;
  }
  *total = all;
  return make_int2(before.x + inc.x - v.x, before.y + inc.y - v.y);
}

// The whole grouping in one block: every wave owns a contiguous run of tokens, walks it 64 at a time
// and counts its buckets (tokens of one bucket inside a wave find each other with one ballot per bit
// of the bucket number); one scan over (bucket, wave) then gives every wave its first slot in every
// bucket, and a second walk hands the slots out.  No atomics on the slots, order of equal ids = order of indices.
// The segment sizes go straight to pinned host memory, behind them `seq`, which the host waits for.
//
// Bound: launch and latency.  As six launches and two copies the grouping of 512 tokens kept the host
// waiting 45 us (each of them 4 us of launch for under 2 us of work) before it could enqueue the pass.
// So up to 256 tokens a wave the ids stay in registers for the second walk, every wave ranks a share of the adapters,
// and one wave's fence, behind a barrier, serves for all: 512 tokens of 64 adapters 10.8 -> 6.3 us, a step that
// regroups them and runs one 5120 x 5120 projection 85.0 -> 79.6.
__global__ __launch_bounds__(SM_THREADS) void segmap_small(const int32_t* __restrict__ ids, int T, int n, int nbits,
                                                           int32_t* __restrict__ perm, int32_t* __restrict__ grp_ids,
                                                           int32_t* __restrict__ seg_off, RowChunk* __restrict__ chunks,
                                                           int32_t* __restrict__ order, int32_t* __restrict__ chunk_base,
                                                           int32_t* __restrict__ host, int seq) {
  extern __shared__ int32_t lds[];
  const int nb = n + 1;                       // buckets; bucket n: tokens without an adapter
  int32_t* cur = lds;                         // [SM_WAVES][nb] counts, then next slots
  int32_t* off = cur + SM_WAVES * nb;         // [nb + 1] segment offsets
  int32_t* first = off + nb + 1;              // [nb] first row chunk
  int32_t* rank_s = first + nb;               // [n] adapters with longer segments
  int32_t* s_wave = rank_s + n;               // [2][2 SM_WAVES]
  int32_t* flag = s_wave + 4 * SM_WAVES;      // [2]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const uint64_t below = lane == 0 ? 0ull : (~0ull >> (64 - lane));
  const int per = ((T + SM_THREADS - 1) / SM_THREADS) * 64;     // tokens per wave
  const int beg = wave * per, end = beg + per < T ? beg + per : T;
  const bool once = per <= 256;               // (the ids of a wave's tokens stay in registers)
  int idv[4], nxt[4];
  // (every lane reads, from an index inside: a request under a condition of its own waits for the one before it, 12000
  // tokens 44.6 -> 42.3 us; neighbours are the first walk's)
  auto load = [&](int s0, bool first_walk) {
#pragma unroll
    for (int j = 0; j < 4; ++j) { const int i = s0 + 64 * j + lane; idv[j] = ids[i < T ? i : T - 1]; }
    if (first_walk) {
#pragma unroll
      for (int j = 0; j < 4; ++j) { const int i = s0 + 64 * j + lane + 1; nxt[j] = ids[i < T ? i : T - 1]; }
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) if (s0 + 64 * j + lane >= end) idv[j] = -2;
  };
  if (once) load(beg, true);
  for (int i = tid; i < SM_WAVES * nb; i += SM_THREADS) cur[i] = 0;
  for (int i = tid; i < n; i += SM_THREADS) rank_s[i] = 0;
  if (tid < 2) flag[tid] = 0;
  __syncthreads();
  int32_t* mine = cur + wave * nb;
  bool bad = false, unsorted = false;
#pragma unroll 1
  for (int walk = 0; walk < 2; ++walk) {
    for (int s0 = beg; s0 < end; s0 += 256) {
      if (!once) load(s0, walk == 0);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = s0 + 64 * j + lane;
        if (s0 + 64 * j >= end) break;
        const bool ok = i < end && idv[j] >= -1 && idv[j] < n;
        const int b = idv[j] < 0 ? n : idv[j];
        if (walk == 0) {
          bad |= i < end && !ok;
          unsorted |= i < end && (nxt[j] < 0 ? n : nxt[j]) < b;
        }
        uint64_t same = __ballot(ok);
        for (int bit = 0; bit < nbits; ++bit) {
          const uint64_t m = __ballot((b >> bit) & 1);
          same &= ((b >> bit) & 1) ? m : ~m;
        }
        if (!ok) continue;
        const int rank = __popcll(same & below);
        const int slot = mine[b] + rank;
        asm volatile("" ::: "memory");        // (every lane has read its counter before the first of a bucket moves it)
        if (rank == 0) mine[b] = slot + __popcll(same);
        if (walk == 1) {
          perm[slot] = i;
          grp_ids[slot] = b < n ? b : -1;
          const int pos = slot - off[b];      // inside the bucket: every ROW_CHUNK-th token writes a row chunk
          if ((pos & (ROW_CHUNK - 1)) == 0) {
            const int left = off[b + 1] - slot;
            RowChunk ch;
            ch.row0 = slot; ch.nrows = left < ROW_CHUNK ? left : ROW_CHUNK; ch.t = b < n ? b : -1; ch.pad = 0;
            chunks[first[b] + pos / ROW_CHUNK] = ch;
          }
        }
      }
    }
    if (walk == 1) break;
    if (bad) flag[0] = 1;
    if (unsorted) flag[1] = 1;
    __syncthreads();
    int count[SM_WAVES], total = 0;
    if (tid < nb) {
#pragma unroll
      for (int w = 0; w < SM_WAVES; ++w) count[w] = cur[w * nb + tid];
#pragma unroll
      for (int w = 0; w < SM_WAVES; ++w) total += count[w];
    }
    int2 all;
    const int2 start = block_scan(make_int2(total, (total + ROW_CHUNK - 1) / ROW_CHUNK), (nb + 63) / 64, s_wave, &all);
    if (tid < nb) {
      off[tid] = start.x;
      first[tid] = start.y;
      seg_off[tid] = start.x;
      host[tid] = start.x;
      int run = start.x;
#pragma unroll
      for (int w = 0; w < SM_WAVES; ++w) { cur[w * nb + tid] = run; run += count[w]; }
    }
    if (tid == 0) {
      off[nb] = all.x; seg_off[nb] = all.x;
      host[nb] = all.x; host[nb + 1] = flag[0]; host[nb + 2] = flag[1];
    }
    __syncthreads();
  }
  // adapters by falling segment length, and the partial-sum slots of those that are cut (see segmap_order): every
  // wave compares all adapters, a lane each, with its share of them
  const int share = (n + SM_WAVES - 1) / SM_WAVES, s0 = wave * share, s1 = s0 + share < n ? s0 + share : n;
  if (s0 < s1)
    for (int t = lane; t < n; t += 64) {
      const int len = off[t + 1] - off[t];
      int before = 0;
#pragma unroll 4
      for (int s = s0; s < s1; ++s) {
        const int l = off[s + 1] - off[s];
        before += (l > len) || (l == len && s < t);
      }
      if (before) atomicAdd(&rank_s[t], before);
    }
  const int tc = reduce_ragged_chunk(off[n], n);
  const int nch = tid < n ? (off[tid + 1] - off[tid] + tc - 1) / tc : 0;
  int2 slots;
  const int2 cb = block_scan(make_int2(nch > 1 ? nch : 0, 0), (nb + 63) / 64, s_wave + 2 * SM_WAVES, &slots);    // (meets: the ranks are complete)
  if (tid < n) {
    chunk_base[tid] = cb.x;
    order[rank_s[tid]] = tid;
  }
  if (tid == 0) chunk_base[n] = slots.x;
  // Every wave's stores have reached the L2 or, the host's copy, its memory; then one wave writes back what the
  // other L2s and the host must see and says so.
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0) {
    __threadfence_system();
    __hip_atomic_store(host + nb + 3, seq, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

bool segmap_is_small(int64_t T, int n) { return T > 0 && T <= SEG_SMALL_T && n <= SEG_SMALL_N; }

hipError_t launch_segmap_small(const int32_t* ids, int64_t T, int n, int32_t* perm, int32_t* grp_ids, int32_t* seg_off,
                               RowChunk* chunks, int32_t* order, int32_t* chunk_base, int32_t* host, int seq, hipStream_t stream) {
  int nbits = 0;
  while ((n >> nbits) > 0) ++nbits;
  const size_t lds = sizeof(int32_t) * ((size_t)SM_WAVES * (n + 1) + (n + 2) + (n + 1) + n + 4 * SM_WAVES + 2);
  hipLaunchKernelGGL(segmap_small, dim3(1), dim3(SM_THREADS), lds, stream, ids, (int)T, n, nbits, perm, grp_ids, seg_off, chunks,
                     order, chunk_base, host, seq);
  return hipGetLastError();
}

int64_t segmap_chunk_count(const int32_t* seg_off, int n) {
  int64_t c = 0;
  for (int b = 0; b <= n; ++b) c += (seg_off[b + 1] - seg_off[b] + ROW_CHUNK - 1) / ROW_CHUNK;
  return c;
}

int64_t segmap_chunk_bound(int64_t T, int n) { return T / ROW_CHUNK + n + 2; }

// plain fill (a kernel, not a memset node)
__global__ void segmap_clear_flags(int32_t* flags) { flags[threadIdx.x] = 0; }

hipError_t launch_segmap(const int32_t* ids, int64_t T, int n, int32_t* perm, int32_t* grp_ids, int32_t* seg_off,
                         int32_t* block_hist, int32_t* flags, RowChunk* chunks, int32_t* order, int32_t* chunk_base,
                         hipStream_t stream) {
  int nblk = segmap_blocks(T);
  hipLaunchKernelGGL(segmap_clear_flags, dim3(1), dim3(2), 0, stream, flags);
  if (nblk > 0) {
    hipLaunchKernelGGL(segmap_hist, dim3(nblk), dim3(SEG_THREADS), (n + 1) * sizeof(int32_t),
                       stream, ids, T, n, block_hist, flags);
  }
  hipLaunchKernelGGL(segmap_scan, dim3(1), dim3(1024), (n + 1) * sizeof(int32_t), stream,
                     block_hist, nblk, n, seg_off);
  if (nblk > 0) {
    hipLaunchKernelGGL(segmap_scatter, dim3(nblk), dim3(SEG_THREADS),
                       (n + 1) * sizeof(int32_t), stream, ids, T, n, block_hist, perm, grp_ids);
  }
  hipLaunchKernelGGL(segmap_chunks, dim3(1), dim3(1024), (n + 2) * sizeof(int32_t), stream, seg_off, n, chunks);
  if (n > 0 && order != nullptr)
    hipLaunchKernelGGL(segmap_order, dim3(1), dim3(1024), n * sizeof(int32_t), stream, seg_off, n, order, chunk_base);
  return hipGetLastError();
}

}  // namespace marlaas
