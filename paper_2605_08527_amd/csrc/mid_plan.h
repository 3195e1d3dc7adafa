// How a call of some rows in one launch (gemm_mid.hip) is tiled, and whether it is.  Host code only.
#pragma once
#include "gemm_args.h"

#include <algorithm>
#include <cmath>

namespace marlaas {

static constexpr int MID_WAVES = 8;

// Pieces of a producer's contraction.  A compute unit that has a producer besides its consumer is behind the
// others by what the producer reads (256 rows, 4096 x 4096: first tile after 9 us instead of 4 with two pieces,
// 6 with four), and a last wave of workgroups costs more than that.
//   Whole (up to 16 steps a wave), where every workgroup has a unit of its own: 157 rows 22.7 -> 19.9 us.
//   Else four pieces, if all workgroups are on the chip at once: 256 rows 23.8 -> 22.4, 157 rows 14336 x 4096
//   51 -> 43; two, if only those are, but for a few (q/k/v of 256 rows: four pieces 47 us, two 33; 256 rows of
//   rank 64, 568 workgroups in two pieces at most: 33.3, whole 36.5).
//   Else whole as far as the steps allow (300 rows of rank 128: 50 us, in two 62; 512 rows, 5120 x 5120, 64
//   adapters, with their regrouping 82 and 88).
// Few steps are not cut: a value of u is read once for each piece.  More than 24 always are (eight projections of 1024
// columns, contraction 8192, 1000 rows of 4 adapters of rank 128: 364 us, whole 402, 600 rows of 8 adapters 288 and 282; of
// 512 columns, contraction 7168, 640 rows of 32 adapters: 340 and 1035).
//   u_room: floats of u that there is room for.
inline int mid_u_splits(int64_t Kc, int64_t u_floats, int64_t u_room, int64_t consumers, int64_t jobs, int cu_count) {
  const int64_t steps = ((Kc + 31) / 32 + MID_WAVES - 1) / MID_WAVES;      // 32-deep steps of a wave
  if (steps <= 8 || (steps <= 16 && consumers + jobs <= cu_count)) return 1;
  int s = MID_SPLITS;
  while (s > 1 && (consumers + jobs * s > (s == 2 ? 9 : 8) * cu_count / 4 || u_floats * s > u_room)) s /= 2;
  return s == 1 && steps > 24 && 2 * u_floats <= u_room ? 2 : s;
}

// Estimated run time of a tiling in microseconds, for the order of the tilings.  A k-tile's time when a workgroup has
// its compute unit to itself, which two on one unit take 1.8 times as long for; against it what the fabric
// delivers; the expand by the ranks and row blocks of a wave; producers, where they share a unit with a consumer
// or make a last wave of workgroups; the exchange of split contractions, which costs more where no producers are waited
// for anyway (298 rows without adapters, 1496 x 1160, 11.5 us in two splits, whole 9.5).
//   Against 425 sets of 17 to 1024 rows, contractions of 1024 to 14336, 1024 to 28672 columns in one to three
// projections, without adapters and with 1 to 96 of ranks 8 to 128, timed in every tiling with weights from the
// memory-side cache and from memory (tests/golden/some_rows_tilings.json): the one chosen takes 2.5 % longer than the
// best on the average, at most 1.31 times as long.
//   Few units with two workgroups count for little (64 units, over which a second workgroup comes to count in
// full): with weights from memory 512 rows, 5120 x 5120, 32 adapters of rank 16, take 54 us in 280 workgroups of 80
// rows and 67 in 320 of 64; from the cache 53 and 52.
inline MidPlan mid_plan(int64_t T, int64_t Kc, const ProjEntry* proj, int n_proj, const MidLora& lora, int max_split) {
  static const double tile_us[2][2] = {{0.306, 0.252}, {0.334, 0.282}};   // [rb - 4][wn == 4]
  MidPlan best;
  int64_t cols = 0;
  for (int q = 0; q < n_proj; ++q) cols += proj[q].Nout;
  auto up_to_1 = [](double v) { return v < 0.0 ? 0.0 : v > 1.0 ? 1.0 : v; };
  for (int wn = 2; wn <= 4; wn += 2) {
    const int64_t kt = 32 * (MID_WAVES / wn), ktiles = (Kc + kt - 1) / kt;
    int64_t tiles_n = 0;
    for (int q = 0; q < n_proj; ++q) tiles_n += (proj[q].Nout + 32 * wn - 1) / (32 * wn);
    for (int rb = 4; rb <= 5; ++rb) {
      const int64_t tiles_m = (T + 16 * rb - 1) / (16 * rb);
      for (int s = 1; s <= max_split; s *= 2) {
        const int64_t wgs = tiles_m * tiles_n * s;
        if (s > 1 && (wgs > MID_SPLIT_WGS || ktiles < 4 * s)) continue;
        const double t1 = tile_us[rb - 4][wn == 4] * (double)((ktiles + s - 1) / s), t2 = 1.827 * t1;
        double fill;
        if (wgs <= 256) {
          fill = t1 * (wgs > 128 ? 1.0 + 0.066 * (double)(wgs - 128) / 128.0 : 1.0);
        } else {
          const int64_t left = wgs % 512;
          fill = (double)(wgs / 512) * (t2 + 2.172);
          if (left > 0) fill += 2.172 + 1.066 * t1 + (t2 - 1.066 * t1) * up_to_1((double)(left - 256) / 64.0);
        }
        const double fabric = (2.0 * cols * Kc + 16.0 * T * Kc / s) / 11.6e6;
        double us = 7.687 + cbrt(fill * fill * fill + fabric * fabric * fabric);
        if (lora.n > 0) {
          // (the most u there can be, of five projections and more, counts as whole: the estimate of such calls is low, and with
          // two pieces would take six of 1024 columns, contraction 14336, 1000 rows of rank 128, here, 496 us, not one by one, 298)
          const int pieces = mid_u_splits(Kc, T * lora.r_stride * n_proj, MID_U_FLOATS / 2, wgs, (int64_t)n_proj * mid_max_jobs(T, rb, lora), 256);
          const int64_t with_rows = (int64_t)(0.6 * T) + 1 < lora.n ? (int64_t)(0.6 * T) + 1 : lora.n;      // (adapters, about)
          const int64_t prods = n_proj * pieces * (with_rows * (lora.tiles / lora.n > 1 ? lora.tiles / lora.n : 1) + T / (16 * rb) * ((rb + 1) / 2));
          // (the expand of more ranks is not proportionally more: 184 rows, 1872 x 8368, rank 32, 23.1 -> 22.1 us
          // in tiles of 128 columns; a split makes every rank's u travel to more readers: 277 rows, 2144 x 1048, rank 64,
          // 20.0 -> 18.4 unsplit)
          const double rank = std::min(16.0, (double)lora.ranks / lora.n);
          const double prod_us = 10.735 * Kc / 4096.0 / pieces + 0.498;
          us += 0.562 + 2.009 * ((rb * wn + 7) / 8) * rank / 16.0 + (s > 1 ? 0.02 * lora.ranks / lora.n : 0.0);
          us += prod_us * (wgs <= 256 ? 0.574 * up_to_1((double)(wgs + prods - 256) / 17.45) : 0.289 * up_to_1((double)prods / 256.0));
          us += prod_us * 0.918 * up_to_1((double)((wgs < 512 ? wgs : 512) + prods - 512) / 17.45);
        }
        if (s > 1) us += (lora.n > 0 ? 0.0 : 1.5) + (s > 2 ? 2.442 : 2.257) * (0.5 + rb * wn / 32.0) + (wgs > 192 ? 0.186 * (double)(wgs - 192) / 64.0 : 0.0);
        if (best.rb == 0 || us < best.us) { best.us = us; best.rb = rb; best.wn = wn; best.ksplit = s; best.tiles_m = (int)tiles_m; }
      }
    }
  }
  return best;
}

// Whether the call is better off elsewhere (ext: ranks of all adapters in the batch, 0: no adapters).
//   Up to 16 rows the few-row kernel, up to 32 while its workgroups, which hold all of x, have little of it.
//   Above 384 rows the wide kernel.  With adapters where its rate, which has to make up for its shrink's launch and its
// ext columns, says so (400 rows, 4096 x 14336, 32 adapters of rank 16 86 against 75 us; 14336 x 4096 109 / 75).
// Without where its plan does, in the room for sums that the call has (wide_us: its estimated time, asked for there); the
// estimate leaves out the 6 us of a launch and its first requests, and the one here what rows of x above 4096 cost: of 24
// sizes of 395 to 995 rows the choice costs 0.7 % on the average, 4.5 % without both (407 rows, 1608 x 5544, 28 / 21; 422
// rows, 5048 x 13864, 79 / 106; 751 rows, 10784 x 10280, 143 / 250).
//   Up to 256 rows the split kernel with its separate finish on a long contraction and few columns, where the row
//   tiles here are few and their splits expensive (256 rows, 14336 x 4096, no adapter: 36 / 41, 157 rows 37 / 31;
//   200 rows, 20480 x 2048, 32 adapters of rank 16: 44 / 52; 256 rows, 14336 x 4096 from memory 63 / 70; up to 128
//   rows with adapters never: 100 rows 45 / 35 and 37 / 36).
template <typename Wide>
inline bool mid_pays(const MidPlan& p, int64_t T, int64_t Kc, int64_t cols, int ext, Wide wide_us) {
  if (T <= 16) return false;
  if (T <= 32) return T * Kc > 140000 || Kc * cols > 50000000;
  if (T > 384 && ext > 0) return p.us < 20.0 + 2.0 * T * Kc * cols / 1.25e9 + 0.1 * ext;
  if (T > 384) return p.us * (Kc > 4096 ? 1.0 + 0.2 * log2((double)Kc / 4096.0) : 1.0) < 6.0 + wide_us();
  if (T > 64 && T <= 256 && Kc >= 2 * cols && Kc * cols >= 40000000) {
    if (ext == 0) return p.us < 15.0 + Kc * cols * (T <= 128 ? 0.29e-6 : 0.365e-6);
    if (T > 128 && ext <= 512) return 1.15 * p.us < 15.0 + Kc * cols * 0.67e-6;
  }
  return true;
}

}  // namespace marlaas
