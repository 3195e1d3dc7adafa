// How a call of some rows in one launch (gemm_mid.hip) is tiled, and whether it is.  Host code only.
#pragma once
#include "gemm_args.h"

#include <algorithm>
#include <cmath>

namespace marlaas {

static constexpr int MID_WAVES = 8;
// Tiles of 128 rows and more take all of a compute unit's registers.
__host__ __device__ constexpr bool mid_alone(int rb) { return rb > 6; }
// Whether producers take several jobs each: `free` units that the consumers leave, in whole rounds over the XCDs.
inline int64_t mid_free_units(int64_t cu_count, int64_t consumers) { return (cu_count - consumers) & ~7; }
inline bool mid_jobs_in_turn(int64_t free, int64_t jobs) { return free >= 32 && jobs > free && jobs <= 5 * free; }

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
//   Tiles of 96 rows (rb 6) are taken with all workgroups on the chip only (mid_taller), so theirs are never more than fit.
//   u_room: floats of u that there is room for.
inline int mid_u_splits(int64_t Kc, int64_t u_floats, int64_t u_room, int64_t consumers, int64_t jobs, int cu_count, int rb = 4) {
  const int64_t steps = ((Kc + 31) / 32 + MID_WAVES - 1) / MID_WAVES;      // 32-deep steps of a wave
  if (steps <= 8 || (steps <= 16 && consumers + jobs <= cu_count)) return 1;
  int s = MID_SPLITS;
  while (s > 1 && (consumers + jobs * s > (mid_alone(rb) ? 4 : s == 2 && rb < 6 ? 9 : 8) * cu_count / 4 || u_floats * s > u_room)) s /= 2;
  return s == 1 && steps > 24 && 2 * u_floats <= u_room ? 2 : s;
}

// Estimated run time of a tiling in microseconds, for the order of the tilings.  A k-tile's time when a workgroup has
// its compute unit to itself, which two on one unit take 1.8 times as long for; against it what the fabric
// delivers; the expand by the ranks and row blocks of a wave; producers, where they share a unit with a consumer
// or make a last wave of workgroups; the exchange of split contractions, which costs more where no producers are waited
// for anyway (298 rows without adapters, 1496 x 1160, 11.5 us in two splits, whole 9.5).
//   Against 425 sets of 17 to 1024 rows, contractions of 1024 to 14336, 1024 to 28672 columns in one to three
// projections, without adapters and with 1 to 96 of ranks 8 to 128, timed in every tiling with weights from the
// memory-side cache and from memory (tests/golden/some_rows_tilings.json): the one chosen takes 2.3 % longer than the
// best on the average, at most 1.31 times as long.
//   Few units with two workgroups count for little (64 units, over which a second workgroup comes to count in
// full): with weights from memory 512 rows, 5120 x 5120, 32 adapters of rank 16, take 54 us in 280 workgroups of 80
// rows and 67 in 320 of 64; from the cache 53 and 52.
static constexpr double mid_tile_us[2][2] = {{0.306, 0.252}, {0.334, 0.282}};   // [rb - 4][wn == 4]

// What the comparisons differ in: the rank up to which the expand takes longer, units with two workgroups that count in full, the
// fabric's rate and the share of a weight that a further row tile reads again, and the producers beside more consumers than units.
struct MidRates { double rank_cap, ramp, rate, again, beside; };
static constexpr MidRates MID_SMALL = {16.0, 64.0, 11.6e6, 0.0, 256.0}, MID_TALL = {12.3, 15.5, 32.0e6, 0.042, 102.0};

struct MidModel {
  int64_t T, Kc, cols;
  const MidRates c;
  const ProjEntry* proj; int n_proj;
  const MidLora& lora;
  MidModel(int64_t T_, int64_t Kc_, const ProjEntry* proj_, int n_proj_, const MidLora& lora_, const MidRates& rates)
      : T(T_), Kc(Kc_), cols(0), c(rates), proj(proj_), n_proj(n_proj_), lora(lora_) {
    for (int q = 0; q < n_proj; ++q) cols += proj[q].Nout;
  }
  static double up_to_1(double v) { return v < 0.0 ? 0.0 : v > 1.0 ? 1.0 : v; }
  int64_t ktiles(int wn) const { const int64_t kt = 32 * (MID_WAVES / wn); return (Kc + kt - 1) / kt; }
  int64_t tiles_m(int rb) const { return (T + 16 * rb - 1) / (16 * rb); }
  int64_t tiles_n(int wn) const {
    int64_t n = 0;
    for (int q = 0; q < n_proj; ++q) n += (proj[q].Nout + 32 * wn - 1) / (32 * wn);
    return n;
  }
  // column tiles (times splits) if all XCDs, which have whole ones, had as many as the fullest
  int64_t over_xcds(int wn, int s) const { return (tiles_n(wn) + 8 / s - 1) / (8 / s) * 8; }
  // the most shrink jobs, and the pieces that each is in
  int64_t jobs(int rb) const { return lora.n > 0 ? (int64_t)n_proj * mid_max_jobs(T, rb, lora) : 0; }
  int pieces(int rb, int64_t wgs, int64_t u_room) const { return mid_u_splits(Kc, T * lora.r_stride * n_proj, u_room, wgs, jobs(rb), 256, rb); }
  // t1: a k-tile's time; wgs: consumers
  double us(int rb, int wn, int s, double t1, int64_t wgs) const {
    const bool alone = mid_alone(rb);
    t1 *= (double)((ktiles(wn) + s - 1) / s);
    const double t2 = 1.827 * t1;
    double fill;
    if (wgs <= 256) {
      fill = t1 * (wgs > 128 ? 1.0 + 0.066 * (double)(wgs - 128) / 128.0 : 1.0);
    } else {
      const int64_t left = wgs % 512;
      fill = (double)(wgs / 512) * (t2 + 2.172);
      if (left > 0) fill += 2.172 + 1.066 * t1 + (t2 - 1.066 * t1) * up_to_1((double)(left - 256) / c.ramp);
    }
    const double fabric = (2.0 * cols * Kc * (1.0 + c.again * (double)(tiles_m(rb) - 1)) + 16.0 * T * Kc / s) / c.rate;
    const double loop = cbrt(fill * fill * fill + fabric * fabric * fabric);
    double us = 7.687 + loop + (alone ? 1.65 + 0.229 * rb : 0.0);     // (alone: nothing else runs on the unit while a tile starts and ends)
    if (lora.n > 0) {
      // (the most u there can be, of five projections and more, counts as whole: the estimate of such calls is low, and with
      // two pieces would take six of 1024 columns, contraction 14336, 1000 rows of rank 128, here, 496 us, not one by one, 298)
      const int p = pieces(rb, wgs, MID_U_FLOATS / 2);
      const int64_t with_rows = (int64_t)(0.6 * T) + 1 < lora.n ? (int64_t)(0.6 * T) + 1 : lora.n;      // (adapters, about)
      const int64_t prods = n_proj * p * (with_rows * (lora.tiles / lora.n > 1 ? lora.tiles / lora.n : 1) + T / (16 * rb) * ((rb + 1) / 2));
      // (the expand of more ranks is not proportionally more: 184 rows, 1872 x 8368, rank 32, 23.1 -> 22.1 us
      // in tiles of 128 columns; a split makes every rank's u travel to more readers: 277 rows, 2144 x 1048, rank 64,
      // 20.0 -> 18.4 unsplit)
      const double rank = std::min(c.rank_cap, (double)lora.ranks / lora.n);
      const double prod_us = 10.735 * Kc / 4096.0 / p + 0.498;
      us += 0.562 + 2.009 * ((rb * wn + 7) / 8) * rank / 16.0 + (s > 1 ? 0.02 * lora.ranks / lora.n : 0.0);
      if (alone) {
        // As the launch has them (launch_mid): the jobs that there can be, each first on a unit of its own, a round of units after
        // another, or in turn on the units that the consumers leave.  Those that no grouping of these rows has look for themselves.
        const int64_t padded = (jobs(rb) * p + 7) / 8 * 8, free = mid_free_units(256, wgs);
        const double real = (double)std::min(prods, padded), none = (double)padded - real;
        if (mid_jobs_in_turn(free, padded)) us += std::max(0.0, prod_us * real / (double)free + 5.39 * none / (double)free - 1.776 * loop);
        else us += prod_us * 0.743 * (up_to_1(((double)wgs + real - 256.0) / 17.45) + std::max(0.0, ceil(((double)wgs + real) / 256.0) - 2.0)) + 5.39 * none / 256.0;
      } else {
        us += prod_us * (wgs <= 256 ? 0.574 * up_to_1((double)(wgs + prods - 256) / 17.45) : 0.289 * up_to_1((double)prods / 256.0) * (256.0 / c.beside));
        us += prod_us * 0.918 * up_to_1((double)((wgs < 512 ? wgs : 512) + prods - 512) / 17.45);
      }
    }
    if (s > 1) us += (lora.n > 0 ? 0.0 : 1.5) + (s > 2 ? 2.442 : 2.257) * (0.5 + rb * wn / 32.0) + (wgs > 192 ? 0.186 * (double)(wgs - 192) / 64.0 : 0.0);
    return us;
  }
};

// Of the smaller tiles.  Without adapters the workgroups count as the fullest XCD has them (1.006 times the best on the average,
// 1.017 as they are); with adapters that is no better.
inline MidPlan mid_plan(int64_t T, int64_t Kc, const ProjEntry* proj, int n_proj, const MidLora& lora, int max_split) {
  const MidModel m(T, Kc, proj, n_proj, lora, MID_SMALL);
  MidPlan best;
  for (int wn = 2; wn <= 4; wn += 2)
    for (int rb = 4; rb <= 5; ++rb)
      for (int s = 1; s <= max_split; s *= 2) {
        const int64_t wgs = m.tiles_m(rb) * m.tiles_n(wn) * s;
        if (s > 1 && (wgs > MID_SPLIT_WGS || m.ktiles(wn) < 4 * s)) continue;
        const int64_t units = lora.n > 0 ? wgs : m.tiles_m(rb) * m.over_xcds(wn, s);
        const double us = m.us(rb, wn, s, mid_tile_us[rb - 4][wn == 4], units);
        if (best.rb == 0 || us < best.us) { best.us = us; best.rb = rb; best.wn = wn; best.ksplit = s; best.tiles_m = (int)m.tiles_m(rb); }
      }
  return best;
}

// The estimate from which on the call is better off elsewhere (ext: ranks of all adapters in the batch, 0: no adapters).
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
inline double mid_limit(int64_t T, int64_t Kc, int64_t cols, int ext, Wide wide_us) {
  const double always = 1e30;
  if (T <= 32) return T * Kc > 140000 || Kc * cols > 50000000 ? always : 0.0;
  if (T > 384 && ext > 0) return 20.0 + 2.0 * T * Kc * cols / 1.25e9 + 0.1 * ext;
  if (T > 384) return (6.0 + wide_us()) / (Kc > 4096 ? 1.0 + 0.2 * log2((double)Kc / 4096.0) : 1.0);
  if (T > 64 && T <= 256 && Kc >= 2 * cols && Kc * cols >= 40000000) {
    if (ext == 0) return 15.0 + Kc * cols * (T <= 128 ? 0.29e-6 : 0.365e-6);
    if (T > 128 && ext <= 512) return (15.0 + Kc * cols * 0.67e-6) / 1.15;
  }
  return always;
}

// The same call in taller tiles of 128 columns, unsplit, where the estimate says that they are faster: than the smaller tile, or,
// where that one does not pay (limit), than the kernel that has the call otherwise.
//   Both sides are estimated with other constants than the smaller tiles have among themselves, fitted to 1758 sets of 33 to 1024
// rows, contractions of 1024 to 14336, 1024 to 28672 columns in one or three projections, without adapters and with up to 400 of
// ranks 8 to 128, timed as they run without taller tiles and in every taller one that fits, with the weight from the memory-side
// cache and from memory, neither of which is to get slower.  Of these and 390 timed afterwards, 2148, 555 change, 500 of them get faster by
// more than 3 % in both, 29 slower in one of the two by more than 1 %, the worst by 20 (tests/golden/tall_tilings.json has 748 of them).
//   96 rows only with all workgroups on the chip at once (669 rows, 6168 x 2248, 32 adapters of rank 64, would be 1.34 times as
// long), 128, 160 and 256 rows where they fill one round and most of the units (512 rows, 5120 x 5120, 160 workgroups of 128 rows: 56.7
// us, 240 of 96 rows 52.4).  Contractions of a few k-tiles are over before a tile
// alone on its unit has started (310 rows, 1608 x 15520, 31.4 -> 35.5 us in tiles of 160 rows; 386 rows, 1280 x 13720, 23.6 -> 26.9
// in tiles of 256; 514 rows, 2400 x 10240, 52.5 and 58.1), and tall tiles win most where the weight comes from memory (362 rows, 2808 x
// 9952, in tiles of 128: from memory 47.3 -> 42.7, from the cache 36.2 -> 40.8): hence the least contractions and a tenth in hand.
//   96 rows whose jobs are whole because two pieces would be a few more workgroups than fit (whole): the smaller tile has its jobs in two
// there, and how long whole ones take is not in the estimate, so 7 % more are asked for, and no more than 20 steps a wave.  46 sizes of such
// calls, from the cache and from memory 0.845 and 0.852 of the time without, at most 1.04 (512 rows, 5120 x 5120, 64 adapters of rank 32,
// 55.2 -> 47.6 us); 17 sizes beyond these lines 0.67 to 1.19 (736 rows, 5176 x 2440, 20 adapters of rank 64, 65.9 -> 78.4).
inline MidPlan mid_taller(const MidPlan& p, int64_t T, int64_t Kc, const ProjEntry* proj, int n_proj, const MidLora& lora, double limit = 1e30) {
  static const int rbs[4] = {6, 8, 10, 16};
  static const double tile_us[4] = {0.320, 0.333, 0.378, 0.650};
  static const int least_k[4] = {1400, 2600, 3200, 3000};
  MidPlan best = p.us < limit ? p : MidPlan();
  if (best.rb == 0 && T <= 384) return best;
  const MidModel m(T, Kc, proj, n_proj, lora, MID_TALL);
  double least = 0.0;                                            // (0: not asked for yet)
  const int64_t steps = ((Kc + 31) / 32 + MID_WAVES - 1) / MID_WAVES;
  for (int i = 0; i < 4; ++i) {
    const int rb = rbs[i];
    const int64_t wgs = m.tiles_m(rb) * m.over_xcds(4, 1);
    if (Kc < least_k[i] || wgs < 176 || (mid_alone(rb) ? wgs > 256 : wgs + m.jobs(rb) * m.pieces(rb, wgs, MID_U_FLOATS) > 512)) continue;
    if (least == 0.0)
      least = p.us < limit ? 0.9 * m.us(p.rb, p.wn, p.ksplit, mid_tile_us[p.rb - 4][p.wn == 4], m.tiles_m(p.rb) * m.over_xcds(p.wn, p.ksplit))
                           : (lora.n == 0 ? 0.85 : n_proj == 1 ? 1.0 : 1.2) * limit;
    const bool whole = rb == 6 && steps > 8 && m.pieces(rb, wgs, MID_U_FLOATS) == 1 && wgs + m.jobs(rb) > 256 && wgs + 2 * m.jobs(rb) <= 576;
    if (whole && steps > 20) continue;
    const double us = m.us(rb, 4, 1, tile_us[i], wgs);
    if (us < (whole ? 0.93 : 1.0) * least) { least = us; best.us = std::min(p.us, us); best.rb = rb; best.wn = 4; best.ksplit = 1; best.tiles_m = (int)m.tiles_m(rb); }
  }
  return best;
}

}  // namespace marlaas
