// Host-side rules of forward/backward: the size of the GEMM tiles, how the backward launch is dealt to
// workgroups, and the scratch that follows from it.  Plain C++, so that the rules can be checked on the
// CPU over everything that the entry points accept.
#pragma once

#include <limits.h>
#include <stdint.h>

#include <algorithm>

namespace pfc {

// ---------------------------------------------------------------------------------------------
// Padded problem geometry.  Every scratch operand of the three GEMMs is padded with zeros to a
// whole number of tiles, so the GEMM main loops need no bounds checks.
// ---------------------------------------------------------------------------------------------
constexpr int kPadB = 256;   // batch rows are padded to at most a multiple of this
constexpr int kPadD = 128;   // row length of the GEMM operands
constexpr int kPadK = 256;   // sampled rows are padded to a multiple of this
constexpr int kMaxSplits = 32;    // slices of S in the dfeatures product (long fp32 sums: twice that)

inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }

// Number of batch slices of the dweight GEMM (1: none): slices only when the tiles alone leave
// most CUs idle, limited by the room in the split buffer and by a minimum slice length.
inline int dweight_slices(int cu, int tiles, int Bp, int64_t kp, int bk) {
  const int slabs_total = Bp / bk;
  int want = cu / tiles;
  const int64_t room = (int64_t)kMaxSplits * Bp / kp;
  if (want > room) want = (int)room;
  if (want > slabs_total / 8) want = slabs_total / 8;   // a slice must stay long enough to pay
                                                        // for its own partial tile
  return want < 1 ? 1 : want;
}

// Geometry of the tiles: reduction steps of a slab.
inline int tile_bk(int es) { return 128 / es; }

// Whether the one-kernel form of the fused call takes the class set: its tile (128 classes x 512
// columns) spans the rows, and there is at least one for every compute unit.
inline bool fits_one_kernel(int cu, int D, int64_t kp) { return D == 512 && kp / 128 >= cu; }

// ---------------------------------------------------------------------------------------------
// Large batches: 256-tiles, one workgroup to a compute unit, and both reductions so long that the
// slices decide how evenly the launch ends.  With slices by number alone (dfeatures half of the
// GPU, the batch cut only below one tile for every compute unit) 4096 samples x 20,000 classes x
// 512 in bf16 made 128 workgroups of 79 slabs and 158 of 64: 286 on 256 compute units, two rounds.
// ---------------------------------------------------------------------------------------------
constexpr int kLongBatch = 2048;      // up to here slices are short and the rules below measured no slower
constexpr int kLongRoom = 3;          // partial tiles of either product for every compute unit, at most
constexpr int kMaxLongSplits = 16;    // slices of the classes
constexpr int kPlainSum = 2048, kMaxPlainSum = 4096;   // products of one fp32 sum without pieces: where
                                                       // the room allows it / at most

// Slabs until the last compute unit is done: `na` workgroups of `a` slabs each, then `nb` of `b` <= a,
// each to the compute unit that is free first.
inline int64_t launch_slabs(int64_t cu, int64_t na, int64_t a, int64_t nb, int64_t b) {
  const int64_t late = na % cu, t0 = na / cu * a, t1 = t0 + a;   // cu - late are free at t0, late at t1
  auto room = [&](int64_t t) {
    return (cu - late) * ((t - t0) / b) + (t >= t1 ? late * ((t - t1) / b) : 0);
  };
  int64_t end = late ? t1 : t0;
  if (nb == 0 || room(end) >= nb) return end;   // b <= a: whatever ends by t1 fits in front of it
  // the end is t0 or t1 plus whole workgroups; no earlier than the mean
  const int64_t mean = (na * a + nb * b + cu - 1) / cu;
  int64_t i0 = std::max<int64_t>((mean - t0) / b, 0), i1 = std::max<int64_t>((mean - t1) / b, 0);
  for (;;) {
    const int64_t e0 = t0 + i0 * b, e1 = t1 + i1 * b;
    const bool first = !late || e0 <= e1;
    const int64_t t = first ? e0 : e1;
    if (t >= end && room(t) >= nb) return t;
    ++(first ? i0 : i1);
  }
}

// Whether there is room for fp32 sums of at most `most` products.
inline bool plain_sums_fit(int cu, int Bp, int Dp, int64_t kp, int most) {
  const int64_t w = (Bp + most - 1) / most, x = (kp + most - 1) / most;
  const int64_t tiles_w = kp / 256 * (Dp / 256), tiles_x = (int64_t)(Bp / 256) * (Dp / 256);
  const int64_t room = (int64_t)kLongRoom * cu;
  return w <= kMaxSplits && x <= kMaxLongSplits &&
         (w == 1 || (w * tiles_w <= room && w * kp <= (int64_t)kMaxSplits * Bp)) &&
         (x == 1 || x * tiles_x <= room);
}

// Slices of the classes (dfeatures) and of the batch (dweight), and which product's workgroups
// start first.
struct LongSlices {
  int dx, dw;
  bool dw_first;
  bool even;   // the launch ends at most a fifth later than with the slabs spread over all compute units
};

// The fewest microseconds by an estimate: a slab of a 256-tile takes 1.45 us (bf16; start and end
// of a workgroup like 10 slabs) or 7.7 us (fp32, 2 slabs), a partial tile of dfeatures 0.06 us to
// add up later, one of dweight 0.05, the result likewise, and the launch that does it 3 us.  Fitted
// to 45 forms of 2,100 .. 65,536 samples, 2,000 .. 30,000 classes, D 128 .. 1024 and all slices
// that fit (7,730 measurements): the pick is 0.5 % behind the best of a form on average, 3 % at
// most.  Against the rules for smaller batches (us, both products):
//   bf16 4096 x 20,000 x 512 217 -> 179, 3000 x 20,000 x 512 166 -> 136, 8192 x 20,000 x 512 423 ->
//     315, 4096 x 20,000 x 1024 338 -> 304, 16,384 x 3,592 x 512 141 -> 130
// fp32: the weights are those of fp32 MFMAs.  A slab of planes takes 3.2 us, and with that (and 4
// slabs for start and end) the pick has up to half the slices, forward/backward 0 - 6 % shorter
// (4774 x 8,175 x 256 504 -> 477 us, 8794 x 6,171 x 192 567 -> 559), but sums twice as long
// (dweight at scale 1, off 64 bits: 3.9e-7 -> 5.5e-7, 4.2e-7 -> 5.9e-7): the slices stay as they
// are.  fp32 sums run without pieces here: only slices of at most kPlainSum products are taken, or
// kMaxPlainSum where those do not fit (the caller sees to it that there are such).  Error against
// 64 bits, 2-norm, both gradients, slices by number alone -> now: 16,384 x 15,700 x 512 7.6e-7 ->
// 6.2e-7, 8192 x 8,100 x 512 7.7e-7 -> 6.9e-7, 4096 x 8,000 x 1024 3.3e-7 -> 2.9e-7.
inline LongSlices long_batch_slices(int cu, int es, int Bp, int Dp, int64_t kp) {
  const int bk = tile_bk(es);
  const int slabs_w = Bp / bk, slabs_x = (int)(kp / bk);
  const int64_t tiles_w = kp / 256 * (Dp / 256), tiles_x = (int64_t)(Bp / 256) * (Dp / 256);
  const int64_t room = (int64_t)kLongRoom * cu, edge = es == 2 ? 10 : 2;
  const int most = es == 2 ? INT_MAX : plain_sums_fit(cu, Bp, Dp, kp, kPlainSum) ? kPlainSum : kMaxPlainSum;
  const double slab_us = es == 2 ? 1.45 : 7.7, dw_tile_us = 0.05, dx_tile_us = 0.06;
  const int64_t work = tiles_w * slabs_w + tiles_x * slabs_x;
  LongSlices best = {0, 0, false, false};
  double best_us = 0;
  for (int w = 1; w <= kMaxSplits && w * 8 <= slabs_w; ++w) {
    if (w > 1 && (w * tiles_w > room || w * kp > (int64_t)kMaxSplits * Bp)) break;
    const int per_w = (slabs_w + w - 1) / w, n_w = (slabs_w + per_w - 1) / per_w;
    if (n_w != w || per_w * bk > most) continue;
    for (int x = 1; x <= kMaxLongSplits && (x == 1 || x * 4 <= slabs_x); ++x) {
      if (x > 1 && x * tiles_x > room) break;
      const int per_x = (slabs_x + x - 1) / x, n_x = (slabs_x + per_x - 1) / per_x;
      if (n_x != x || (int64_t)per_x * bk > most) continue;
      const bool dw_first = per_w > per_x;
      const int64_t slabs = dw_first ? launch_slabs(cu, w * tiles_w, per_w + edge, x * tiles_x, per_x + edge)
                                     : launch_slabs(cu, x * tiles_x, per_x + edge, w * tiles_w, per_w + edge);
      const double us = slab_us * slabs + dx_tile_us * x * tiles_x +
                        (w > 1 ? dw_tile_us * (w + 1) * tiles_w + 3.0 : 0.0);
      if (best.dw == 0 || us < best_us) {
        best = {x, w, dw_first, (slabs - edge) * cu * 5 <= work * 6};
        best_us = us;
      }
    }
  }
  return best;
}

// Whether the backward launch of the call takes them, given 256-tiles.  Not the class sets of the
// one-kernel form, whose dX has the same bits in either call and whose many tiles come out even.
inline bool long_batch(int cu, int D, int Bp, int64_t kp) { return Bp > kLongBatch && !fits_one_kernel(cu, D, kp); }

// How the rows of W and v are loaded, for what the memory-side cache (256 MB) still holds when they are
// next read; their stores are always nontemporal.  A row that is loaded plainly goes to that cache, is
// stored back to it, and leaves it for memory while the next kernels run.
//   gather_plain: the sampled rows of W stay from the gather to the update.
//   resident: W and v as a whole may stay from step to step: the update loads both plainly.
//   reused:   after a plain gather the update loads nontemporally: the rows' last use in the step.
//   streamed: nontemporal, but for v in the update.
// The batch is the context's largest, so that gather and update, which are calls of their own, decide
// alike.  The one-kernel form loads nontemporally in either place.
// Between two steps a program runs its backbone, which leaves the cache full of other, partly dirty
// data: what a plain gather brings in has to push that out first.  Step, us, in the order gather
// nontemporal and update plain / streamed / reused / resident with a plain gather, (a) steps one right
// after the other, (b) behind an in-place pass over 512 MB, (c) behind a copy of as much, (d) behind eight
// bf16 products of 2048 x 4096 x 4096 (bytes of the step as counted below):
//   256 x 25,724 of 85,742 x 128 (47 MB)   (a) 59.8 / 60.1 / 60.5 / 58.2   (b) 71.4 / 70.8 / 70.7 / 70.8
//                                          (c) 68.6 / 68.2 / 68.0 / 67.4   (d) 67.4 / 67.0 / 67.7 / 67.2
//   512 x 9,344 of 93,431 x 512 (66)       (a) 81.9 / 81.3 / 81.5 / 81.9   (b) 90.9 / 90.9 / 91.3 / 91.4
//   700 x 8,000 of 40,000 x 512 (64)       (a) 84.6 / 85.4 / 85.6 / 83.6   (b) 94.9 / 94.3 / 93.5 / 93.7
//   1024 x 18,000 of 90,000 x 256 (91)     (a) 109.9 / 109.0 / 108.4 / 107.5   (b) 119.4 / 118.9 / 118.4 / 118.7
//                                          (c) 116.9 / 117.4 / 113.8 / 113.9   (d) 116.7 / 116.7 / 116.0 / 115.9
//   512 x 16,000 of 40,000 x 512 (107)     (a) 107.5 / 108.8 / 108.8 / 106.9   (b) 118.3 / 117.5 / 121.3 / 121.2
//                                          (c) 113.9 / 114.1 / 115.9 / 116.3   (d) 116.0 / 115.6 / 115.4 / 116.8
//   512 x 18,000 of 300,000 x 512 (119)    (a) 126.3 / 123.5 / 121.9   (b) 136.1 / 135.8 / 139.5
//                                          (c) 130.3 / 131.5 / 133.9   (d) 129.7 / 129.7 / 134.1
//   512 x 30,000 of 300,000 x 512 (193)    (a) 177 / 169 / 167   (b) 190 / 190 / 198   (c) 177 / 179 / 183
//                                          (d) 177 / 177 / 182
//   768 x 20,599 of 205,990 x 1024 (268)   (a) 254 / 247 / 238   (b) 260 / 263 / 279   (c) 248 / 250 / 257
//   1024 x 205,991 of 2,059,906 x 512      (a) 1204 / 1195 / 1202   (b) 1204 / 1192 / 1242   (c) 1178 / 1173 / 1222
// From 107 MB on a plain gather is up to 9 % behind there (64 x 20,000 x 1024 behind layers with weights of their
// own 163 / 178; a state's first step 5 - 7 %: 512 x 30,000 203 / 214, 109 x 17,766 x 768 154 / 163), whatever it
// gains where steps follow each other (1 - 6 %: the last form 123 / 118); up to 91 MB it is even or ahead.  Hence
// the line at 95 MB between them.  (Streamed is up to 2 % behind the first order in (b) and (c) from 200 to 270 MB, 2 - 5 % ahead in
// (a), and ahead everywhere in larger steps.)  The shorter the rows, the less a plain gather loses behind other
// data and the more it gains in a row; at D = 64, rows of two cache lines, it is ahead in nearly all (streamed / reused):
//   67 x 78,698 of 430,107 x 128 (112 MB)  (a) 108.4 / 105.3   (b) 120.1 / 124.1   (c) 116.5 / 117.3   (d) 115.6 / 115.8
//   128 x 120,000 of 1,200,000 x 128 (185) (a) 146.6 / 142.2   (b) 163.0 / 167.4   (c) 151.9 / 154.8   (d) 153.3 / 157.3
//   100 x 150,000 of 1,500,000 x 64 (145)  (a) 134.6 / 130.5   (b) 163.6 / 159.4   (c) 144.0 / 143.3   (d) 146.3 / 149.3
//   64 x 200,000 of 2,000,000 x 64 (179)   (a) 167.5 / 162.6   (b) 207.3 / 202.2   (c) 175.5 / 174.4   (d) 177.4 / 170.6
//   100 x 200,000 of 200,000 x 64 (194)    (a) 150.2 / 149.8   (b) 190.4 / 177.0   (c) 167.2 / 165.8   (d) 163.0 / 162.6
//   900 x 80,000 of 800,000 x 64 (207)     (a) 170.5 / 168.4   (b) 196.8 / 197.0   (c) 179.9 / 178.8   (d) 178.3 / 178.9
// There the line is at 215 MB.
enum RowLoads { ROWS_RESIDENT, ROWS_REUSED, ROWS_STREAMED };
constexpr int64_t kResidentBytes = 200000000, kGatherPlainBytes = 95000000, kGatherPlainBytes64 = 215000000;
struct RowPolicy {
  RowLoads loads;
  bool gather_plain;
};
inline RowPolicy row_policy(int es, int64_t N, int D, int B_max, int64_t k) {
  // W's rows, dWn, Wn, E; features, their gradient and its partial sums, about eight rows of floats a sample
  const int64_t step = k * (8ll * D + es * (round_up(D, kPadD) + B_max)) + 32ll * B_max * D;
  const bool plain = step <= (D == 64 ? kGatherPlainBytes64 : kGatherPlainBytes);
  return {8 * N * D <= kResidentBytes ? ROWS_RESIDENT : plain ? ROWS_REUSED : ROWS_STREAMED, plain};
}

// Size of the GEMM tiles, one for the logits and one for the backward launch of a call.  256 x 256
// moves the least data per flop and fills a compute unit with one workgroup, 128 x 128 puts two on
// it, 64 x 64 three.  Measured on 256 compute units over batches of 48 .. 16,384 samples and 320 ..
// 2 million classes (us for 256 / 128 / 64, D = 512 unless stated):
//   bf16 logits: a round of 256-tiles costs the same however full it is, so they win only where the
//     last round is nearly full (1024 x 205,991: 336 / 347 / 507; 768 x 20,599 x D 1024, 0.95 of a
//     round: 41 / 45 / 64; 1024 x 36,024, 2.2 rounds: 71 / 58 / 83) and the reduction is long (8192
//     x 6,000 x D 256: 71 / 65 / 102); 64-tiles only for a handful of 128-tiles (512 x 4,000: 24 /
//     9.8 / 8.7; 512 x 9,344: 24 / 14.7 / 16.0).
//   bf16 backward: 256-tiles unless they leave compute units idle (512 x 4,000: 22 / 15 / 17; 512 x
//     16,000: 29 / 30 / 45; 1024 x 205,991: 482 / 612 / 996), the batch would be padded much more
//     (128 x 200,000: 210 / 179 / 260) or the reduction is short and the tiles few (256 x 36,000:
//     42 / 39 / 57; 256 x 200,000: 221 / 260 / 368); 64-tiles for the smallest problems (128 x
//     1,000: 15 / 7.3 / 5.8).
//   fp32 logits: the fp32 matrix instruction is the bound at any of the sizes, so what counts is
//     how evenly the compute units are loaded: 64-tiles where a few 128-tiles per compute unit do
//     not come out even (512 x 9,344: 135 / 77 / 57; 128 x 1,000: 129 / 37 / 15).  From one
//     256-tile per compute unit on the sizes are close (2048 x 60,000: 1144 / 1127 / 1207; 512 x
//     60,000: 299 / 315 / 330) and the logits keep 256 and its order of the row sums.
//   fp32 backward: by estimate.  A compute unit full of tiles of one size takes fp32_slab_us for a
//     slab of 32 steps of one tile: a 256-tile reads the least from LDS and splits the fewest
//     values for every product, smaller ones come out more even.  Forward/backward with the
//     backward launch in 64 / 128: 133 x 3,266 x 128 31.5 / 37.7, 63 x 26,135 x 192 58 / 81, 512 x
//     9,344 x 512 143 / 145, 340 x 31,475 x 512 325 / 290, 359 x 9,894 x 896 200 / 185, 879 x
//     12,433 x 192 164 / 144, 2071 x 4,867 x 64 127 / 100, 4096 x 8,000 x 320 575 / 514; 64 / 128 /
//     256: 3000 x 8,000 x 512 661 / 581 / 546, 4096 x 20,000 x 512 1874 / 1675 / 1515, 16,384 x
//     3,000 x 512 1274 / 1220 / 963.  In 40 forms drawn from 48 .. 4096 samples, 1,000 .. 60,000
//     classes and all D the pick is within 2 % of the better of 64 and 128, but for 1757 x 17,102 x
//     64 (219 / 250).
enum TileSize { TILES_64 = 64, TILES_128 = 128, TILES_256 = 256 };

// fp32: microseconds a compute unit takes for one slab of one tile, full of tiles of that size.
inline double fp32_slab_us(TileSize t) { return t == TILES_256 ? 3.2 : t == TILES_128 ? 0.98 : 0.36; }

inline bool even_rounds(int64_t tiles, int64_t cu) {   // at most 15 % of the rounds' room is idle
  return tiles > 4 * cu || (tiles + cu - 1) / cu * cu * 100 <= tiles * 115;
}

inline TileSize logits_tiles(int64_t cu, int es, int B, int64_t kp, int D) {
  const int64_t mid = kp / 128 * ((B + 127) / 128);
  const int64_t big = kp / 256 * ((B + 255) / 256), rounds = (big + cu - 1) / cu;
  if (es == 4) return big >= cu ? TILES_256 : even_rounds(mid, cu) ? TILES_128 : TILES_64;
  if (D > 256 && rounds * cu * 4 * 100 <= mid * 109) return TILES_256;
  return 2 * mid > cu ? TILES_128 : TILES_64;
}

// Whether the fp32 logits take tiles of 64 classes x 16 samples where the rule above says 64-tiles: as
// long as these occupy half of the compute units at most.  Forward/backward, us, 64-tiles / slim ones:
// 32 tiles (128 x 1,000 x 512) 36.0 / 30.8, 96 (100 x 3,000 x 1024) 63.3 / 58.6, 128 (128 x 4,000 x 512)
// 49.6 / 47.6, 160 (64 x 10,000 x 256) 41.1 / 43.1, 256 (256 x 4,000 x 512) 55.0 / 62.1.
inline bool logits_slim(int64_t cu, int B, int64_t kp) { return kp / 64 * ((B + 63) / 64) * 2 <= cu; }

// Workgroups that a compute unit holds.
inline int tiles_per_cu(TileSize t, int es) {
  return t == TILES_256 ? 1 : t == TILES_128 ? 2 : es == 2 ? 3 : 4;
}

// The dfeatures product: slices of S, and workgroups of one tile and slice each.
struct DxShape {
  int slabs_total, slabs_per, splits, tiles_i, tiles_d;
  int wgs;   // workgroups: tiles_i * tiles_d * splits, rounded up to 8
};

// `want` slices of the classes, at least one slab each.
inline DxShape dx_cut(int es, TileSize t, int Bp, int Dp, int64_t kp, int64_t want) {
  DxShape dx;
  dx.tiles_i = Bp / t;
  dx.tiles_d = Dp / t;
  dx.slabs_total = (int)(kp / tile_bk(es));
  dx.slabs_per = (int)((dx.slabs_total + want - 1) / want);
  dx.splits = (dx.slabs_total + dx.slabs_per - 1) / dx.slabs_per;
  dx.wgs = (int)round_up((int64_t)dx.tiles_i * dx.tiles_d * dx.splits, 8);
  return dx;
}

// About `wgs` workgroups, at least 4 slabs each.  The callers ask
// for half of what the GPU holds at a time, or for all the room that the dweight tiles leave:
// measured against all of it and a quarter of it (us a step, quarter / half / all):
// 1024 samples x 205,991 classes x 512 1499 / 1302 / 1365, x 360,232 2511 / 2166 / 2251, fused
// x 205,991 1162 / 1098 / 1161.  Fewer workgroups write fewer partial sums (2 MB a slice there)
// but are longer than everything behind them.
inline DxShape dx_shape(int cu, int es, TileSize t, int Bp, int Dp, int D, int64_t kp, int64_t wgs) {
  const int slabs_total = (int)(kp / tile_bk(es));
  int64_t want = wgs / ((int64_t)(Bp / t) * (Dp / t));
  // fp32 sums that are not cut into pieces: slices of more than 4096 classes are halved, for the
  // rounding of the sums (100 samples x 400,000 classes dX 2.81e-7 off, halved 2.70e-7) and, fused, for
  // workgroups that are not the end of the launch (4.23 -> 3.18 ms; 512 x 200,000 2.85 -> 2.92)
  const bool halve = es == 4 && fits_one_kernel(cu, D, kp) && kp > (int64_t)kMaxSplits * 4096;
  want = std::min<int64_t>({want, halve ? 2 * kMaxSplits : kMaxSplits, slabs_total / 4});
  return dx_cut(es, t, Bp, Dp, kp, want < 1 ? 1 : want);
}

// bf16: no more slices than `most` has, and as few of them as let the launch end within 2 % of the
// earliest by an estimate: a slab takes a workgroup 0.75 us (128- and 64-tiles; its start and end 6
// slabs) or 1.75 us (256-tiles, 4), a slice of partial sums goes to memory and back.  What this
// avoids is a few workgroups in a round of their own, and partial sums of dfeatures workgroups that
// are shorter than those of dweight.  Forward/backward by the share of the GPU's room that
// dfeatures takes, us, 0.2 / 0.3 / 0.4 / half and more -> taken: 512 samples x 9,344 classes x 512
// 58.2 / 55.0 / 55.6 / 60.8 -> 0.4; 800 x 3,000 x 512 45.1 / 45.8 / 48.3 / 49.0 -> 0.2; 200 x 3,000
// x 768 40.1 / 41.9 / 42.2 / 42.1 -> 0.2; 1700 x 12,547 x 512 176 / 157 / 151 / 150 -> 0.4; 1000 x
// 30,000 x 256 119 / 110 / 112 / 113 -> 0.4; 768 x 20,599 x 1024 191 / 167 / 162 / 163 -> 0.4.
// (More than two rounds of dweight tiles fill every gap: 1024 x 205,991 with 14 slices in place of
// 16 is 1 % slower.)
inline DxShape dx_even(int64_t slots, TileSize t, int Bp, int Dp, int64_t kp, int64_t wgs_w, int slabs_w,
                       const DxShape& most) {
  const int edge = t == TILES_256 ? 4 : 6;
  const double slab_us = t == TILES_256 ? 1.75 : 0.75, slice_us = (double)Bp * Dp * 8 / 3e6;
  auto us = [&](const DxShape& d) {
    const int64_t n = (int64_t)d.tiles_i * d.tiles_d * d.splits;
    const int x = d.slabs_per + edge, w = slabs_w + edge;
    return slab_us * (x >= w ? launch_slabs(slots, n, x, wgs_w, w) : launch_slabs(slots, wgs_w, w, n, x)) +
           slice_us * d.splits;
  };
  double best = us(most);
  for (int pass = 0; pass < 2; ++pass)
    for (int n = 1; n < most.splits; ++n) {
      const DxShape d = dx_cut(2, t, Bp, Dp, kp, n);
      const double d_us = us(d);
      if (pass == 1 && d_us <= 1.02 * best) return d;
      if (d_us < best) best = d_us;
    }
  return most;
}

// Slices of the batch in the dweight product, and the shape of the dfeatures product beside it
// (the same with and without the update, so that dX has the same bits).
struct BackwardShape {
  int slabs_per, splits;   // of the batch
  bool dw_first;           // the dweight workgroups are the longer ones and start first
  DxShape dx;
};
inline BackwardShape backward_shape(int cu, int es, TileSize t, int Bp, int Dp, int D, int64_t kp) {
  BackwardShape s;
  const int tiles_w = (int)(kp / t) * (Dp / t);
  const int slabs_total = Bp / tile_bk(es);
  const LongSlices cut = t == TILES_256 && long_batch(cu, D, Bp, kp) ? long_batch_slices(cu, es, Bp, Dp, kp)
                                                                     : LongSlices{0, 0, false, false};
  const int want = cut.dw ? cut.dw : dweight_slices(cu, tiles_w, Bp, kp, tile_bk(es));
  s.dw_first = cut.dw_first;
  s.slabs_per = (slabs_total + want - 1) / want;
  s.splits = (slabs_total + s.slabs_per - 1) / s.slabs_per;
  if (cut.dw) {
    s.dx = dx_cut(es, t, Bp, Dp, kp, cut.dx);
    return s;
  }
  const int64_t slots = (int64_t)cu * tiles_per_cu(t, es);
  const int64_t wgs_w = (int64_t)tiles_w * s.splits;
  // fp32 tiles take long: dfeatures workgroups no longer than those, so that the end comes out even
  const int64_t wgs = es == 4 && wgs_w > 2 * slots ? 2 * slots : std::max(slots / 2, slots - wgs_w);
  s.dx = dx_shape(cu, es, t, Bp, Dp, D, kp, wgs);
  // (The class sets of the one-kernel form too, whose dfeatures slices are those of the three
  // calls, though its dweight workgroups are of another size: with the slices of the GPU's room ->
  // now, us, 4096 x 33,000 three calls 589 -> 557, fused 610 -> 605; 2048 x 40,000 342 -> 337, 379
  // -> 387; 700 x 34,000 157 -> 158, 191 -> 194; 512 x 50,000 162 -> 163, 218 -> 215; 1024 x 36,024
  // and 1024 x 60,000 even.)
  if (es == 2 && wgs_w <= 2 * slots) s.dx = dx_even(slots, t, Bp, Dp, kp, wgs_w, s.slabs_per, s.dx);
  return s;
}

// Microseconds of the backward launch with fp32 operands, by estimate: the longer workgroups first,
// each to the slot that is free first, 4 slabs for its start and end; partial sums at 5 TB/s.
inline double fp32_backward_us(int cu, TileSize t, int Bp, int Dp, int D, int64_t kp) {
  const BackwardShape s = backward_shape(cu, 4, t, Bp, Dp, D, kp);
  const int per = tiles_per_cu(t, 4), edge = 4, w = s.slabs_per + edge, x = s.dx.slabs_per + edge;
  const int64_t nw = kp / t * (Dp / t) * s.splits, nx = (int64_t)s.dx.tiles_i * s.dx.tiles_d * s.dx.splits;
  const int64_t slabs = w > x ? launch_slabs((int64_t)cu * per, nw, w, nx, x) : launch_slabs((int64_t)cu * per, nx, x, nw, w);
  return (double)slabs * fp32_slab_us(t) * per + 0.8e-6 * s.dx.splits * Bp * Dp +
         (s.splits > 1 ? 3.0 + 0.8e-6 * (s.splits + 1) * kp * Dp : 0.0);
}

// Microseconds of the backward launch with bf16 operands, by estimate (up to kLongBatch samples): a slab
// takes a workgroup 1.75, 0.8 (0.95 in more than one round of workgroups) or 0.55 us, its start and end
// 4, 8 or 10 slabs; partial sums are written and read.
inline double bf16_backward_us(int cu, TileSize t, int B, int64_t kp, int D) {
  const int Bp = (int)round_up(B, std::max<int>(t, logits_tiles(cu, 2, B, kp, D)));
  const int Dp = (int)round_up(D, t == TILES_256 ? 256 : kPadD);
  const BackwardShape s = backward_shape(cu, 2, t, Bp, Dp, D, kp);
  const int edge = t == TILES_256 ? 4 : t == TILES_128 ? 8 : 10, w = s.slabs_per + edge, x = s.dx.slabs_per + edge;
  const int64_t slots = (int64_t)cu * tiles_per_cu(t, 2);
  const int64_t nw = kp / t * (Dp / t) * s.splits, nx = (int64_t)s.dx.tiles_i * s.dx.tiles_d * s.dx.splits;
  const bool one = nw + nx <= slots;
  const double slab_us = t == TILES_256 ? 1.75 : t == TILES_128 ? (one ? 0.8 : 0.95) : 0.55;
  const int64_t slabs = w > x ? launch_slabs(slots, nw, w, nx, x) : launch_slabs(slots, nx, x, nw, w);
  return (double)slabs * slab_us + 2.4e-6 * s.dx.splits * Bp * Dp + (s.splits > 1 ? 3.0 + 2.4e-6 * s.splits * kp * Dp : 0.0);
}

inline TileSize backward_tiles(int cu, int es, int B, int64_t kp, int D) {
  const int Bp = (int)round_up(B, 128), Bp256 = (int)round_up(B, 256);
  const int Dp = (int)round_up(D, kPadD), Dp256 = (int)round_up(D, 256);
  const int64_t mid = kp / 128 * (Dp / 128), big = kp / 256 * (Dp256 / 256);
  if (es == 4) {
    // The launch that ends first by estimate; 64-tiles are no tiles of the one-kernel form.
    // 256-tiles add up without pieces, which for the same slices is less exact, so only batches
    // that fill them and whose slices end evenly take them, and never batches up to kLongBatch.
    // (dweight at scale 1 off 64 bits, 2-norm, and forward/backward in us, with 256-tiles wherever
    // their estimate is the lowest -> now: 3864 x 29,707 x 1024 9.7e-7 -> 3.6e-7, 4380 -> 4840;
    // 4096 x 8,000 x 320 6.8e-7 -> 3.4e-7, 492 -> 514; 2048 x 16,000 x 512 5.0e-7 -> 3.6e-7, 642 ->
    // 670; 4096 x 33,000 x 64 9.1e-7 -> 2.7e-7, 1079 -> 854.)
    TileSize best = TILES_128;
    double best_us = fp32_backward_us(cu, TILES_128, Bp, Dp, D, kp);
    auto take = [&](TileSize t, double us) {
      if (us < best_us) best = t, best_us = us;
    };
    if (!fits_one_kernel(cu, D, kp)) {
      take(TILES_64, fp32_backward_us(cu, TILES_64, (int)round_up(B, logits_tiles(cu, es, B, kp, D)), Dp, D, kp));
      if (long_batch(cu, D, Bp256, kp) && Dp256 * 100 <= Dp * 115 && Bp256 * 100 <= B * 105 &&
          plain_sums_fit(cu, Bp256, Dp256, kp, kMaxPlainSum) && long_batch_slices(cu, es, Bp256, Dp256, kp).even)
        take(TILES_256, fp32_backward_us(cu, TILES_256, Bp256, Dp256, D, kp));
    }
    return best;
  }
  // (columns: 640 -> 768 and 896 -> 1024 cost less than the smaller tile, 384 -> 512 more)
  const bool fill = Dp256 * 100 <= Dp * 125 && Bp256 * 100 <= Bp * 115 &&
                    big * dweight_slices(cu, (int)big, Bp256, kp, 64) * 2 >= cu && (B >= 512 || big * 2 >= cu * 3);
  const TileSize usual = fill ? TILES_256 : B > 128 || 2 * mid > cu ? TILES_128 : TILES_64;
  // Another size where an estimate of the launch is 6 % lower: a launch of one to three rounds ends
  // with its last workgroup, which the number of tiles alone does not tell.  Step, us, by number / now:
  // 1106 x 5,673 x 1024 163 / 139 (128), 1359 x 7,578 x 512 134 / 118 (128), 1891 x 15,915 x 448 217 / 204
  // (128), 913 x 4,403 x 384 72 / 65 (64), 1018 x 12,161 x 128 73 / 66 (64), 153 x 4,761 x 64 42 / 39 (64),
  // 484 x 24,076 x 768 203 / 191 (256).  In 88 forms drawn from 50 .. 2048 samples, 1,000 .. 60,000 classes
  // and all D that change to a smaller size the step is 3.9 % shorter on average; 128 -> 64 costs up to 3.7 %
  // (790 x 2,932 x 448 58.2 / 60.4) around 800 samples of 3,000 classes, where it is 2.7 % shorter on average.
  // 256-tiles that the number does not suggest only where D is whole tiles of columns: 21 forms, 0.4 %
  // shorter on average, 3.7 % longer at most (570 x 25,793 x 1024 290 / 301).  24 forms with other D were 3.8 %
  // longer on average, up to 8 %, whatever the estimate (187 x 29,073 x 576 152 / 164, 474 x 18,827 x 896
  // 183 / 196, 531 x 51,903 x 448 275 / 289): beyond 512 their rows get longer, which the launches around pay
  // for as well.
  // (Where 256-tiles of dweight alone are half a round or more, they stay: 1756 x 27,321 x 512 286 / 297.)
  if (B > kLongBatch || fits_one_kernel(cu, D, kp) || (usual == TILES_256 && big * 2 > cu)) return usual;
  TileSize best = usual;
  double best_us = 0.94 * bf16_backward_us(cu, usual, B, kp, D);
  for (TileSize t : {TILES_256, TILES_128, TILES_64}) {
    if (t == TILES_256 && D % 256 != 0) continue;
    const double us = t == usual ? best_us : bf16_backward_us(cu, t, B, kp, D);
    if (us < best_us) best = t, best_us = us;
  }
  return best;
}

// ---------------------------------------------------------------------------------------------
// Scratch of a context for up to B_max samples and kp_cap (padded) classes, in floats.
// ---------------------------------------------------------------------------------------------
// Partial sums of the backward launch: those of dfeatures in front, those of a dweight product cut over
// the batch behind.  A product is cut only as far as its workgroups fill the GPU, so either stays
// below one 256 x 256 tile for every compute unit (large batches: kLongRoom of them), or is one copy of
// its result.
inline int64_t part_floats(int cu, int D, int B_max) {
  const int64_t Bp = round_up(B_max, kPadB), Dp = round_up(D, 256), all = (int64_t)cu * 256 * 256;
  const int64_t any = std::min(2 * kMaxSplits * Bp * Dp, std::max(all, Bp * Dp) + all);
  if (Bp <= kLongBatch) return any;
  return std::max(any, std::min((kMaxLongSplits + kMaxSplits) * Bp * Dp,
                                std::max(kLongRoom * all, Bp * Dp) + kLongRoom * all));
}

// Partial row sums of the logits: one for every sample and tile.  64-tiles are taken only for few
// tiles.
inline int64_t rowpart_floats(int cu, int B_max, int64_t kp_cap) {
  const int64_t Bp = round_up(B_max, kPadB);
  return std::max(kp_cap / 128 * Bp, std::min(kp_cap / 64 * Bp, (int64_t)2048 * cu));
}

}  // namespace pfc
