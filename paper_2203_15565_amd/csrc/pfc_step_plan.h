// Host-side rules of forward/backward: the size of the GEMM tiles, how the backward launch is dealt to
// workgroups, and the scratch that follows from it.  Plain C++, so that the rules can be checked on the
// CPU over everything that the entry points accept.
#pragma once

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

// Size of the GEMM tiles, one for the logits and one for the backward launch of a call.  256 x 256
// moves the least data per flop and fills a compute unit with one workgroup, 128 x 128 puts two on
// it, 64 x 64 three.  Measured on 256 compute units over batches of 48 .. 16,384 samples and 320 ..
// 2 million classes (us for 256 / 128 / 64, D = 512 unless stated):
//   bf16 logits: a round of 256-tiles costs the same however full it is, so they win only where the
//     last round is nearly full (1024 x 205,991: 336 / 347 / 507; 768 x 20,599 x D 1024, 0.95 of a
//     round: 41 / 45 / 64; 1024 x 36,024, 2.2 rounds: 71 / 58 / 83) and the reduction is long
//     (8192 x 6,000 x D 256: 71 / 65 / 102); 64-tiles only for a handful of 128-tiles (512 x 4,000:
//     24 / 9.8 / 8.7; 512 x 9,344: 24 / 14.7 / 16.0).
//   bf16 backward: 256-tiles unless they leave compute units idle (512 x 4,000: 22 / 15 / 17;
//     512 x 16,000: 29 / 30 / 45; 1024 x 205,991: 482 / 612 / 996), the batch would be padded much
//     more (128 x 200,000: 210 / 179 / 260) or the reduction is short and the tiles few
//     (256 x 36,000: 42 / 39 / 57; 256 x 200,000: 221 / 260 / 368); 64-tiles for the smallest
//     problems (128 x 1,000: 15 / 7.3 / 5.8).
//   fp32: the matrix cores are the bound at any of the sizes, so what counts is how evenly the
//     compute units are loaded: 64-tiles where a few 128-tiles per compute unit do not come out
//     even (logits 512 x 9,344: 135 / 77 / 57; 128 x 1,000: 129 / 37 / 15).  From one 256-tile per
//     compute unit on the sizes are close (2048 x 60,000: 1144 / 1127 / 1207; 512 x 60,000: 299 /
//     315 / 330) and the logits keep 256 and its order of the row sums.
enum TileSize { TILES_64 = 64, TILES_128 = 128, TILES_256 = 256 };

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

inline TileSize backward_tiles(int cu, int es, int B, int64_t kp, int D) {
  const int Bp = (int)round_up(B, 128), Bp256 = (int)round_up(B, 256);
  const int Dp = (int)round_up(D, kPadD), Dp256 = (int)round_up(D, 256);
  const int64_t mid = kp / 128 * (Dp / 128), big = kp / 256 * (Dp256 / 256);
  if (es == 4)
    return even_rounds(mid * dweight_slices(cu, (int)mid, Bp, kp, 32), cu) ? TILES_128 : TILES_64;
  // (columns: 640 -> 768 and 896 -> 1024 cost less than the smaller tile, 384 -> 512 more)
  if (Dp256 * 100 <= Dp * 125 && Bp256 * 100 <= Bp * 115 &&
      big * dweight_slices(cu, (int)big, Bp256, kp, 64) * 2 >= cu && (B >= 512 || big * 2 >= cu * 3))
    return TILES_256;
  return B > 128 || 2 * mid > cu ? TILES_128 : TILES_64;
}

// Geometry of the tiles: reduction steps of a slab, workgroups that a compute unit holds.
inline int tile_bk(int es) { return 128 / es; }
inline int tiles_per_cu(TileSize t, int es) {
  return t == TILES_256 ? 1 : t == TILES_128 ? 2 : es == 2 ? 3 : 4;
}

// Whether the one-kernel form of the fused call takes the class set: its tile (128 classes x 512 columns)
// spans the rows, and there is at least one for every compute unit.
inline bool fits_one_kernel(int cu, int D, int64_t kp) { return D == 512 && kp / 128 >= cu; }

// The dfeatures product: slices of S, and workgroups of one tile and slice each.
struct DxShape {
  int slabs_total, slabs_per, splits, tiles_i, tiles_d;
  int wgs;   // workgroups: tiles_i * tiles_d * splits, rounded up to 8
};

// About `wgs` workgroups, at least 4 slabs each.  The callers ask
// for half of what the GPU holds at a time, or for all the room that the dweight tiles leave:
// measured against all of it and a quarter of it (us a step, quarter / half / all):
// 1024 samples x 205,991 classes x 512 1499 / 1302 / 1365, x 360,232 2511 / 2166 / 2251, fused
// x 205,991 1162 / 1098 / 1161.  Fewer workgroups write fewer partial sums (2 MB a slice there)
// but are longer than everything behind them.
inline DxShape dx_shape(int cu, int es, TileSize t, int Bp, int Dp, int D, int64_t kp, int64_t wgs) {
  DxShape dx;
  dx.tiles_i = Bp / t;
  dx.tiles_d = Dp / t;
  dx.slabs_total = (int)(kp / tile_bk(es));
  int64_t want = wgs / (dx.tiles_i * dx.tiles_d);
  // fp32 sums that are not cut into pieces: slices of more than 4096 classes are halved, for the
  // rounding of the sums (100 samples x 400,000 classes dX 2.81e-7 off, halved 2.70e-7) and, fused, for
  // workgroups that are not the end of the launch (4.23 -> 3.18 ms; 512 x 200,000 2.85 -> 2.92)
  const bool halve = es == 4 && fits_one_kernel(cu, D, kp) && kp > (int64_t)kMaxSplits * 4096;
  want = std::min<int64_t>({want, halve ? 2 * kMaxSplits : kMaxSplits, dx.slabs_total / 4});
  if (want < 1) want = 1;
  dx.slabs_per = (int)((dx.slabs_total + want - 1) / want);
  dx.splits = (dx.slabs_total + dx.slabs_per - 1) / dx.slabs_per;
  dx.wgs = (int)round_up((int64_t)dx.tiles_i * dx.tiles_d * dx.splits, 8);
  return dx;
}

// Slices of the batch in the dweight product, and the shape of the dfeatures product beside it
// (the same with and without the update, so that dX has the same bits).
struct BackwardShape {
  int slabs_per, splits;   // of the batch
  DxShape dx;
};
inline BackwardShape backward_shape(int cu, int es, TileSize t, int Bp, int Dp, int D, int64_t kp) {
  BackwardShape s;
  const int tiles_w = (int)(kp / t) * (Dp / t);
  const int slabs_total = Bp / tile_bk(es);
  const int want = dweight_slices(cu, tiles_w, Bp, kp, tile_bk(es));
  s.slabs_per = (slabs_total + want - 1) / want;
  s.splits = (slabs_total + s.slabs_per - 1) / s.slabs_per;
  const int64_t slots = (int64_t)cu * tiles_per_cu(t, es);
  const int64_t wgs_w = (int64_t)tiles_w * s.splits;
  // fp32 tiles take long: dfeatures workgroups no longer than those, so that the end comes out even
  // (fused, 1024 x 36,024 x 512: half of the GPU's room 1546 us a step, twice the room 1212)
  const int64_t wgs = es == 4 && wgs_w > 2 * slots ? 2 * slots : std::max(slots / 2, slots - wgs_w);
  s.dx = dx_shape(cu, es, t, Bp, Dp, D, kp, wgs);
  return s;
}

// ---------------------------------------------------------------------------------------------
// Scratch of a context for up to B_max samples and kp_cap (padded) classes, in floats.
// ---------------------------------------------------------------------------------------------
// Partial sums of the backward launch: those of dfeatures in front, those of a dweight product cut over
// the batch behind.  A product is cut only as far as its workgroups fill the GPU, so either stays
// below one 256 x 256 tile for every compute unit, or is one copy of its result.
inline int64_t part_floats(int cu, int D, int B_max) {
  const int64_t Bp = round_up(B_max, kPadB), Dp = round_up(D, 256), all = (int64_t)cu * 256 * 256;
  return std::min(2 * kMaxSplits * Bp * Dp, std::max(all, Bp * Dp) + all);
}

// Partial row sums of the logits: one for every sample and tile.  64-tiles are taken only for few tiles.
inline int64_t rowpart_floats(int cu, int B_max, int64_t kp_cap) {
  const int64_t Bp = round_up(B_max, kPadB);
  return std::max(kp_cap / 128 * Bp, std::min(kp_cap / 64 * Bp, (int64_t)2048 * cu));
}

}  // namespace pfc
