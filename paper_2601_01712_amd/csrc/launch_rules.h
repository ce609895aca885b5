// Which kernel of the 16-bit path a launch takes, by its sizes.  No HIP in this file: the tests compile it with the host compiler, so that a
// test of a kernel can say that its launches take that kernel.
#pragma once

#include "plan.h"

namespace relaygr {

// Tiles of the projection, rows x columns of [u | v | q | k].  Launches of few thousand rows: the largest tile that still gives the chip one round of
// workgroups; then those of which two (at d = 128 three) share a compute unit, up to three rounds' worth: their stages in flight add up.  What such a
// launch takes is the round trips of its operand stream, so that the smallest has the whole of K in flight (64 x 64: 128 KiB of LDS up to d = 512).
// Beyond them the weight-stationary form, at d = 1024 the 256 x 128 tile.
enum class F1Tile { k64x64, k64x128, k128x128, k128x128x3, kStationary, k256x128 };
// Row groups of the weight-stationary form: one persistent workgroup per compute unit, (units / slices of 128 columns) groups, a multiple of 8 so
// that each XCD takes whole groups; 0: not that form.
inline int f1_row_groups(int d, int nblk, int n_cus) { return d <= 512 ? n_cus / (nblk * (d / 128)) & ~7 : 0; }
// us a call of 4 layers over 64 keys by rows, 64 x 64 / 64 x 128 / 128 x 128 with 4 stages / with 3 / weight-stationary / 256 x 128:
//   d = 512 :  512 93 / 95 / 103 / 105 / 125 / 129    1024 114 / 105 / 109 / 112 / 131 / 135    1536 132 / 123 / 113 / 114 / 137 / 142
//             2048 148 / 124 / 119 / 119 / 138 / 140    3072 175 / 140 / 142 / 140 / 146 / 147    4096 220 / 165 / 158 / 163 / 163 / 158
//             6144 307 / 219 / 219 / 203 / 214 / 211    8192 - / 266 / 260 / 240 / 243 / 241    16384 - / 467 / 435 / 419 / 414 / 434
//   d = 256 : 1024 71 / 74 / 79    2048 84 / 83 / 85    4096 101 / 102 / 100 / 101 / 114    6144 123 / 120 / 127 / 127 / 133    8192 144 / 135 / 131 / 134 / 139
//   d = 1024:  256 225 / 227 / 239    512 239 / 227 / 237    768 259 / 243 / 240    1536 320 / 269 / 280 / 278 / - / 289    2048 388 / 298 / 302 / 307 / - / 297
//   d = 128 , 64 x 128 / weight-stationary: 8250 107.8 / 116.6    9000 116.9 / 120.1    10 200 118.3 / 123.6    12 200 114.8 / 128.4
// (64 x 128 with twelve stages instead of six was never the fastest.)  nblk: column blocks of width d in the launch.
inline F1Tile f1_tile(int d, int nblk, int rows, int n_cus) {
  const int cols = nblk * (d / 128), t128 = (rows + 63) / 64 * cols, t64 = 2 * t128, tbig = (rows + 127) / 128 * cols;   // workgroups of each tile
  if (t64 <= n_cus) return F1Tile::k64x64;
  if (t128 <= n_cus) return F1Tile::k64x128;
  if (d > 256 && tbig <= n_cus) return F1Tile::k128x128;
  if (t128 <= 3 * n_cus) return F1Tile::k64x128;
  if (d > 128 && d <= 512 && tbig <= 2 * n_cus) return F1Tile::k128x128;
  if (d > 128 && d <= 512 && tbig <= 3 * n_cus) return F1Tile::k128x128x3;
  return f1_row_groups(d, nblk, n_cus) >= 8 ? F1Tile::kStationary : F1Tile::k256x128;
}

// Rows of a layer-tail workgroup.  A few hundred rows (one user per call): 8 each, so that four times as many compute units share the split partial
// sums; then 16; both as long as that is at most one workgroup per compute unit.  Four row blocks of 16 halve the passes over W2 once that still
// leaves every compute unit about two workgroups.  (d = 1024, 8 layers, us a call with 32 rows / with 8 or 16: one user of 4096 keys and 512 candidates 599 /
// 442, 100 and 1000 keys 516 / 376, 1000 and 1000 540 / 447, 1500 and 1000 590 / 519; 5 users of 500 and 1000 772 / 713, 8 864 / 831; pre-inference of
// 3500 keys 889 / 845.  At d = 128 not tried.)
constexpr int kTailVr8MaxRows = 1024, kTailVr16MaxRows = 4096, kTailVr64MinRows = 64 * 384;
inline int tail_rows(int d, int rows) {
  if (d >= 256) {
    if (rows <= kTailVr8MaxRows) return 8;
    if (rows <= kTailVr16MaxRows) return 16;
  }
  return d <= 512 && rows >= kTailVr64MinRows ? 64 : 32;
}

// Partial sums of a row that the layer tail has in flight at once: one, two, four, or all a row can have.  It loads that many of every row, whether
// the row has them or not, so that launches whose rows have fewer take kernels that ask for fewer: every batch that is not cut along the keys, or whose
// pieces meet inside a workgroup, has one; short histories have three or four.  (us a call with as many as before, two in large launches and
// eight in those of up to 1024 rows / with as many as there are: one sum, d = 512, 8 layers, 6144 rows 544.0 / 538.9, 20 000 in fp16 1358 / 1348, 32 000
// 1938 / 1926, and in the softmax form 2012 / 1984, in fp16 2099 / 2032; 4 layers, 512 rows 91.5 / 87.8; d = 256, 512 rows 67.0 / 65.0.  Two sums, 512
// rows, d = 512 95.8 / 92.6; d = 256, softmax 68.3 / 65.5.  Three sums, 1000 rows, d = 512 113.8 / 111.0; four, 512 rows 101.3 / 98.7, softmax in fp16
// 99.7 / 97.1, 1600 rows 154.7 / 150.8; d = 256, 2000 rows 98.6 / 96.7.)
// parts_all: the number all rows of the launch have, 0 where they differ; nsplit: the most a row of the call has.
inline int sums_at_once(int parts_all, int nsplit) {
  const int most = parts_all ? parts_all : nsplit;
  return most <= 2 ? most : most <= 4 ? 4 : kMaxPieces;
}

// Key tiles from which on the two wavefront groups of an attention workgroup share a piece (kNoneShared: workgroups of one group).  Pairs that the plan has
// made are always shared.  Else, at d_head 64, in rankings of cached users with no more pieces than the chip has compute units: a workgroup then has its
// unit to itself, and a second group that takes half of a long piece's keys and whose sums are added in LDS gives every SIMD a second wavefront, one's
// SiLU beside the other's products, without a partial sum more.  The hand-over costs about as much as five key tiles of the SiLU form, and more of the
// softmax form, which does half as much on the vector ALU and has the sums to rescale.  us a call with one group / two, key tiles of a piece in brackets, d =
// 512, two runs of one side differ by 0.1 to 2 us: one user of 512 candidates [7] 230.1 / 231.9, [8] 231.8 / 230.7, [9] 241.2 / 240.1, [10] 241.6 / 238.5, [12]
// 254.9 / 249.7; of 100 [8] 211.8 / 209.6, [9] 217.1 / 215.5, [10] 221.9 / 217.9, [14] 243.7 / 235.9; of 32 [17] 245.2 / 236.2; of 250 [32] 365.7 / 328.2; two
// of 256 [11] 240.3 / 240.7, [17] 286.0 / 282.7; three of 100 [4] 198.2 / 211.6, [9] 222.9 / 225.5, [10] 241.1 / 238.8, [13] 266.7 / 260.8; seven of 32 [8]
// 205.7 / 210.1, [11] 227.9 / 228.9, [17] 270.0 / 271.2 (bound by the K/V they fetch); d = 256, 256 candidates [8] 82.6 / 81.8, [10] 88.3 / 86.8, [12] 94.1 /
// 91.3.  Softmax: 512 [8] 238.4 / 241.0, [10] 247.6 / 248.1, [16] 275.3 / 268.9; 100 [16] 257.0 / 247.1; two of 32 [9] 210.4 / 214.4, [17] 280.9 / 265.2; three
// of 100 [9] 224.3 / 228.2, [17] 301.3 / 295.2; seven of 32 [8] 206.9 / 213.5, [17] 271.5 / 271.1.
// The pieces of a launch decide one by one, so that a row's sums do not depend on the other users' pieces, and short ones do not pay for a hand-over.
// (256-row items are that few only where each unit has one uncut, of at most 8 key tiles.)  Not for lists with prefix rows, whose causal pieces end in
// tiles that only some wavefronts see (pre-inference of 1000 keys 193 / 200).
constexpr int kNoneShared = 1 << 20;
inline int attn_shared_tiles(bool softmax, int heads, int dh, bool prefix_rows, const AttnCut& cut, int n_cus) {
  if (cut.gs == 2) return 0;
  const int least = softmax ? 16 : 10;
  const bool pays = dh == 64 && !prefix_rows && (int64_t)cut.all.size() * heads <= n_cus;
  return pays && !cut.all.empty() && cut.all[0].t1 - cut.all[0].t0 >= least ? least : kNoneShared;    // (the list is sorted, longest first)
}

}  // namespace relaygr
