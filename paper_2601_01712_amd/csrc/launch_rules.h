// Which kernel of the 16-bit path a launch takes, by its sizes.  No HIP in this file: the tests compile it with the host compiler, so that a
// test of a kernel can say that its launches take that kernel.
#pragma once

#include "plan.h"

namespace relaygr {

// Rows of a layer-tail workgroup.  A few hundred rows (one user per call): 8 each, so that four times as many compute units share the split partial
// sums; then 16; both as long as that is at most one workgroup per compute unit.  Four row blocks of 16 halve the passes over W2 once that still
// leaves every compute unit about two workgroups.
constexpr int kTailVr8MaxRows = 1024, kTailVr16MaxRows = 4096, kTailVr64MinRows = 64 * 384;
inline int tail_rows(int d, int rows) {
  if (d == 256 || d == 512) {
    if (rows <= kTailVr8MaxRows) return 8;
    if (rows <= kTailVr16MaxRows) return 16;
  }
  return d <= 512 && rows >= kTailVr64MinRows ? 64 : 32;
}

// Partial sums of a row that the layer tail has in flight at once: one, two, or all a row can have.  It loads that many of every row, whether
// the row has them or not, so that launches whose rows have one or two (every batch that is not cut along the keys, or whose pieces meet inside a
// workgroup) take kernels that ask for no more.  (us a call with as many as before, two in large launches and eight in those of up to 1024 rows /
// with as many as there are: one sum, d = 512, 8 layers, 6144 rows 544.0 / 538.9, 20 000 in fp16 1358 / 1348, 32 000 1938 / 1926, and in the softmax
// form 2012 / 1984, in fp16 2099 / 2032; 4 layers, 512 rows 91.5 / 87.8; d = 256, 512 rows 67.0 / 65.0.  Two sums, 512 rows, d = 512 95.8 / 92.6;
// d = 256, softmax 68.3 / 65.5.)  parts_all: the number all rows of the launch have, 0 where they differ; nsplit: the most a row of the call has.
inline int sums_at_once(int parts_all, int nsplit) {
  const int most = parts_all ? parts_all : nsplit;
  return most <= 2 ? most : kMaxPieces;
}

}  // namespace relaygr
