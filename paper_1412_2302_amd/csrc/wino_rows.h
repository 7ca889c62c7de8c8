// Which tiles of a transformed layer have which of the 36 positions (winograd.h), for the products over them (gemm_split.h).
#pragma once

#include "gemm.h"

namespace ax {

// The short transform, F(1, 3): three of the six points, 0, 1 and -1.  At these x^3 = x, so that a patch goes on as d3 = d1, d4 =
// d2 and the matrices of a whole tile serve it, taps and gradients as everybody else has them:
//     y = m0 + m1 + m2,  m0 = 4 (d0 - d2) g(0),  m1 = -3 (d1 + d2) g(1),  m2 = 3 (d1 - d2) g(-1).
// Errors of the products reach y with a variance of sum_p |G[p]|^2 |B[p]|^2 over the inputs that lie in the map: 5, 2.5 and 1 for
// a padding of 0, 1 and 2, where the first output of a whole tile has 9.0, 4.0 and 1.  (1, -1 and infinity would have 5, 4 and
// 2.5.)
AX_HD constexpr bool in_short(int i) { return i < 3; }
// The s-th position of a launch over all 36: one that short tiles have in both directions, in one, in neither, in the other, and
// so on. Compute units that share a second-level cache take neighbouring positions; in their own order the first half of them had
// a seventh more to do (third to fifth layer of 128 pictures, forward 78.7, 66.6 and 47.8 us).
AX_HD int wino_spread(int s) {
  const int b = s >> 2, r = s & 3, i = b / 3, j = b - 3 * i;
  return 6 * (i + (r >= 2 ? 3 : 0)) + j + (r == 1 || r == 2 ? 3 : 0);
}
// Rows of the transformed tensors that have position p = 6 * row + column
struct RowRange {
  int lo, hi;
};
AX_HD RowRange wino_rows(int p, int short_y, int whole, int short_x, int tiles) {
  const bool i = in_short(p / 6), j = in_short(p % 6);
  RowRange r;
  r.lo = i ? 0 : short_y;
  r.hi = !j ? short_y + whole : i ? tiles : short_y + whole + short_x;
  return r;
}
}  // namespace ax
