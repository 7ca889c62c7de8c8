// Which tiles of a transformed layer have which of the 36 positions (winograd.h), for the products over them (gemm_split.h).
#pragma once

#include "gemm.h"

namespace ax {

// The short transform, F(1, 3): of the six points 1, -1 and infinity, with the taps as everybody else has them,
//     y = m1 + m2 + m5,  m1 = -3 (d0 + d1) g(1),  m2 = -3 (d0 - d1) g(-1),  m5 = (d2 - d0) g(inf).
constexpr unsigned kShortPoints = 1u << 1 | 1u << 2 | 1u << 5;
AX_HD bool in_short(int i) { return kShortPoints >> i & 1u; }
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
