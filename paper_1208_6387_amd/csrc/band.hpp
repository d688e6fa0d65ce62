// Storage of the interior factor L_ii (host only: no HIP header).
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

namespace rpf {

// Entry (r, c) of the n x n factor is at r + c ld: dense (ld = n), or in a band that holds its envelope on both
// sides of the diagonal, |r - c| < hw, with ld = 2 hw - 1.  The diagonal then advances ld + 1 = 2 hw from
// column to column, so columns do not overlap, the first entry is at 0, and the last one, (n - 1, n - 1), at
// (n - 1) (ld + 1): len doubles hold it.
struct FactorLayout {
  int64_t ld = 0, len = 0;
  int64_t hw = 0;  // 0: dense
};

// rend[t]: one past the last row that the envelope of the column block t (bs columns) reaches.  Up to `wide`
// rows or columns are read as one rectangle, so the band holds rend[t] - t bs + wide on each side.  The band
// is taken where it has fewer rows than the dense matrix.
inline FactorLayout factor_layout(int64_t n, const std::vector<int64_t>& rend, int64_t bs, int64_t wide) {
  int64_t hw = wide;
  for (size_t t = 0; t < rend.size(); ++t) hw = std::max(hw, rend[t] - (int64_t)t * bs + wide);
  FactorLayout f;
  if (2 * hw - 1 < n) {
    f.hw = hw;
    f.ld = 2 * hw - 1;
    f.len = (f.ld + 1) * n;
  } else {
    f.ld = n;
    f.len = n * n;
  }
  return f;
}

}  // namespace rpf
