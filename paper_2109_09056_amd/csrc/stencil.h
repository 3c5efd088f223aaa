// Size of the candidate stencil of a binning grid (host code, plain C++).
#pragma once

#include <stdint.h>

namespace ljmd {

// Whether the stencil of a cell holds at most `most` of the n atoms of the grid on average.
// A dimension contributes the cell and its two neighbours, or all of its one or two cells.
inline bool mean_stencil_within(const int32_t nc[3], int64_t n, int64_t most) {
  int64_t cells = 1, stencil = n;
  for (int k = 0; k < 3; ++k) {
    cells *= nc[k];
    stencil *= nc[k] < 3 ? nc[k] : 3;
  }
  return stencil <= cells * most;
}

}  // namespace ljmd
