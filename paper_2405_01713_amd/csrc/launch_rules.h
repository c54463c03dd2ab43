// launch_rules.h -- choices of the launch code that need no device: plain host
// arithmetic, so that they can be checked without a GPU.
#pragma once

#include <stdint.h>

#include <algorithm>

namespace bdfx {

// Cells per work-queue pop.  Each of the `poppers` lane groups of the grid pops
// until it meets a count past the last cell, so a launch of `cells` adds at
// most cells + (poppers + 1) * chunk to the counter.  That has to stay below
// 2^32: a counter that wraps hands cells out twice.  (`asked` otherwise; the
// results do not depend on it.)
inline int32_t pop_chunk(int32_t asked, int64_t cells, int64_t poppers) {
  const int64_t most = ((int64_t{1} << 32) - 1 - cells) / (poppers + 1);
  return static_cast<int32_t>(std::max<int64_t>(1, std::min<int64_t>(asked, most)));
}

// Blocks of a persistent grid: `asked` per CU (0: as many as reside), and no more
// than the cells fill.
inline int32_t persistent_grid(int32_t asked, int resident, int n_cu, int64_t cells, int64_t per_block) {
  const int64_t per_cu = asked > 0 ? asked : std::max(resident, 1);
  return static_cast<int32_t>(std::min(per_cu * n_cu, (cells + per_block - 1) / per_block));
}

}  // namespace bdfx
