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

// Cells per CU from which a launch of the padded size S is packed (bdf_packed.h), 0
// for never.  `waves`: packed waves that reside on a CU, by their LDS (R rate
// constants a cell) and at most 16.  Fewer cells leave SIMDs without a wave, and
// one cell per wave has the shorter steps.  And the more of the work is
// reactions, which fill the lanes of a wave without packing too, the less packing
// saves, while the rate constants of its cells leave the LDS room for fewer waves.
// Packed against one cell per wave (5-wave budget) on 256 CUs, ms, FP64 unless stated:
//   up to 64 reactions   9 species, R 30: 5.55 / 6.14 on 32 cells a CU, 23.2 / 36.0 on 256;
//   (one pass of a wave) 14, R 40: 7.25 / 7.29 on 32; 16, R 64: 7.26 / 7.34 on 32; 9, R 64:
//                        3.90 / 3.82 on 32, 4.52 / 5.31 on 48; 4, R 60: 5.26 / 5.45 on 40
//   13 waves and more    9, R 100: 4.53 / 4.12 on 32, 5.17 / 5.56 on 48
//   10 to 12 waves       8, R 150: 7.08 / 6.68 on 32, 12.2 / 11.6 on 64, 21.2 / 22.0 on
//                        128; 16, R 100 FP32: 11.6 / 11.0 on 32, 34.4 / 36.7 on 128
//   9 waves              16, R 100: 18.4 / 18.2 on 64, 32.1 / 33.2 on 128; 14, R 100: 39.2 /
//                        38.7 on 128, 71.7 / 74.5 on 256; 4, R 200: 30.7 / 31.1 on 128
//   8 and fewer          9, R 200: 40.1 / 39.8 on 256; 16, R 400: 121 / 87.4 on 256
//   17 to 21 species     FP32, R 84: 20.8 / 19.9 on 64, 28.2 / 29.1 on 96, 257 / 275 on
//                        1,024; R 110 (16 waves): 26.6 / 26.9 on 96; R 128 (15): 30.9 /
//                        30.3 on 96; R 160: 49.1 / 47.9 on 192.  FP64, R 84: 71.7 /
//                        70.5 on 256, 271.4 / 270.1 on 1,024; R 325: 175 / 147 on 256
inline int packed_min_cells_per_cu(int S, int R, bool fp32, int waves) {
  if (S > 16) return fp32 && waves >= 16 ? 96 : 0;
  if (R <= 64) return S <= 4 ? 40 : 32;
  if (waves >= 13) return 48;
  return waves >= 10 ? 128 : waves == 9 ? 256 : 0;
}

}  // namespace bdfx
