// Sub-tile shapes of the tiled numeric kernel and its launch per value type and
// number of directions.
#pragma once
#include "tc2_internal.h"

namespace tc2 {

// Sub-tile shapes (rows of cluster P x columns of cluster Q per work item).
// Which ones exist depends on the kernel kind and D: the accumulators of a
// wave ((1 + D) tiles per owned output) must stay within its register budget.
constexpr int SHAPE_SP[TS_N] = {8, 4, 8, 4};
constexpr int SHAPE_TQ[TS_N] = {8, 8, 4, 4};

constexpr bool shape_ok(int kind, int D, int s) {
  return ((kind == K_FP64 || kind == K_WIDE) && D >= 2)
             ? s == TS_4x4
             : (s == TS_8x8 || ((D == 1 || D == 3) && s == TS_4x8) ||
                (D == 1 && kind != K_BF16 && s == TS_8x4));
}

// the kernel of one value type and number of directions; false when the shape
// does not exist for the kind
template <typename T, int D>
bool tile_launch(hipStream_t st, const TileArgs& a);

}  // namespace tc2
