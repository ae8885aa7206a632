// The tiled numeric kernel: FP32 values, 2 directions.
#include "tc2_tile_numeric.h"

namespace tc2 {
template bool tile_launch<float, 2>(hipStream_t, const TileArgs&);
}  // namespace tc2
