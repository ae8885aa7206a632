// The tiled numeric kernel: FP64 values, 3 directions.
#include "tc2_tile_numeric.h"

namespace tc2 {
template bool tile_launch<double, 3>(hipStream_t, const TileArgs&);
}  // namespace tc2
