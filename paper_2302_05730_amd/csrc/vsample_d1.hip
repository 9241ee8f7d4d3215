// The batched V-Sample kernels in 1 dimension, of every family (one file per
// dimension so that the instantiations compile in parallel).
#include "vsample_impl.h"

namespace mcubes {
MCUBES_VS_TILES(1)
}  // namespace mcubes
