// The batched V-Sample kernels in 10 dimensions, of every family (one file per
// dimension so that the instantiations compile in parallel).
#include "vsample_impl.h"

namespace mcubes {
MCUBES_VS_TILES(10)
}  // namespace mcubes
