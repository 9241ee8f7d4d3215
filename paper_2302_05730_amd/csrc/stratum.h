// The coordinate the flow-mapped iteration draws in a stratum: (digit + u) / g
// with u = (r + 1/2) 2^-32, in FP64, then FP32.  A quotient: it may lie halfway
// between two floats (digit 0, 2 r + 1 a multiple of g, below 2^-8), where a
// product with the rounded 1 / g falls to either side.  Usable on the host as
// well, so that it can be checked there.
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

namespace mcubes {

__host__ __device__ __forceinline__ float stratum_coordinate(uint32_t digit, uint32_t r, uint32_t g) {
    const double u = std::fma((double)r, 0x1p-32, 0x1p-33);
    return (float)(((double)digit + u) / (double)g);
}

}  // namespace mcubes
