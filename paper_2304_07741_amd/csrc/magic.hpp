// Division by a launch constant as a product.
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace canvas {

// The multiplier of a division by d: ceil(2^32 / d), 0 for d = 1.
inline uint32_t magic_u32(uint32_t d) { return d <= 1 ? 0u : (uint32_t)((((uint64_t)1 << 32) + d - 1) / d); }

// x / d.  Exact while x * d stays below 2^32; one too high at most for any x below 2^32 (x * (2^32 + e) / (d * 2^32) with e < d).
__host__ __device__ inline uint32_t div_magic(uint32_t x, uint32_t magic) { return magic ? (uint32_t)(((uint64_t)x * magic) >> 32) : x; }

// x / d for any 0 <= x < 2^31; rem: what is left.
__host__ __device__ inline int div_magic(int x, int d, uint32_t magic, int& rem) {
    int q = (int)div_magic((uint32_t)x, magic);
    rem = x - q * d;
    if (rem < 0) {  // (one too high)
        q--;
        rem += d;
    }
    return q;
}

}  // namespace canvas
