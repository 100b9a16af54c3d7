// Index arithmetic shared by the fp32 FC kernels.
#pragma once
#include <hip/hip_runtime.h>

#include "sfc_kernels.hpp"

namespace canvas {
namespace sfc {

// Consecutive workgroups go to consecutive XCDs, each with an L2 of its own; this renumbers them so that an XCD works on
// neighbouring tiles, whose operands overlap (the margin of a window, the other outputs of the same pixels).  The grid is
// a multiple of eight workgroups, in rows if it is long (grid_of); the numbers past the last tile have no work.
__device__ __forceinline__ unsigned tile_of_block() {
    const unsigned per = gridDim.x / 8;
    return blockIdx.y * gridDim.x + (blockIdx.x % 8) * per + blockIdx.x / 8;
}

// x / d for the small dividends of index arithmetic: exact while x * d < 2^32 (the host checks the image's sizes)
__device__ __forceinline__ int quotient(int x, int d, uint32_t m) { return d == 1 ? x : (int)__umulhi((uint32_t)x, m); }
// image of pixel p, counted from an image at whose pixel p0 < P a tile of at most 128 pixels begins
__device__ __forceinline__ int image_of(const Params& Q, int p) { return Q.P >= 128 ? (p >= Q.P ? 1 : 0) : quotient(p, Q.P, Q.mP); }

// Position j of a window's operand tile whose first pixel is (n0, h0, .) -> element offset of that source pixel in
// channel 0 of the group, or -1 in the margin.  Rows are numbered through the batch with HP = H + KH - 1 rows per image.
__device__ __forceinline__ int64_t window_source(const Params& Q, int64_t n0, int h0, int j) {
    const int s = quotient(j, Q.Wp, Q.mWp), c = j - s * Q.Wp;
    const int q = h0 + s;
    const int dn = quotient(q, Q.HP, Q.mHP);
    const int h = q - dn * Q.HP - Q.KH / 2, w = c - Q.KW / 2;
    const int64_t n = n0 + dn;
    if (n >= Q.N || h < 0 || h >= Q.H || w < 0 || w >= Q.W) return -1;
    return n * Q.G * Q.R * (int64_t)Q.P + (int64_t)h * Q.W + w;
}

}  // namespace sfc
}  // namespace canvas
