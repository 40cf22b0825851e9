// Order in which a launch's blocks take the tiles of a grid.
#pragma once

#include <algorithm>
#include <cstdint>
#include <numeric>

namespace sdf {

namespace {

// Consecutive blocks go to the XCDs and their shader engines in turn, 32 in
// all, and neighbouring tiles have much the same work.  Block b of n takes tile
// scattered_tile(b, n, tile_step(n)), a bijection: each row of 32 blocks is
// turned by another amount, or n a multiple of 32 would leave every engine the
// tiles of one residue, and the rows' tiles lie n over the golden ratio apart,
// so that each engine, and each stretch of the launch, has tiles from all over
// the grid.
inline int64_t tile_step(int64_t n) {
    int64_t step = std::max<int64_t>(1, int64_t(0.6180339887498949 * double(n)));
    while (std::gcd(step, n) != 1) ++step;
    return step;
}
__host__ __device__ inline int64_t scattered_tile(int64_t b, int64_t n, int64_t step) {
    const int64_t row = b >> 5;
    const int64_t turned = 32 * row + 32 <= n ? 32 * row + ((b + 5 * row + 11 * (row >> 5)) & 31) : b;
    return turned * step % n;
}

}  // namespace

}  // namespace sdf
