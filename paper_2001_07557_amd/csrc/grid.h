// Grids of kernels that take one item per thread.  A launch counts its work
// items in 32 bits per dimension and drops what is beyond, with no error (an FP64
// full field of V >= 357.9M sites, 69 GB, has more 16-byte words than that), so
// the blocks beyond 2^23 go into y.
#pragma once

#include "lqcd_internal.h"

namespace lqcd {

constexpr int64_t GRID_ROW = (int64_t)1 << 23;  // a multiple of the 8 XCDs
static_assert(GRID_ROW * 256 < ((int64_t)1 << 32), "rows of blocks of 256 threads");

inline dim3 block_grid(int64_t blocks) {
    return dim3((unsigned)(blocks < GRID_ROW ? blocks : GRID_ROW), (unsigned)((blocks + GRID_ROW - 1) / GRID_ROW));
}
// index of this block, and the blocks of the launch, the last row's surplus
// included
__device__ __forceinline__ int64_t block_index() { return (int64_t)blockIdx.y * gridDim.x + blockIdx.x; }
__device__ __forceinline__ uint32_t block_count() { return gridDim.x * gridDim.y; }

}  // namespace lqcd
