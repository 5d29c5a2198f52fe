// Launch sizes of the kernels that give a row several lanes or a slice a block.
// HIP refuses a launch of 2^32 threads or more in a dimension, which such
// kernels reach within the interface's 2^29 - 1 rows.
#pragma once
#include <algorithm>
#include <cstdint>

namespace amgiga {

constexpr unsigned MAX_BLOCKS = 65536;   // 256 a CU; the kernels stride over the rest

// blocks of 256 threads for n rows of `lanes` threads, at most MAX_BLOCKS
inline unsigned lanes_grid(int64_t n, int lanes)
{
    return (unsigned)std::min<int64_t>((n * lanes + 255) / 256, MAX_BLOCKS);
}

}  // namespace amgiga
