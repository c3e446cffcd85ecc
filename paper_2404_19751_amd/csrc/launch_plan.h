// Host arithmetic of launches and scratch memory, free of HIP.
#pragma once
#include <stdint.h>

#include <algorithm>

namespace gsim {

// Blocks of a kernel that strides over n items (fills of tables that may hold
// billions of entries): a launch takes fewer than 2^32 threads, and 2^20
// blocks keep every compute unit busy to the end.
constexpr int64_t kFillBlocksMax = 1 << 20;
inline int fill_blocks(int64_t n, int block) {
    return (int)std::min<int64_t>((n + block - 1) / block, kFillBlocksMax);
}

}  // namespace gsim
