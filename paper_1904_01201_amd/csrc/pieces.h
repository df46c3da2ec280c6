// Launches over more items than one grid holds (host only).
#pragma once
#include <stdint.h>

#include <algorithm>

namespace habmi {

// Threads of one launch: a grid of 2^32 threads or more is refused, and the
// kernels keep thread and item indices in 32 bits.
constexpr uint64_t kMaxThreads = 1ull << 31;

// fn(first, count, blocks) for consecutive pieces of n items, `per_block` of
// them to a block of `threads` threads, each piece a launch of its own.
template <class F>
void in_pieces(uint32_t n, uint32_t per_block, uint32_t threads, F &&fn)
{
    const uint64_t most = kMaxThreads / threads * per_block;
    for (uint64_t first = 0; first < n; first += most) {
        const uint32_t count = (uint32_t)std::min<uint64_t>(most, n - first);
        fn((uint32_t)first, count, (uint32_t)(((uint64_t)count + per_block - 1) / per_block));
    }
}

}  // namespace habmi
