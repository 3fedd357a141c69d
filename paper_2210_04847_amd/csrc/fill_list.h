// Output positions of the sample lists that the fill kernels store in whole
// blocks of kListBlock positions.  Plain C++, so that the walk over the
// blocks can be checked on the host.
#pragma once

#include <cstdint>

namespace {

constexpr int kListBlock = 64;  // one position per lane

// The list of a wave: it holds the positions [block, pos); `queued` halves
// wait for it; head_end: the end of the wave's first block, if the wave does
// not begin it (-1 if it does).
struct FillList {
    int pos, block, head_end, queued;
};

// Whether a wave's n samples from position pos0 on may go through the list:
// inside the output, and, as the walk forms positions up to a block past the
// last sample in 32 bits, a block short of 2^31.
__host__ __device__ inline bool list_fits(int64_t pos0, int64_t n, int64_t capacity) {
    return pos0 >= 0 && pos0 + n <= capacity && pos0 + n <= INT32_MAX - kListBlock;
}

// (Unsigned: a wave that list_fits refuses begins a list too and never uses it.)
__host__ __device__ inline FillList begin_list(int pos) {
    const uint32_t block = static_cast<uint32_t>(pos) & ~static_cast<uint32_t>(kListBlock - 1);
    return FillList{pos, static_cast<int>(block),
                    block == static_cast<uint32_t>(pos) ? -1 : static_cast<int>(block + kListBlock), 0};
}

// Walks the complete blocks of the list's positions [block, end): head() for
// a first one that other waves' samples precede, store(b) for the block of
// positions [b, b + kListBlock).  Returns the first position behind them.
template <typename Head, typename Store>
__host__ __device__ inline int walk_blocks(int block, int head_end, int end, Head head, Store store) {
    int b = block;
    if (b + kListBlock == head_end && head_end <= end) {
        head();
        b += kListBlock;
    }
    for (; b + kListBlock <= end; b += kListBlock) store(b);
    return b;
}

}  // namespace
