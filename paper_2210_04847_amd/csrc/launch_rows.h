// Launches of more workgroups than one dimension holds.  Plain C++, so that
// the split can be checked on the host.
#pragma once

#include <cstdint>

namespace {

// A dimension of a launch holds less than 2^32 threads: more workgroups are
// laid out in rows of equal length, the last of them past the end of the work
// (fewer of those than rows).
struct LaunchRows {
    uint32_t length, rows;
};

inline LaunchRows launch_rows(int64_t blocks, int threads) {
    const int64_t most = ((int64_t{1} << 32) - 1) / threads;
    const int64_t rows = (blocks + most - 1) / most;
    return LaunchRows{static_cast<uint32_t>((blocks + rows - 1) / rows), static_cast<uint32_t>(rows)};
}

}  // namespace
