// Checks the split of workgroups into rows: every launch dimension below 2^32
// threads, every workgroup there, one row wherever one is enough.
#include <algorithm>
#include <cstdio>

#include "launch_rows.h"

int main() {
    constexpr int64_t kDim = int64_t{1} << 32;
    for (int threads : {64, 128, 256, 1024}) {
        for (int shift = 0; shift < 31; ++shift) {
            for (int64_t off = -3; off <= 3; ++off) {
                for (int64_t blocks : {(int64_t{1} << shift) + off, kDim / threads + off, 3 * (kDim / threads) + off}) {
                    if (blocks < 1) continue;
                    const LaunchRows l = launch_rows(blocks, threads);
                    const int64_t all = static_cast<int64_t>(l.length) * l.rows;
                    const bool one = blocks * threads < kDim;
                    if (static_cast<int64_t>(l.length) * threads >= kDim || all < blocks || all - blocks >= l.rows ||
                        l.rows > 65535 || (one && (l.rows != 1 || l.length != blocks))) {
                        std::printf("%lld workgroups of %d threads: %u x %u\n", static_cast<long long>(blocks), threads,
                                    l.length, l.rows);
                        return 1;
                    }
                }
            }
        }
    }
    return 0;
}
