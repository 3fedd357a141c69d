// Walks sample lists over output positions as the fill kernels do, and checks
// that every position of an accepted list is stored exactly once, inside the
// list.  Prints the first violation and returns 1.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <vector>

#define __host__
#define __device__
#include "fill_list.h"

namespace {

constexpr int kLimit = 3000;  // blocks a list of this test can hold at most
constexpr int kPiece = 2048;  // samples of 64 halves

// Samples [pos0, pos0 + n) in pieces of `piece`: the block walk of each
// piece, then the ends.  False: a position stored twice, missed or outside.
bool walk(int64_t pos0, int64_t n, int piece) {
    std::vector<int> stored(static_cast<size_t>(n), 0);
    bool ok = true;
    auto store = [&](int64_t b, int64_t from, int64_t to) {  // of the block at b, the positions in [from, to)
        for (int64_t p = std::max(b, from); p < std::min(b + kListBlock, to); ++p) {
            if (p < pos0 || p >= pos0 + n) {
                ok = false;
            } else {
                ++stored[static_cast<size_t>(p - pos0)];
            }
        }
    };
    FillList l = begin_list(static_cast<int>(pos0));
    bool head = false;
    for (int64_t left = n; left > 0 && ok;) {
        const int take = static_cast<int>(std::min<int64_t>(left, piece));
        const int end = l.pos + take;
        int blocks = 0;
        const int block = l.block;
        l.block = walk_blocks(
            block, l.head_end, end, [&]() { head = true; },
            [&](int b) {
                if (++blocks > kLimit) {
                    std::printf("the walk from %lld does not end\n", static_cast<long long>(pos0));
                    std::exit(1);
                }
                store(b, b, static_cast<int64_t>(b) + kListBlock);
            });
        l.pos = end;
        left -= take;
    }
    if (head) store(l.head_end - kListBlock, pos0, l.head_end);
    store(l.block, std::max<int64_t>(l.block, pos0), l.pos);
    for (int s : stored) ok = ok && s == 1;
    if (!ok) std::printf("positions [%lld, %lld) in pieces of %d\n", static_cast<long long>(pos0),
                         static_cast<long long>(pos0 + n), piece);
    return ok;
}

}  // namespace

int main() {
    constexpr int64_t kTop = INT32_MAX;
    int accepted = 0, refused = 0;
    for (int64_t base : {int64_t{0}, int64_t{1} << 20, kTop - 5000, kTop - 300}) {
        for (int64_t off = 0; off < 300; ++off) {
            for (int64_t n : {0, 1, 2, 63, 64, 65, 127, 128, 129, 200, 2047, 2048, 2111, 4500}) {
                const int64_t pos0 = base + off;
                for (int64_t capacity : {kTop, pos0 + n, pos0 + n - 1}) {
                    if (capacity > kTop || capacity < 0) continue;
                    if (!list_fits(pos0, n, capacity)) {
                        ++refused;
                        continue;
                    }
                    ++accepted;
                    if (pos0 + n > capacity) return std::printf("accepted past the output\n"), 1;
                    for (int piece : {kPiece, 32, 1}) {
                        if (!walk(pos0, n, piece)) return 1;
                    }
                }
            }
        }
    }
    // what lies well inside the output is listed
    if (list_fits(-1, 1, kTop) || !list_fits(0, 0, 0) || !list_fits(kTop - 200, 100, kTop)) return 1;
    std::printf("%d lists, %d refused\n", accepted, refused);
    return 0;
}
