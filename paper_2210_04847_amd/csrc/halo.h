// Halo bits of a bit-packed occupancy grid (layout in common.h), built by
// nacc_grid_build_skip into the skip buffer and by the marching count pass
// into its workspace when the caller passes no skip buffer; and hole bits,
// the halo of the empty cells (a clear bit: every cell within kHaloReach is
// occupied), built by the count pass.
#pragma once

#include "common.h"

namespace {

using namespace nacc;
using namespace nacc::dev;

constexpr int kHaloThreads = 64;

// Even bits of w, gathered in its low 16 bits.
__device__ __forceinline__ uint32_t even_bits(uint32_t w) {
    w &= 0x55555555u;
    w = (w | (w >> 1)) & 0x33333333u;
    w = (w | (w >> 2)) & 0x0f0f0f0fu;
    w = (w | (w >> 4)) & 0x00ff00ffu;
    return (w | (w >> 8)) & 0xffffu;
}

// Four consecutive words from q on, as one load where all of them exist.
struct __attribute__((packed, aligned(4))) Words4 {
    uint32_t v[4];
};

// ORs the bits [z0, z0 + 96) of the fine rows (x, y) for 3 values of x from
// x0 and kHaloReach rows of y on either side of the block's two (`w`), and
// their complements (`e`); rows are clamped into the grid (a clamped row is
// one of the others).  WHOLE: every row's four words lie inside the grid.
template <bool WHOLE>
__device__ __forceinline__ void or_rows(const uint32_t* __restrict__ fine, uint32_t last, int res, int x0, int cy,
                                        uint32_t z0, uint32_t w[3], uint32_t e[3]) {
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const int x = min(max(x0 + i, 0), res - 1);
#pragma unroll
        for (int k = -kHaloReach; k < 2 + kHaloReach; ++k) {
            const int y = min(max(2 * cy + k, 0), res - 1);
            const uint32_t a = static_cast<uint32_t>(x * res + y) * static_cast<uint32_t>(res) + z0;
            const uint32_t q = a >> 5;
            Words4 v;
            if (WHOLE) {
                v = *reinterpret_cast<const Words4*>(fine + q);
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) v.v[j] = fine[min(q + j, last)];
            }
#pragma unroll
            for (int j = 0; j < 3; ++j) {
                const uint32_t row = __builtin_amdgcn_alignbit(v.v[j + 1], v.v[j], a);  // a's low 5 bits
                w[j] |= row;
                e[j] |= ~row;
            }
        }
    }
}

// The run of halo cells from cz0 on: the rows' pairs of bits folded and spread
// by one cell either way.  The other lane of the word holds the other half
// of the rows.
__device__ __forceinline__ uint32_t halo_run(uint32_t w[3], uint32_t cz0, uint32_t h, uint32_t len) {
#pragma unroll
    for (int j = 0; j < 3; ++j) {  // the other lane's rows (quad permutation 1, 0, 3, 2)
        w[j] |=
            static_cast<uint32_t>(__builtin_amdgcn_update_dpp(0, static_cast<int>(w[j]), 0xB1, 0xf, 0xf, false));
    }
    // pairs cz0 - 1 .. cz0 + 32 of the row (none before its first cell,
    // none past its end)
    uint64_t pairs = static_cast<uint64_t>(even_bits(w[0] | (w[0] >> 1))) |
                     (static_cast<uint64_t>(even_bits(w[1] | (w[1] >> 1))) << 16) |
                     (static_cast<uint64_t>(even_bits(w[2] | (w[2] >> 1))) << 32);
    if (cz0 == 0u) pairs <<= 1;
    const uint32_t n = h - cz0 + 1u;
    if (n < 34u) pairs &= (1ull << n) - 1ull;
    uint32_t run = static_cast<uint32_t>(pairs | (pairs >> 1) | (pairs >> 2));
    if (len < 32u) run &= (1u << len) - 1u;
    return run;
}

// Two lanes per word of the halo bits (32 consecutive cells in C order,
// whose rows may end inside the word).  The fine cells within kHaloReach = 2
// of a halo cell's 2 x 2 x 2 block are the blocks of its 3 x 3 x 3
// neighbourhood, so the word is the OR of 6 x 6 fine rows (each of the two
// lanes takes 18), whose pairs of bits are then folded once and spread by
// one cell either way.  Bound by the latency of the rows' loads, one
// dwordx4 each and all of a lane's in flight together.
// Four 128^3 grids: 35.5 us with a lane per cell and early exits, 8.6 us
// with a lane per word and a load per fine word, 4.5 us so.
// HALO and HOLES: which of the two to write.
template <bool HALO, bool HOLES>
__global__ __launch_bounds__(kHaloThreads) void halo_kernel(const uint32_t* __restrict__ bits, int res, int n_grids,
                                                            uint32_t words, uint32_t out_words,
                                                            uint32_t* __restrict__ out, uint32_t* __restrict__ holes) {
    const int64_t lane = static_cast<int64_t>(blockIdx.x) * kHaloThreads + threadIdx.x;
    const int64_t id = lane >> 1;
    const int half = static_cast<int>(lane & 1);
    const bool mine = id < static_cast<int64_t>(out_words) * n_grids;
    const int64_t grid = mine ? id / out_words : 0;
    const uint32_t first = mine ? static_cast<uint32_t>(id - grid * out_words) * 32u : 0u;
    const uint32_t* fine = bits + grid * words;
    const uint32_t h = static_cast<uint32_t>(res) >> 1;
    const uint32_t cells = h * h * h, last = words - 1u;
    uint32_t word = 0u, hole_word = 0u;
    // every lane takes every step (the two lanes of a word exchange their
    // halves): a step is a run of cells within one row
    uint32_t b = 0u;
    while (ballot(mine && b < 32u && first + b < cells) != 0ull) {
        const bool on = mine && b < 32u && first + b < cells;
        const uint32_t cell = on ? first + b : 0u;
        const uint32_t row = cell / h, cz0 = cell - row * h;
        const int cx = static_cast<int>(row / h), cy = static_cast<int>(row % h);
        const uint32_t len = min(32u - min(b, 31u), h - cz0);
        const uint32_t z0 = cz0 > 0u ? 2u * cz0 - 2u : 0u;  // first bit read of a row
        const int x0 = 2 * cx - kHaloReach + 3 * half;
        const int xl = min(max(x0 + 2, 0), res - 1), yl = min(2 * cy + 1 + kHaloReach, res - 1);
        const uint32_t end = static_cast<uint32_t>(xl * res + yl) * static_cast<uint32_t>(res) + z0;
        uint32_t w[3] = {0u, 0u, 0u}, e[3] = {0u, 0u, 0u};
        if (ballot((end >> 5) + 3u > last) == 0ull) {
            or_rows<true>(fine, last, res, x0, cy, z0, w, e);
        } else {
            or_rows<false>(fine, last, res, x0, cy, z0, w, e);
        }
        const uint32_t run = HALO ? halo_run(w, cz0, h, len) : 0u;
        const uint32_t hole_run = HOLES ? halo_run(e, cz0, h, len) : 0u;
        if (on) {
            word |= run << b;
            hole_word |= hole_run << b;
            b += len;
        }
    }
    if (mine && half == 0) {
        if (HALO) out[id] = word;
        if (HOLES) holes[id] = hole_word;
    }
}

// Halo bits of grids of 8^3 cells: a wave a grid, a lane a halo cell, whose 6 x
// 6 rows lie in a word each.  (Two lanes a word take its eight rows of four
// cells one after the other: skip buffers of 512 grids 26 us, 12.5 us so.  4^3
// cells would leave 56 lanes idle: 262,144 grids 78 us and 154 us.)
constexpr int kSmallHaloRes = 8;

__global__ __launch_bounds__(kHaloThreads) void halo_small_kernel(const uint32_t* __restrict__ bits,
                                                                  uint32_t* __restrict__ out) {
    constexpr int kRes = kSmallHaloRes, kWords = kRes * kRes * kRes / 32, kHalf = kRes / 2;
    static_assert(kHalf * kHalf * kHalf == kWave, "a lane a halo cell");
    const int lane = lane_id();
    const uint32_t* fine = bits + static_cast<int64_t>(blockIdx.x) * kWords;
    const int cx = lane / (kHalf * kHalf), cy = lane / kHalf % kHalf, cz = lane % kHalf;
    uint32_t any = 0u;
#pragma unroll
    for (int i = 0; i < 36; ++i) {
        const int x = min(max(2 * cx - kHaloReach + i / 6, 0), kRes - 1);
        const int y = min(max(2 * cy - kHaloReach + i % 6, 0), kRes - 1);
        const int b = (x * kRes + y) * kRes;
        any |= fine[b >> 5] >> (b & 31);
    }
    const int z0 = max(2 * cz - kHaloReach, 0), z1 = min(2 * cz + 1 + kHaloReach, kRes - 1);
    const uint64_t m = ballot((any & ((2u << z1) - (1u << z0))) != 0u);
    if (lane < 2) out[2 * static_cast<int64_t>(blockIdx.x) + lane] = static_cast<uint32_t>(m >> (32 * lane));
}

// Halo bits of every grid (res % 4 == 0) into `out` and hole bits into
// `holes`, either of them nullptr, on stream s.
inline void launch_halo(const uint32_t* bits, int res, int n_grids, uint32_t* out, uint32_t* holes, hipStream_t s) {
    const int64_t words = static_cast<int64_t>(res) * res * res / 32;
    const int64_t n = halo_words(res) * n_grids;
    if (holes == nullptr && res == kSmallHaloRes) {
        hipLaunchKernelGGL(halo_small_kernel, dim3(static_cast<unsigned>(n_grids)), dim3(kHaloThreads), 0, s, bits, out);
        return;
    }
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>((2 * n + kHaloThreads - 1) / kHaloThreads)),
                           dim3(kHaloThreads), 0, s, bits, res, n_grids, static_cast<uint32_t>(words),
                           static_cast<uint32_t>(halo_words(res)), out, holes);
    };
    if (holes == nullptr) launch(halo_kernel<true, false>);
    else if (out == nullptr) launch(halo_kernel<false, true>);
    else launch(halo_kernel<true, true>);
}

}  // namespace
