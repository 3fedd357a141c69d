// Exact integer scan turning per-ray counts into packed_info starts, shared
// by the compacting passes (marching, visibility pruning).  The counting
// kernels leave one int64 sum per workgroup; launch_starts turns them into
// each ray's start and the device-side total.
#pragma once

#include "common.h"

namespace {

using namespace nacc;
using namespace nacc::dev;

constexpr int kRaysPerBlock = 64;  // rays per workgroup of the counting passes

// Exclusive scan of n int64 values in place (exact, deterministic), in
// tiles of kScanTile values: one workgroup per tile adds its values, one
// workgroup scans the tile sums, and one workgroup per tile rewrites its
// values as offsets from its tile's offset.  Each thread of a tile takes a
// contiguous run of kScanPer values; the runs' sums are scanned in LDS.
constexpr int kScanThreads = 1024;
constexpr int kScanPer = 8;
constexpr int64_t kScanTile = static_cast<int64_t>(kScanThreads) * kScanPer;

__global__ __launch_bounds__(kScanThreads) void scan_tile_sums_kernel(const int64_t* __restrict__ v, int64_t n,
                                                                      int64_t* __restrict__ tile_sums) {
    __shared__ int64_t part[kScanThreads];
    const int t = threadIdx.x;
    const int64_t base = static_cast<int64_t>(blockIdx.x) * kScanTile;
    int64_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        const int64_t i = base + static_cast<int64_t>(k) * kScanThreads + t;  // coalesced
        if (i < n) s += v[i];
    }
    part[t] = s;
    __syncthreads();
    for (int off = kScanThreads / 2; off > 0; off >>= 1) {
        if (t < off) part[t] += part[t + off];
        __syncthreads();
    }
    if (t == 0) tile_sums[blockIdx.x] = part[0];
}

// tile_offsets: the scanned tile sums (nullptr: one tile, offset 0); total
// (nullable) receives the sum of all n values.
__global__ __launch_bounds__(kScanThreads) void scan_tiles_kernel(int64_t* __restrict__ v, int64_t n,
                                                                  const int64_t* __restrict__ tile_offsets,
                                                                  int64_t* __restrict__ total) {
    __shared__ int64_t part[kScanThreads];
    const int t = threadIdx.x;
    const int64_t a = static_cast<int64_t>(blockIdx.x) * kScanTile + static_cast<int64_t>(t) * kScanPer;
    int64_t run[kScanPer];
    int64_t s = 0;
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        run[k] = a + k < n ? v[a + k] : 0;
        s += run[k];
    }
    part[t] = s;
    __syncthreads();
    for (int off = 1; off < kScanThreads; off <<= 1) {
        const int64_t x = t >= off ? part[t - off] : 0;
        __syncthreads();
        part[t] += x;
        __syncthreads();
    }
    int64_t off = (tile_offsets != nullptr ? tile_offsets[blockIdx.x] : 0) + (part[t] - s);
#pragma unroll
    for (int k = 0; k < kScanPer; ++k) {
        if (a + k < n) v[a + k] = off;
        off += run[k];
    }
    if (total != nullptr && blockIdx.x == gridDim.x - 1 && t == kScanThreads - 1) *total = off;
}

// int64 scratch values scan_exclusive needs for n values (the tile sums).
inline int64_t scan_scratch_values(int64_t n) {
    const int64_t tiles = (n + kScanTile - 1) / kScanTile;
    return tiles > 1 ? tiles : 0;
}

// Launches the exclusive scan of v[0, n) on stream s; *total (nullable, on
// the device) receives the sum.  n <= kScanTile^2.
inline void scan_exclusive(int64_t* v, int64_t n, int64_t* total, int64_t* scratch, hipStream_t s) {
    const int64_t tiles = (n + kScanTile - 1) / kScanTile;
    if (tiles <= 1) {
        hipLaunchKernelGGL(scan_tiles_kernel, dim3(1), dim3(kScanThreads), 0, s, v, n, nullptr, total);
        return;
    }
    hipLaunchKernelGGL(scan_tile_sums_kernel, dim3(static_cast<unsigned>(tiles)), dim3(kScanThreads), 0, s, v, n,
                       scratch);
    hipLaunchKernelGGL(scan_tiles_kernel, dim3(1), dim3(kScanThreads), 0, s, scratch, tiles, nullptr, nullptr);
    hipLaunchKernelGGL(scan_tiles_kernel, dim3(static_cast<unsigned>(tiles)), dim3(kScanThreads), 0, s, v, n,
                       scratch, total);
}

// packed_info[r].start = offset of r's part (of `1 << log_part` rays, at most
// 64) + exclusive scan of the counts inside it (one wave = 64 rays).  Starts
// that do not fit int32 saturate; the fill pass then reports NACC_ECAPACITY.
__global__ __launch_bounds__(kRaysPerBlock) void finalize_starts_kernel(
    const int64_t* __restrict__ part_offsets, int log_part, int64_t n_rays, int32_t* __restrict__ packed_info) {
    const int64_t r = static_cast<int64_t>(blockIdx.x) * kRaysPerBlock + threadIdx.x;
    const int n = r < n_rays ? packed_info[2 * r + 1] : 0;
    const int before = wave_inclusive_sum(n) - n;
    const int part_before = __builtin_amdgcn_ds_bpermute(((lane_id() >> log_part) << log_part) << 2, before);
    if (r >= n_rays) return;
    const int64_t start = part_offsets[r >> log_part] + (before - part_before);
    packed_info[2 * r] = static_cast<int32_t>(min(start, static_cast<int64_t>(INT32_MAX)));
}

// The same and the total in one launch, for up to kMaxParts sums of
// `1 << log_part` rays each (at most 64): every workgroup of 256 rays adds up
// all sums before its own, which come from the L2 (64 KB at most), eight of
// each thread's in flight together.  4,096 sums: 6.1 us, where the scan and
// the starts took 5.9 + 6.0 us and a launch more; 16 sums: 2.1 us for 3.9 +
// 2.3 us.
constexpr int kStartsThreads = 256;
constexpr int64_t kMaxParts = 8192;
constexpr int kStartsUnroll = 8;

__global__ __launch_bounds__(kStartsThreads) void starts_kernel(const int64_t* __restrict__ part_sums, int log_part,
                                                                int64_t n_rays, int32_t* __restrict__ packed_info,
                                                                int64_t* __restrict__ total) {
    __shared__ double wave_before[kStartsThreads / kWave];
    __shared__ int wave_count[kStartsThreads / kWave];
    const int64_t first = static_cast<int64_t>(blockIdx.x) * kStartsThreads;
    const int64_t r = first + threadIdx.x;
    const int wave = uniform<int>(static_cast<int>(threadIdx.x) / kWave);
    const int n = r < n_rays ? packed_info[2 * r + 1] : 0;
    const int64_t n_before = first >> log_part;
    int64_t sum = 0;
    for (int64_t i = threadIdx.x; i < n_before; i += kStartsThreads * kStartsUnroll) {
#pragma unroll
        for (int u = 0; u < kStartsUnroll; ++u) {  // all in flight together
            const int64_t k = i + u * kStartsThreads;
            const int64_t v = part_sums[min(k, n_before - 1)];
            sum += k < n_before ? v : 0;
        }
    }
    // (2^19 rays of at most 2^31 samples: every sum is exact in FP64)
    const double wave_sums = wave_sum(static_cast<double>(sum));
    const int incl = wave_inclusive_sum(n);
    if (lane_id() == kWave - 1) {
        wave_before[wave] = wave_sums;
        wave_count[wave] = incl;
    }
    __syncthreads();
    double before = 0.0;
#pragma unroll
    for (int w = 0; w < kStartsThreads / kWave; ++w) before += wave_before[w];
    int64_t start = static_cast<int64_t>(before);
    for (int w = 0; w < wave; ++w) start += wave_count[w];
    if (total != nullptr && first + kStartsThreads >= n_rays && threadIdx.x == kStartsThreads - 1) {
        *total = start + incl;
    }
    start += incl - n;
    if (r < n_rays) packed_info[2 * r] = static_cast<int32_t>(min(start, static_cast<int64_t>(INT32_MAX)));
}

// Starts and total from the counts in packed_info and their sums over parts
// of `1 << log_part` consecutive rays (n_rays >= 1).  `sums` is followed by
// the scan's scratch, and overwritten, if there are more than kMaxParts.
inline void launch_starts(int64_t* sums, int64_t n_parts, int log_part, int64_t n_rays, int32_t* packed_info,
                          int64_t* total, hipStream_t s) {
    if (n_parts <= kMaxParts) {
        hipLaunchKernelGGL(starts_kernel,
                           dim3(static_cast<unsigned>((n_rays + kStartsThreads - 1) / kStartsThreads)),
                           dim3(kStartsThreads), 0, s, sums, log_part, n_rays, packed_info, total);
        return;
    }
    scan_exclusive(sums, n_parts, total, sums + n_parts, s);
    hipLaunchKernelGGL(finalize_starts_kernel, dim3(static_cast<unsigned>((n_rays + kRaysPerBlock - 1) / kRaysPerBlock)),
                       dim3(kRaysPerBlock), 0, s, sums, log_part, n_rays, packed_info);
}

inline int64_t num_blocks(int64_t n_rays) { return (n_rays + kRaysPerBlock - 1) / kRaysPerBlock; }

}  // namespace
