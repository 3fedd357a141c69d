// Occupancy-grid update on gfx950 (NerfAcc, Sec. 2.1: a binary grid cached
// and updated during training).  The update rule is delegated by the paper to
// Instant-NGP; it is read here as: decay every cell, take the maximum with
// fresh density samples at random jittered cell positions, threshold.
//
//   decay        occ[c] *= decay                       (streaming, float4)
//   sample_cells Philox4x64-10 per sample -> cell, jittered position
//   update_max   atomic max on the FP32 bit patterns (order-independent)
//   pack         one ballot per wavefront -> two 32-bit words of bits
#include <algorithm>
#include <cmath>

#include "common.h"
#include "halo.h"

#pragma clang fp contract(off)

namespace {

using namespace nacc;
using namespace nacc::dev;

constexpr int kThreads = 256;

__global__ __launch_bounds__(kThreads) void decay_kernel(float* __restrict__ occ, int64_t n, float decay) {
    const int64_t n4 = n / 4;
    float4* occ4 = reinterpret_cast<float4*>(occ);
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kThreads;
    for (int64_t i = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; i < n4; i += stride) {
        float4 v = occ4[i];
        v.x = v.x * decay;
        v.y = v.y * decay;
        v.z = v.z * decay;
        v.w = v.w * decay;
        occ4[i] = v;
    }
    for (int64_t i = 4 * n4 + static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x; i < n; i += stride) {
        occ[i] = occ[i] * decay;
    }
}

// Philox4x64-10 (Salmon, Moraes, Dror, Shaw, SC 2011): ten rounds of two
// 64x64 -> 128-bit products with the published multipliers, keys bumped by
// the published Weyl constants between rounds.
struct U64x4 {
    uint64_t v[4];
};

__device__ __forceinline__ U64x4 philox4x64_10(uint64_t c0, uint64_t c1, uint64_t c2, uint64_t c3, uint64_t k0,
                                               uint64_t k1) {
    constexpr uint64_t kMul0 = 0xD2E7470EE14C6C93ull;
    constexpr uint64_t kMul1 = 0xCA5A826395121157ull;
    constexpr uint64_t kWeyl0 = 0x9E3779B97F4A7C15ull;
    constexpr uint64_t kWeyl1 = 0xBB67AE8584CAA73Bull;
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        const uint64_t lo0 = kMul0 * c0, hi0 = __umul64hi(kMul0, c0);
        const uint64_t lo1 = kMul1 * c2, hi1 = __umul64hi(kMul1, c2);
        const uint64_t n0 = hi1 ^ c1 ^ k0;
        const uint64_t n2 = hi0 ^ c3 ^ k1;
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
        k0 += kWeyl0;
        k1 += kWeyl1;
    }
    return U64x4{{c0, c1, c2, c3}};
}

__global__ __launch_bounds__(kThreads) void sample_cells_kernel(uint64_t seed, uint64_t step,
                                                                 const uint64_t* __restrict__ step_dev, int64_t n,
                                                                 int res,
                                                                 uint64_t n_cells, float lo0, float lo1, float lo2,
                                                                 float h0, float h1, float h2, int cascade,
                                                                 int32_t* __restrict__ cells,
                                                                 float* __restrict__ positions) {
    const int64_t q = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (q >= n) return;
    const uint64_t update = step_dev != nullptr ? *step_dev : step;
    const U64x4 r = philox4x64_10(static_cast<uint64_t>(q), update, 0, 0, seed, 0);
    const uint64_t cell = ((r.v[0] >> 32) * n_cells) >> 32;
    cells[q] = static_cast<int32_t>(cell);
    const uint64_t per_grid = static_cast<uint64_t>(res) * res * res;
    const int level = cascade ? static_cast<int>(cell / per_grid) : 0;
    const uint64_t local = cell % per_grid;
    const int j0 = static_cast<int>(local / (static_cast<uint64_t>(res) * res));
    const int j1 = static_cast<int>((local / res) % res);
    const int j2 = static_cast<int>(local % res);
    const float jit0 = static_cast<float>(r.v[1] >> 40) * 0x1p-24f;
    const float jit1 = static_cast<float>(r.v[2] >> 40) * 0x1p-24f;
    const float jit2 = static_cast<float>(r.v[3] >> 40) * 0x1p-24f;
    positions[3 * q] = ldexpf(lo0 + (static_cast<float>(j0) + jit0) * h0, level);
    positions[3 * q + 1] = ldexpf(lo1 + (static_cast<float>(j1) + jit1) * h1, level);
    positions[3 * q + 2] = ldexpf(lo2 + (static_cast<float>(j2) + jit2) * h2, level);
}

// max on FP32 through integer atomics: non-negative floats order like their
// signed bit patterns, negative floats order in reverse of their unsigned
// bit patterns, and every non-negative pattern is below every negative one
// as unsigned.  NaN values are skipped.
__global__ __launch_bounds__(kThreads) void update_max_kernel(float* __restrict__ occ,
                                                               const int32_t* __restrict__ cells,
                                                               const float* __restrict__ values, int64_t n,
                                                               int64_t n_cells) {
    const int64_t q = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (q >= n) return;
    const int32_t c = cells[q];
    const float v = values[q];
    if (c < 0 || c >= n_cells || v != v) return;
    if (!signbit(v)) {
        atomicMax(reinterpret_cast<int*>(occ) + c, __float_as_int(v));
    } else {
        atomicMin(reinterpret_cast<unsigned int*>(occ) + c, __float_as_uint(v));
    }
}

// A wave packs kPackRuns runs of 64 cells, one ballot each, all their loads
// in flight together; its words are stored in one piece, lane i the run's
// half i.  Bound by HBM: 8.4 M cells 15 us with one run per wave -> 6.1 us.
constexpr int kPackRuns = 16;

__global__ __launch_bounds__(kThreads) void pack_kernel(const float* __restrict__ occ, int64_t n_cells,
                                                         float threshold, uint32_t* __restrict__ bits) {
    const int lane = lane_id();
    const int64_t first = (static_cast<int64_t>(blockIdx.x) * (kThreads / kWave) +
                           uniform<int>(static_cast<int>(threadIdx.x) / kWave)) *
                          (kPackRuns * kWave);
    float v[kPackRuns];
#pragma unroll
    for (int k = 0; k < kPackRuns; ++k) {
        const int64_t i = first + k * kWave + lane;
        v[k] = i < n_cells ? occ[i] : threshold;  // not above the threshold
    }
    uint32_t word = 0u;
#pragma unroll
    for (int k = 0; k < kPackRuns; ++k) {
        const uint64_t m = ballot(v[k] > threshold);
        if (lane >> 1 == k) word = static_cast<uint32_t>((lane & 1) != 0 ? m >> 32 : m);
    }
    const int64_t w = first / 32 + lane;
    if (lane < 2 * kPackRuns && w < n_cells / 32) bits[w] = word;
}

// Skip field, per grid: one byte per coarse cell of 4x4x4 fine cells (C
// order), min(NACC_SKIP_CAP, Chebyshev distance in coarse cells to the
// nearest coarse cell that holds an occupied fine cell).  The L-infinity
// distance separates over the axes,
//   dist(a,b,c) = min_da max(|da|, min_db max(|db|, min_dc max(|dc|, e))),
// e = 0 at occupied coarse cells and the cap elsewhere.  Grids of up to
// kPlaneCells coarse cells per axis (res <= 512) are built plane by plane in
// LDS: the coarse occupancy of a plane of constant x and its distances along
// z and y in one launch, those along x in planes of constant y in another.
// Bound by latency (a few dependent LDS reads per cell and axis): four grids
// of 128^3 cells 5.6 + 3.6 us, 3.3 + 3 x 5.5 us with a launch for the occupancy and
// one per axis, each reading its window from memory; larger grids, and many
// small ones (by_planes), still are.

// Coarse occupancy: one lane per coarse cell, 16 fine-row reads (the 4 bits
// of a row lie in one word since 4 | res).
__global__ __launch_bounds__(kThreads) void coarse_kernel(const uint32_t* __restrict__ bits, int res, int n_grids,
                                                          uint32_t words, uint8_t* __restrict__ out) {
    const int c = res / 4;
    const int64_t per_grid = static_cast<int64_t>(c) * c * c;
    const int64_t id = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (id >= per_grid * n_grids) return;
    const int grid = static_cast<int>(id / per_grid);
    const int64_t cell = id % per_grid;
    const int cx = static_cast<int>(cell / (static_cast<int64_t>(c) * c));
    const int cy = static_cast<int>((cell / c) % c);
    const int cz = static_cast<int>(cell % c);
    const uint32_t* fine = bits + static_cast<int64_t>(grid) * words;
    uint32_t any = 0u;
    for (int x = 4 * cx; x < 4 * cx + 4; ++x) {
        for (int y = 4 * cy; y < 4 * cy + 4; ++y) {
            const int64_t b = (static_cast<int64_t>(x) * res + y) * res + 4 * cz;
            any |= (fine[b >> 5] >> (b & 31)) & 0xFu;
        }
    }
    out[id] = any != 0u ? 0 : NACC_SKIP_CAP;
}

// Whether the coarse cell (x, y, z) holds an occupied fine cell.
__device__ __forceinline__ bool coarse_occupied(const uint32_t* __restrict__ fine, int res, int x, int y, int z) {
    uint32_t any = 0u;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const uint32_t b = (static_cast<uint32_t>(4 * x + (i >> 2)) * static_cast<uint32_t>(res) +
                            static_cast<uint32_t>(4 * y + (i & 3))) *
                               static_cast<uint32_t>(res) +
                           static_cast<uint32_t>(4 * z);
        any |= fine[b >> 5] >> (b & 31u);
    }
    return (any & 0xFu) != 0u;
}

// One axis of the distance of a cell at position `pos` of `c`, from its value
// and its neighbours' at +-t `stride` in LDS, kWindow values of t at a time,
// their reads in flight together.  A neighbour past the end is replaced by
// the last cell, which lies nearer and so never lowers the minimum.
constexpr int kWindow = 5;
static_assert(NACC_SKIP_CAP % kWindow == 0, "whole windows up to the cap");

__device__ __forceinline__ uint8_t axis_distance(const uint8_t* plane, int i, int pos, int c, int stride) {
    int best = plane[i];
    for (int t0 = 1; t0 < best; t0 += kWindow) {  // best <= the cap
        int v[kWindow];
#pragma unroll
        for (int k = 0; k < kWindow; ++k) {
            const int t = t0 + k;
            v[k] = min(static_cast<int>(plane[i - min(t, pos) * stride]),
                       static_cast<int>(plane[i + min(t, c - 1 - pos) * stride]));
        }
#pragma unroll
        for (int k = 0; k < kWindow; ++k) best = min(best, max(t0 + k, v[k]));
    }
    return static_cast<uint8_t>(best);
}

constexpr int kPlaneCells = 128;
constexpr int kPlaneThreads = 1024;  // at most; a thread a cell of smaller planes

int plane_threads(int c) { return std::min(kPlaneThreads, (c * c + kWave - 1) / kWave * kWave); }

// A workgroup a plane pays while the plane has some 128 cells, or the
// workgroups are few enough to be there at once.  Build of the buffer by planes
// and by the passes per axis: 64 grids of 64^3 cells 16 and 27 us, of 16^3 15 and
// 20; 512 grids of 48^3 45 and 55 us; 1,024 of 16^3 27 and 24, 2,048 of 32^3 84 and
// 70, 8,192 of 16^3 154 and 84.  A launch holds less than 2^32 threads.
bool by_planes(int c, int64_t planes) {
    return c <= kPlaneCells && (c * c >= 128 || planes <= 2048) &&
           planes * plane_threads(c) < (int64_t{1} << 32);
}

// Workgroup grid c + x: occupancy, then distances along z and y.
__global__ __launch_bounds__(kPlaneThreads) void skip_planes_kernel(const uint32_t* __restrict__ bits, int res,
                                                                    uint32_t words, uint8_t* __restrict__ out) {
    __shared__ uint8_t a[kPlaneCells * kPlaneCells], b[kPlaneCells * kPlaneCells];
    const int c = res / 4, n = c * c, n_threads = static_cast<int>(blockDim.x);
    const int x = static_cast<int>(blockIdx.x) % c;
    const uint32_t* fine = bits + static_cast<int64_t>(blockIdx.x / static_cast<unsigned>(c)) * words;
    for (int i = threadIdx.x; i < n; i += n_threads) {
        a[i] = coarse_occupied(fine, res, x, i / c, i % c) ? 0 : NACC_SKIP_CAP;
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += n_threads) b[i] = axis_distance(a, i, i % c, c, 1);
    __syncthreads();
    uint8_t* dst = out + static_cast<int64_t>(blockIdx.x) * n;
    for (int i = threadIdx.x; i < n; i += n_threads) dst[i] = axis_distance(b, i, i / c, c, c);
}

// Workgroup grid c + y: distances along x.
__global__ __launch_bounds__(kPlaneThreads) void skip_x_kernel(const uint8_t* __restrict__ in, int c,
                                                               uint8_t* __restrict__ out) {
    __shared__ uint8_t a[kPlaneCells * kPlaneCells];
    const int n = c * c, n_threads = static_cast<int>(blockDim.x);
    const int64_t first = static_cast<int64_t>(blockIdx.x / static_cast<unsigned>(c)) * n * c +
                          static_cast<int64_t>(blockIdx.x % static_cast<unsigned>(c)) * c;
    for (int i = threadIdx.x; i < n; i += n_threads) a[i] = in[first + static_cast<int64_t>(i / c) * n + i % c];
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += n_threads) {
        out[first + static_cast<int64_t>(i / c) * n + i % c] = axis_distance(a, i, i / c, c, c);
    }
}

// One axis of the distance: out = min over |t| <= cap of max(|t|, in[cell + t
// along the axis]), inside the grid.  stride: cells between neighbours along
// the axis (c^2, c or 1).
__global__ __launch_bounds__(kThreads) void distance_pass_kernel(const uint8_t* __restrict__ in, int c,
                                                                 int64_t n_cells, int64_t stride,
                                                                 uint8_t* __restrict__ out) {
    const int64_t id = static_cast<int64_t>(blockIdx.x) * kThreads + threadIdx.x;
    if (id >= n_cells) return;
    const int pos = static_cast<int>((id / stride) % c);
    int best = in[id];
    for (int t = 1; t <= NACC_SKIP_CAP && t < best; ++t) {
        const int lo = pos - t, hi = pos + t;
        int v = NACC_SKIP_CAP;
        if (lo >= 0) v = min(v, static_cast<int>(in[id - t * stride]));
        if (hi < c) v = min(v, static_cast<int>(in[id + t * stride]));
        best = min(best, max(t, v));
    }
    out[id] = static_cast<uint8_t>(best);
}

unsigned blocks_for(int64_t n) { return static_cast<unsigned>((n + kThreads - 1) / kThreads); }

}  // namespace

extern "C" {

int nacc_grid_decay(float* occ, int64_t n_cells, float decay, void* stream) {
    clear_error();
    NACC_REQUIRE(n_cells >= 0, NACC_EINVAL, "n_cells < 0");
    NACC_REQUIRE(n_cells == 0 || occ != nullptr, NACC_EINVAL, "occ must be non-NULL");
    NACC_REQUIRE(reinterpret_cast<uintptr_t>(occ) % 16 == 0, NACC_EINVAL, "occ must be 16-byte aligned");
    if (n_cells == 0) return NACC_OK;
    const int64_t work = (n_cells + 3) / 4;
    const unsigned nb = static_cast<unsigned>(std::min<int64_t>(blocks_for(work), 8192));
    hipLaunchKernelGGL(decay_kernel, dim3(nb), dim3(kThreads), 0, as_stream(stream), occ, n_cells, decay);
    return check_launch("grid decay");
}

int nacc_grid_sample_cells(uint64_t seed, uint64_t step, const uint64_t* step_dev, int64_t n,
                           const nacc_grid_desc* grid, int32_t levels, int32_t* cells, float* positions,
                           void* stream) {
    clear_error();
    NACC_REQUIRE(grid != nullptr, NACC_EINVAL, "grid must be non-NULL");
    NACC_REQUIRE(n >= 0 && n <= INT32_MAX, NACC_EINVAL, "n = %lld out of [0, 2^31-1]", static_cast<long long>(n));
    NACC_REQUIRE(n == 0 || (cells != nullptr && positions != nullptr), NACC_EINVAL, "outputs must be non-NULL");
    NACC_REQUIRE(grid->res >= 1 && grid->res <= 1024, NACC_EINVAL, "grid res = %d out of [1, 1024]", grid->res);
    const bool cascade = grid->lookup == NACC_LOOKUP_CASCADE;
    NACC_REQUIRE(levels >= 1 && (!cascade || levels <= 16), NACC_EINVAL, "levels = %d out of [1, %s]", levels,
                 cascade ? "16" : "2^31");
    const uint64_t n_cells = static_cast<uint64_t>(grid->res) * grid->res * grid->res * levels;
    NACC_REQUIRE(n_cells <= static_cast<uint64_t>(INT32_MAX), NACC_ESHAPE, "too many cells for int32 indices");
    for (int i = 0; i < 3; ++i) {
        NACC_REQUIRE(std::isfinite(grid->lo[i]) && std::isfinite(grid->hi[i]) && grid->lo[i] < grid->hi[i],
                     NACC_EINVAL, "grid box axis %d is empty or not finite", i);
    }
    if (n == 0) return NACC_OK;
    float h[3];
    for (int i = 0; i < 3; ++i) {
        h[i] = static_cast<float>((static_cast<double>(grid->hi[i]) - static_cast<double>(grid->lo[i])) /
                                  static_cast<double>(grid->res));
    }
    hipLaunchKernelGGL(sample_cells_kernel, dim3(blocks_for(n)), dim3(kThreads), 0, as_stream(stream), seed, step,
                       step_dev, n, grid->res, n_cells, grid->lo[0], grid->lo[1], grid->lo[2], h[0], h[1], h[2],
                       cascade ? 1 : 0, cells, positions);
    return check_launch("grid sample cells");
}

int nacc_grid_update_max(float* occ, const int32_t* cells, const float* values, int64_t n, int64_t n_cells,
                         void* stream) {
    clear_error();
    NACC_REQUIRE(n >= 0 && n_cells >= 0, NACC_EINVAL, "negative size");
    NACC_REQUIRE(n == 0 || (occ != nullptr && cells != nullptr && values != nullptr), NACC_EINVAL,
                 "arguments must be non-NULL");
    if (n == 0) return NACC_OK;
    hipLaunchKernelGGL(update_max_kernel, dim3(blocks_for(n)), dim3(kThreads), 0, as_stream(stream), occ, cells,
                       values, n, n_cells);
    return check_launch("grid update max");
}

int64_t nacc_grid_skip_bytes(const nacc_grid_desc* grid) {
    if (grid == nullptr || grid->res < 4 || grid->res % 4 != 0 || grid->n_grids < 1) return 0;
    return halo_offset(grid->res, grid->n_grids) + halo_words(grid->res) * 4 * grid->n_grids;
}

int nacc_grid_build_skip(const uint32_t* bits, const nacc_grid_desc* grid, uint8_t* skip, void* stream) {
    clear_error();
    NACC_REQUIRE(grid != nullptr, NACC_EINVAL, "grid must be non-NULL");
    NACC_REQUIRE(grid->res >= 4 && grid->res <= 1024 && grid->res % 4 == 0, NACC_ENOTSUP,
                 "the skip field needs res %% 4 == 0 (res = %d)", grid->res);
    NACC_REQUIRE(grid->n_grids >= 1, NACC_EINVAL, "n_grids = %d < 1", grid->n_grids);
    const int64_t cells = static_cast<int64_t>(grid->res) * grid->res * grid->res;
    NACC_REQUIRE(cells % 32 == 0, NACC_ESHAPE, "res^3 is not a multiple of 32");
    NACC_REQUIRE(bits != nullptr && skip != nullptr, NACC_EINVAL, "bits and skip must be non-NULL");
    NACC_REQUIRE(reinterpret_cast<uintptr_t>(skip) % 4 == 0, NACC_EINVAL, "skip must be 4-byte aligned");
    const int c = grid->res / 4;
    const int64_t n = static_cast<int64_t>(c) * c * c * grid->n_grids;
    uint8_t* field = skip;
    uint8_t* scratch = skip + n;
    hipStream_t s = as_stream(stream);
    uint32_t* halo = reinterpret_cast<uint32_t*>(skip + halo_offset(grid->res, grid->n_grids));
    const int64_t n_planes = static_cast<int64_t>(c) * grid->n_grids;
    if (by_planes(c, n_planes)) {
        const dim3 planes(static_cast<unsigned>(n_planes)), threads(static_cast<unsigned>(plane_threads(c)));
        hipLaunchKernelGGL(skip_planes_kernel, planes, threads, 0, s, bits, grid->res,
                           static_cast<uint32_t>(cells / 32), scratch);
        int st = check_launch("grid skip planes");
        if (st != NACC_OK) return st;
        hipLaunchKernelGGL(skip_x_kernel, planes, threads, 0, s, scratch, c, field);
        st = check_launch("grid skip distance");
        if (st != NACC_OK) return st;
        launch_halo(bits, grid->res, grid->n_grids, halo, nullptr, s);
        return check_launch("grid skip halo");
    }
    hipLaunchKernelGGL(coarse_kernel, dim3(blocks_for(n)), dim3(kThreads), 0, s, bits, grid->res, grid->n_grids,
                       static_cast<uint32_t>(cells / 32), scratch);
    int st = check_launch("grid skip coarse");
    if (st != NACC_OK) return st;
    const int64_t strides[3] = {1, c, static_cast<int64_t>(c) * c};
    uint8_t* src = scratch;
    uint8_t* dst = field;
    for (int axis = 0; axis < 3; ++axis) {  // z, y, x: the third pass lands in `field`
        hipLaunchKernelGGL(distance_pass_kernel, dim3(blocks_for(n)), dim3(kThreads), 0, s, src, c, n,
                           strides[axis], dst);
        st = check_launch("grid skip distance");
        if (st != NACC_OK) return st;
        uint8_t* t = src;
        src = dst;
        dst = t;
    }
    launch_halo(bits, grid->res, grid->n_grids, halo, nullptr, s);
    return check_launch("grid skip halo");
}

int nacc_grid_pack(const float* occ, int64_t n_cells, float threshold, uint32_t* bits, void* stream) {
    clear_error();
    NACC_REQUIRE(n_cells >= 0 && n_cells % 32 == 0, NACC_ESHAPE, "n_cells = %lld must be a multiple of 32",
                 static_cast<long long>(n_cells));
    NACC_REQUIRE(n_cells == 0 || (occ != nullptr && bits != nullptr), NACC_EINVAL, "arguments must be non-NULL");
    if (n_cells == 0) return NACC_OK;
    hipLaunchKernelGGL(pack_kernel, dim3(blocks_for((n_cells + kPackRuns - 1) / kPackRuns)), dim3(kThreads), 0,
                       as_stream(stream), occ, n_cells, threshold, bits);
    return check_launch("grid pack");
}

}  // extern "C"
