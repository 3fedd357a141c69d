// Occupancy-grid ray marching on gfx950 (NerfAcc, Sec. 2.1 "Ray Marching",
// "Pruning Empty and Occluded Regions", "GPU Memory Efficiency").
//
// Samples are the lattice intervals of each ray whose midpoint lies in an
// occupied cell.  Empty space is pruned while marching, so the ragged output
// is produced by three steps:
//   count   every ray's samples, one sum per part of 4 to 64 rays, and, where a
//           workspace is given, a 64-bit mask of the samples of every chunk of 64
//           candidates (the first kMaxMaskChunks of a ray);
//   starts  exclusive sums of the parts and of the counts inside them ->
//           packed_info (start, count) and the total (scan.h);
//   fill    the samples of the masks, at their offsets; without masks, and past
//           the chunks that have them, the rays are traversed again.
//
// Which kernels run:
//   uniform steps, box lookup, halo bits (the skip buffer's, or built for the
//     call, halo.h): count_box_kernel, segments of many rays tested and looked
//     up together;
//   other uniform steps: count_uniform_kernel, a wavefront per ray whose lanes
//     test 64 consecutive candidates at once; the cascades and the contraction
//     pass over stretches that the skip buffer's distances clear;
//   every uniform fill: fill_uniform_kernel, up to 8 rays a wave;
//   cone steps with halo bits: count_cone_kernel (chunks, segments and lookups
//     of many rays, 64 at a time) and fill_cone_rays_kernel;
//   cone steps without (a few rays over many grids): a lane per chunk,
//     cone_starts_kernel, count_cone_chunks_kernel, cone_counts_kernel,
//     fill_cone_chunks_kernel; without a workspace fill_cone_kernel, a lane per
//     ray.
// What a test leaves out is proven empty with the FP32 rounding of positions
// allowed for, so that every way gives exactly the samples of the plain
// traversal.
//
// All lattice arithmetic follows the FP32 contract in nacc.h: this file is
// compiled with -ffp-contract=off and `fp contract(off)`, and uses only
// correctly rounded + - * / sqrt, min/max, ldexp and float->int truncation of
// non-negative values.
#include <cmath>
#include <type_traits>

#include "common.h"
#include "fill_list.h"
#include "halo.h"
#include "lattice.h"
#include "scan.h"

#pragma clang fp contract(off)

namespace {

using namespace nacc;
using namespace nacc::dev;

// Per-ray constants of the skip-field test.
//   slack_x: allowance for the FP32 rounding of sample positions: two
//            positions of the ray differ by at most |d_i| |tm_k - tm_0| plus
//            slack_x on every axis (a few ulps of the largest coordinate the
//            ray reaches, taken generously);
//   inv_v:   1 / (fine cells per unit t on the fastest axis, at level 0);
//   inv_dmax: 1 / max_i |d_i|.
//   contraction lookup: t_out, from which on the ray moves away from the
//   origin (past its closest approach, rounded up), |d| rounded up, the
//   largest |o_i|, |d_i| and the grid's largest cells-per-unit scale.
struct SkipRay {
    float slack_x;
    float slack_s;  // slack_x in fine cells at level 0
    float inv_v;
    float inv_dmax;
    float t_out, dnorm, omax, dmax, smax;
};

__device__ __forceinline__ SkipRay skip_ray(const GridK& g, const float o[3], const float d[3], float t_far) {
    SkipRay k;
    const float omax = fmaxf(fmaxf(fabsf(o[0]), fabsf(o[1])), fabsf(o[2]));
    const float dmax = fmaxf(fmaxf(fabsf(d[0]), fabsf(d[1])), fabsf(d[2]));
    k.slack_x = (omax + dmax * fabsf(t_far) + 1.0f) * 0x1p-20f;
    const float smax = fmaxf(fmaxf(g.s[0], g.s[1]), g.s[2]);
    k.slack_s = smax * k.slack_x;
    k.inv_v = 1.0f / fmaxf(fmaxf(g.s[0] * fabsf(d[0]), g.s[1] * fabsf(d[1])), g.s[2] * fabsf(d[2]));
    k.inv_dmax = 1.0f / dmax;
    const float dd = (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2];
    const float od = (o[0] * d[0] + o[1] * d[1]) + o[2] * d[2];
    const float t_star = -od / dd;
    k.t_out = t_star + (fabsf(t_star) + 1.0f) * 0x1p-16f;
    k.dnorm = sqrtf(dd) * (1.0f + 0x1p-18f);
    k.omax = omax;
    k.dmax = dmax;
    k.smax = smax;
    return k;
}

// Contraction lookup: the end of the stretch past tm whose candidates all
// map to empty fine cells.  The contraction c(x) = (2 - 1/|x|) x/|x| is
// Lipschitz with constant L(r) = (2 - 1/r)/r on |x| >= r >= 1 (its
// derivative stretches tangential directions by that factor and the radial
// one by 1/r^2 <= L(r); L <= 1 everywhere).  Past the closest approach |x|
// only grows along the ray, so candidates a distance D_t further along t
// map within L(r) |d| D_t of c(x(tm)), r a lower bound of |x(tm)|; before
// it L = 1.  The byte `dist` guarantees empty fine cells within
// 4 (dist - 1) cells on every axis; the stretch is kept inside that after
// allowing for the FP32 rounding of positions (a few ulps of the largest
// coordinate reached, at most 2 tm + 1 along the ray: the stretch is capped
// there) and of the contraction (2^-16 in contracted units).
__device__ __forceinline__ float skip_end_contract(const SkipRay& k, const Probe& q, int dist, float tm, int res) {
    float lip = 1.0f;
    if (tm > k.t_out) {
        const float t_reach = 2.0f * fabsf(tm) + 1.0f;
        const float slack = (k.omax + k.dmax * t_reach + 1.0f) * 0x1p-20f;
        const float r = q.m * (1.0f - 0x1p-18f) - 2.0f * slack;
        if (r > 1.0f) lip = ((2.0f - 1.0f / r) / r) * (1.0f + 0x1p-18f);
    }
    const float slack_pos = (k.omax + k.dmax * (2.0f * fabsf(tm) + 1.0f) + 1.0f) * 0x1p-20f;
    const float slack_cells = k.smax * 3.5f * (lip * slack_pos + 0x1p-16f) + static_cast<float>(res) * 0x1p-18f;
    const float budget = 4.0f * static_cast<float>(dist - 1) - slack_cells;
    float span = budget / (k.smax * lip * k.dnorm);
    span = fminf(span, fabsf(tm) + 1.0f);  // the reach the slack allows for
    span = span * (1.0f - 0x1p-10f) - fabsf(tm) * 0x1p-21f;
    return (dist >= 2 && span > 0.0f) ? tm + span : -INFINITY;
}

// End (in t) of the stretch past the candidate midpoint tm over which every
// candidate midpoint of the ray falls in an empty fine cell, from the skip
// byte `dist` of tm's coarse cell (probe q); -inf if there is none.  The
// byte bounds the stretch at 4 (dist - 1) fine cells on every axis of q's
// grid level; a cascade stretch also ends before the point could change
// level.  Rounding margins keep the bound strict.
template <int LOOKUP>
__device__ __forceinline__ float skip_end_at(const GridK& g, const SkipRay& k, const Probe& q, int dist, float tm) {
    if (LOOKUP == NACC_LOOKUP_CONTRACT) return skip_end_contract(k, q, dist, tm, g.res);
    // fine cells at level l are 2^l times larger: the slack in fine cells
    // shrinks and the stretch in t grows by 2^l
    const float budget =
        4.0f * static_cast<float>(dist - 1) - (ldexpf(k.slack_s, -q.level) + static_cast<float>(g.res) * 0x1p-18f);
    float span = ldexpf(budget * k.inv_v, q.level);
    if (LOOKUP == NACC_LOOKUP_CASCADE) {
        float room = INFINITY;
        if (q.level < g.n_grids - 1) room = fminf(room, ldexpf(g.base, q.level) - q.m);
        if (q.level > 0) room = fminf(room, q.m - ldexpf(g.base, q.level - 1));
        span = fminf(span, (room - k.slack_x) * k.inv_dmax);
    }
    span = span * (1.0f - 0x1p-10f) - fabsf(tm) * 0x1p-21f;
    return (dist >= 2 && span > 0.0f) ? tm + span : -INFINITY;
}

// DPP move that leaves a lane's own value where the source lane is out of
// range or its row is masked off (the identity for max).
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ float dpp_or_self(float v) {
    const int b = __builtin_bit_cast(int, v);
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(b, b, CTRL, ROW_MASK, 0xf, false));
}

// Maximum over the 64 lanes (every lane active): prefix maxima within each
// row of 16 lanes, then the row maxima carried by two row broadcasts.
__device__ __forceinline__ float wave_max(float x) {
    x = fmaxf(x, dpp_or_self<kRowShr1>(x));
    x = fmaxf(x, dpp_or_self<kRowShr2>(x));
    x = fmaxf(x, dpp_or_self<kRowShr4>(x));
    x = fmaxf(x, dpp_or_self<kRowShr8>(x));
    x = fmaxf(x, dpp_or_self<kRowBcast15, 0xa>(x));
    x = fmaxf(x, dpp_or_self<kRowBcast31, 0xc>(x));
    return read_lane(x, kWave - 1);
}

// Chunk masks of the count pass, one per lane: lane j holds the ballot of
// chunk j (as two 32-bit halves).  The chunk index and the ballot are
// wave-uniform, so the ballot is written into lane j directly.
struct ChunkMasks {
    int lo = 0, hi = 0;
    __device__ __forceinline__ void keep(int chunk, uint64_t m) {
        if (chunk < kWave) {
            const uint32_t m_lo = static_cast<uint32_t>(m), m_hi = static_cast<uint32_t>(m >> 32);
            // one scalar operand per instruction: the lane select goes in m0
            asm volatile("v_writelane_b32 %0, %1, m0" : "+v"(lo) : "s"(m_lo), "{m0}"(chunk));
            asm volatile("v_writelane_b32 %0, %1, m0" : "+v"(hi) : "s"(m_hi), "{m0}"(chunk));
        }
    }
    __device__ __forceinline__ uint64_t mine() const {
        return (static_cast<uint64_t>(static_cast<uint32_t>(hi)) << 32) | static_cast<uint32_t>(lo);
    }
};

// Uniform steps without the skip field, two chunks of 64 candidates per
// iteration: both chunks' grid words are loaded before either is tested, so
// each wave keeps two lookups in flight instead of waiting on one at a time
// (a chunk past the ray's end is looked up and ignored; its cell indices are
// clamped into the grid like any other).  Same samples, same order, same
// masks as one chunk at a time.
template <int LOOKUP, bool FILL>
__device__ __forceinline__ int march_ray_uniform_x2(
    int64_t r, const RaySpan& span, const uint32_t* __restrict__ bits, const GridK& g, const StepK& p, int64_t start,
    int limit, int64_t capacity, int32_t* __restrict__ ray_indices, float* __restrict__ t_starts,
    float* __restrict__ t_ends, bool& overflow, uint64_t* __restrict__ masks, int n_masks, int first_chunk, int count0) {
    if (!span.valid) return 0;
    const int lane = lane_id();
    const float* o = span.o;
    const float* d = span.d;
    const uint32_t word0 = span.word0;
    const float t_near = span.t_near, t_far = span.t_far;
    ChunkMasks my_masks;  // count pass
    int count = count0;
    bool done = false;
    for (int k0 = first_chunk * kWave; k0 < kMaxCandidates && !done; k0 += 2 * kWave) {
        float t0[2], t1[2];
        uint64_t live[2];  // ballots of t0 < t_far
        uint64_t ms[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int k = k0 + u * kWave + lane;
            t0[u] = t_near + static_cast<float>(k) * p.dt;
            live[u] = ballot(t0[u] < t_far);
            t1[u] = t_near + static_cast<float>(k + 1) * p.dt;
        }
        if (live[0] == 0ull) break;  // t_k is non-decreasing in k
        // both words are loaded, and both ballots taken, before any branch
        // on them (a ballot cannot move into a branch)
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const float tm = (t0[u] + t1[u]) * 0.5f;
            const Probe q = probe<LOOKUP>(g, word0, o[0] + d[0] * tm, o[1] + d[1] * tm, o[2] + d[2] * tm);
            const uint32_t w = grid_word(grid_rsrc(bits, g), q.word);  // every lane: the index is clamped into the grid
            // ballots of plain comparisons, combined as masks (a ballot of
            // a combined condition costs two more vector instructions)
            ms[u] = live[u] & ballot(((w >> q.bit) & 1u) != 0u);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int chunk = k0 / kWave + u;
            if (u == 1 && (live[1] == 0ull || k0 + kWave >= kMaxCandidates)) {
                done = true;
                break;
            }
            const uint64_t m = ms[u];
            const bool hit = ((m >> lane) & 1ull) != 0ull;
            if (!FILL) my_masks.keep(chunk, m);
            if (FILL && hit) {
                const int idx = count + bits_below(m);
                if (idx < limit) {
                    const int64_t pos = start + idx;
                    if (pos >= 0 && pos < capacity) {
                        ray_indices[pos] = static_cast<int32_t>(r);
                        t_starts[pos] = t0[u];
                        t_ends[pos] = t1[u];
                    } else {
                        overflow = true;
                    }
                }
            }
            count += __popcll(m);
            if (p.max_per_ray > 0 && count >= p.max_per_ray) {
                count = p.max_per_ray;
                done = true;
                break;
            }
            if (FILL && count >= limit) {
                done = true;
                break;
            }
        }
    }
    if (!FILL && lane < n_masks) masks[lane] = my_masks.mine();
    return count;
}

// One ray, uniform steps, whole wave.  Returns the ray's sample count (the
// same value in every lane).  FILL writes samples [0, limit) at `start`.
// With SKIP, candidates inside a stretch the skip field clears are not
// looked up; a chunk of 64 candidates that lies wholly inside one is passed
// over at the cost of its lattice arithmetic.
template <int LOOKUP, bool FILL, bool SKIP>
__device__ __forceinline__ int march_ray_uniform(
    int64_t r, const RaySpan& span, const uint32_t* __restrict__ bits, const uint8_t* __restrict__ skip,
    const GridK& g, const StepK& p, int64_t start, int limit, int64_t capacity, int32_t* __restrict__ ray_indices,
    float* __restrict__ t_starts, float* __restrict__ t_ends, bool& overflow, uint64_t* __restrict__ masks = nullptr, int n_masks = 0, int first_chunk = 0,
    int count0 = 0) {
    if constexpr (!SKIP) {
        return march_ray_uniform_x2<LOOKUP, FILL>(r, span, bits, g, p, start, limit, capacity, ray_indices, t_starts,
                                                  t_ends, overflow, masks, n_masks, first_chunk, count0);
    }
    if (!span.valid) return 0;
    const int lane = lane_id();
    const float* o = span.o;
    const float* d = span.d;
    const uint32_t word0 = span.word0;
    const float t_near = span.t_near, t_far = span.t_far;
    SkipRay sk{};
    if (SKIP) sk = skip_ray(g, o, d, t_far);
    float skip_end = -INFINITY;  // candidates with midpoint below it are empty
    ChunkMasks my_masks;         // count pass
    int count = count0;
    for (int k0 = first_chunk * kWave; k0 < kMaxCandidates; k0 += kWave) {
        const int chunk = k0 / kWave;
        const int k = k0 + lane;
        const float t0 = t_near + static_cast<float>(k) * p.dt;
        const bool live = t0 < t_far;
        if (ballot(live) == 0) break;  // t_k is non-decreasing in k
        const float t1 = t_near + static_cast<float>(k + 1) * p.dt;
        const float tm = (t0 + t1) * 0.5f;
        const bool todo = live && !(tm < skip_end);
        bool hit = false;
        if (ballot(todo) != 0ull) {
            // every lane probes its candidate (the index is in range whatever
            // the candidate), so the grid word and the skip byte are loaded
            // together; lanes inside a cleared stretch ignore the word
            const Probe q = probe<LOOKUP>(g, word0, o[0] + d[0] * tm, o[1] + d[1] * tm, o[2] + d[2] * tm);
            const uint32_t w = grid_word(grid_rsrc(bits, g), q.word);
            if (SKIP) {
                const int dist = skip[q.coarse];
                const float e = live ? skip_end_at<LOOKUP>(g, sk, q, dist, tm) : -INFINITY;
                // the stretches start at this chunk's candidates, so any of
                // them that reaches past the chunk covers the next candidates
                skip_end = fmaxf(skip_end, wave_max(e));
            }
            hit = todo && ((w >> q.bit) & 1u) != 0u;
        }
        const uint64_t m = ballot(hit);
        if (!FILL) my_masks.keep(chunk, m);
        if (FILL && hit) {
            const int idx = count + bits_below(m);
            if (idx < limit) {
                const int64_t pos = start + idx;
                if (pos >= 0 && pos < capacity) {
                    ray_indices[pos] = static_cast<int32_t>(r);
                    t_starts[pos] = t0;
                    t_ends[pos] = t1;
                } else {
                    overflow = true;
                }
            }
        }
        count += __popcll(m);
        if (p.max_per_ray > 0 && count >= p.max_per_ray) {
            count = p.max_per_ray;
            break;
        }
        if (FILL && count >= limit) break;
    }
    if (!FILL && lane < n_masks) masks[lane] = my_masks.mine();
    return count;
}

template <int LOOKUP, bool SKIP, int WAVES>
__global__ __launch_bounds__(WAVES * kWave) void count_uniform_kernel(
    const float* __restrict__ rays_o, const float* __restrict__ rays_d,
    const int32_t* __restrict__ grid_id, int64_t n_rays, const uint32_t* __restrict__ bits,
    const uint8_t* __restrict__ skip, GridK g, ClipK c, StepK p, int32_t* __restrict__ packed_info,
    int64_t* __restrict__ block_sums, uint64_t* __restrict__ masks, int n_masks, int split) {
    __shared__ int64_t wave_total[WAVES];
    const int wave = uniform<int>(static_cast<int>(threadIdx.x) / kWave);
    // workgroup b takes part b % split of the group of kRaysPerBlock rays
    // b / split: per = kRaysPerBlock / split rays from `first`; its samples
    // are part b of the scan
    const int per = kRaysPerBlock / split;
    const int64_t group = static_cast<int64_t>(blockIdx.x) / split;
    const int64_t first = group * kRaysPerBlock + static_cast<int64_t>(blockIdx.x % split) * per;
    // this wave's rays are first + wave + j WAVES; lane j clips ray j
    const int64_t mine = first + wave + static_cast<int64_t>(lane_id()) * WAVES;
    RaySpan spans{};
    if (wave + lane_id() * WAVES < per && mine < n_rays) {
        spans = ray_span<LOOKUP>(mine, rays_o, rays_d, grid_id, g, c, p);
    }
    int64_t total = 0;
    bool unused = false;
    for (int i = wave; i < per; i += WAVES) {
        const int64_t r = first + i;
        if (r >= n_rays) break;
        const RaySpan span = read_span(spans, i / WAVES);
        uint64_t* ray_masks = masks != nullptr ? masks + r * n_masks : nullptr;
        const int ray_n_masks = masks != nullptr ? n_masks : 0;
        const int n = march_ray_uniform<LOOKUP, false, SKIP>(r, span, bits, skip, g, p, 0, 0, 0, nullptr, nullptr,
                                                             nullptr, unused, ray_masks, ray_n_masks);
        if (lane_id() == 0) packed_info[2 * r + 1] = n;
        total += n;
    }
    if (lane_id() == 0) wave_total[wave] = total;
    __syncthreads();
    if (threadIdx.x == 0) {
        int64_t s = 0;
        for (int w = 0; w < WAVES; ++w) s += wave_total[w];
        block_sums[blockIdx.x] = s;
    }
}

// 32-bit value of lane `src` (per lane) through the LDS crossbar; every lane
// must be active.
__device__ __forceinline__ float lane_value(float v, int src) {
    return __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(src << 2, __builtin_bit_cast(int, v)));
}
__device__ __forceinline__ int lane_value(int v, int src) { return __builtin_amdgcn_ds_bpermute(src << 2, v); }

// Position of the k-th set bit of v (k < popcount(v)).
__device__ __forceinline__ int nth_set_bit(uint64_t v, int k) {
    int pos = 0;
#pragma unroll
    for (int w = 32; w >= 1; w >>= 1) {
        const int c = static_cast<int>(__popcll(v & ((1ull << w) - 1ull)));
        if (k >= c) {
            k -= c;
            v >>= w;
            pos += w;
        }
    }
    return pos;
}

// The fill pass writes the samples of a ray from the per-chunk occupancy
// masks stored by the count pass (the first n_masks chunks), so the grid is
// not traversed a second time; a ray whose samples continue past those
// chunks is traversed from there on.
//
// A wave takes up to kFillRaysMax consecutive rays, whose samples are
// consecutive in the output.  Their masks are one run of the mask array,
// read as such.  The nonzero halves of the masks (32 candidates each) are
// queued in LDS, 64 at a time are expanded, one lane per half, into a list
// of (ray, candidate) codes in output order, and the list is stored in
// blocks of 64 positions, lane i position 64 q + i, as whole aligned runs of
// 256 bytes with the lattice arithmetic in every lane.  The ends of a wave's
// samples, which share their blocks with the neighbouring waves' samples,
// are stored last, after a barrier of the workgroup: the pieces of such a
// block then reach the L2 together and leave it as one write.
// Bound by the write path.  Three dword streams reach 5.7 TB/s in whole
// blocks, 4.0-4.5 TB/s in stores that start anywhere, and 4.4 TB/s in whole
// blocks whose shared ends are written a wave's lifetime apart.  61.6 M
// samples of 262,144 rays: 243 us with a store per chunk and array, 187 us
// in whole blocks, 162 us (4.6 TB/s) with the shared ends last; 9.8 M
// samples of 65,536 rays 36 -> 30 us.
constexpr int kFillThreads = 256;
constexpr int kFillWaves = kFillThreads / kWave;
constexpr int kFillRaysMax = 8;
constexpr int kFillGroups = 4;               // rays of a wave x chunks <= 4 x 64
constexpr int kFillQueue = 3 * kWave;        // halves left over (< 64) and those of 64 chunks
constexpr int kFillCodes = kWave * 32 + kWave;  // samples of 64 halves, from any place in a block
constexpr int kCodeRayShift = 12;            // code: ray of the wave << 12 | candidate (< 64 chunks x 64)

static_assert(kListBlock == kWave, "a position of a block per lane");

struct FillOut {
    int32_t* ray_indices;
    float* t_starts;
    float* t_ends;
};

struct FillLds {
    uint32_t queue_mask[kFillQueue];
    uint16_t queue_code[kFillQueue];
    uint16_t codes[kFillCodes];  // the list: codes[i] is the sample at position block + i
    uint16_t head[kWave];        // the first block's part of the list, stored last
    float t_near[kFillRaysMax];
    int32_t taken[kFillRaysMax];
};

// Times of the sample `code`: uniform steps from the ray's t_near, or (cone
// steps) entries of the near-plane lattice, in LDS.
struct UniformTimes {
    const float* t_near;
    float dt;
    __device__ __forceinline__ float start(uint32_t code) const {
        return t_near[code >> kCodeRayShift] + static_cast<float>(code & ((1u << kCodeRayShift) - 1u)) * dt;
    }
    __device__ __forceinline__ float end(uint32_t code) const {
        const float k = static_cast<float>(code & ((1u << kCodeRayShift) - 1u));
        return t_near[code >> kCodeRayShift] + (k + 1.0f) * dt;  // k + 1 is exact
    }
};

struct TableTimes {
    const float* t;
    __device__ __forceinline__ float start(uint32_t code) const { return t[code & ((1u << kCodeRayShift) - 1u)]; }
    __device__ __forceinline__ float end(uint32_t code) const { return t[(code & ((1u << kCodeRayShift) - 1u)) + 1u]; }
};

// Stores the sample of `code` at position p = b + lane.
template <typename Times>
__device__ __forceinline__ void store_sample(const FillOut& out, const Times& times, int64_t first_ray, int b,
                                             uint32_t code) {
    const uint32_t off = static_cast<uint32_t>(lane_id());
    (out.ray_indices + b)[off] = static_cast<int32_t>(first_ray + (code >> kCodeRayShift));
    (out.t_starts + b)[off] = times.start(code);
    (out.t_ends + b)[off] = times.end(code);
}

// Expands the first n <= 64 queued halves into the list from position `pos`
// on and stores the blocks that are complete, except for the part of one
// from `head_end` - 64 on that other waves' samples precede (head_end: the
// end of the wave's first block, if it does not begin it).  The incomplete
// last block moves to the list's front.  Returns the position after the
// last sample.
template <typename Times>
__device__ __forceinline__ int store_halves(const FillOut& out, FillLds& q, int n, const Times& times,
                                            int64_t first_ray, int head_end, int pos, int& block) {
    const int lane = lane_id();
    uint32_t m = lane < n ? q.queue_mask[lane] : 0u;
    const uint32_t code = lane < n ? q.queue_code[lane] : 0u;
    const int count = __popc(m);
    const int incl = wave_inclusive_sum(count);
    const int end = pos + read_lane(incl, kWave - 1);
    int slot = pos - block + incl - count;
    while (ballot(m != 0u) != 0ull) {
        if (m != 0u) {
            q.codes[slot++] = static_cast<uint16_t>(code + static_cast<uint32_t>(__builtin_ctz(m)));
            m &= m - 1u;
        }
    }
    wave_lds_sync();
    const int b = walk_blocks(
        block, head_end, end, [&]() { q.head[lane] = q.codes[lane]; },
        [&](int p) { store_sample(out, times, first_ray, p, q.codes[p - block + lane]); });
    if (b > block) {
        const uint16_t c = q.codes[b - block + lane];
        wave_lds_sync();
        q.codes[lane] = c;
        block = b;
    }
    wave_lds_sync();
    return end;
}

// Queues the samples of 64 chunks, a lane's mask and the code of its first
// candidate, in lane order, and lists and stores what fills the wave (`last`:
// everything).
template <typename Times>
__device__ __forceinline__ void queue_chunks(const FillOut& out, FillLds& q, const Times& times, uint64_t m,
                                             uint32_t code, bool last, int64_t first_ray, FillList& list) {
    const int lane = lane_id();
    const uint32_t lo = static_cast<uint32_t>(m), hi = static_cast<uint32_t>(m >> 32);
    const uint64_t has_lo = ballot(lo != 0u), has_hi = ballot(hi != 0u);
    int at = list.queued + bits_below(has_lo) + bits_below(has_hi);
    if (lo != 0u) {
        q.queue_mask[at] = lo;
        q.queue_code[at++] = static_cast<uint16_t>(code);
    }
    if (hi != 0u) {
        q.queue_mask[at] = hi;
        q.queue_code[at] = static_cast<uint16_t>(code + 32u);
    }
    list.queued += static_cast<int>(__popcll(has_lo)) + static_cast<int>(__popcll(has_hi));
    wave_lds_sync();
    while (list.queued >= kWave || (last && list.queued > 0)) {
        const int n = min(list.queued, kWave);
        list.pos = store_halves(out, q, n, times, first_ray, list.head_end, list.pos, list.block);
        list.queued -= n;
        if (list.queued > 0) {  // at most 127 halves move up
            const uint32_t m0 = q.queue_mask[kWave + lane], m1 = q.queue_mask[2 * kWave + lane];
            const uint16_t c0 = q.queue_code[kWave + lane], c1 = q.queue_code[2 * kWave + lane];
            wave_lds_sync();
            q.queue_mask[lane] = m0;
            q.queue_mask[kWave + lane] = m1;
            q.queue_code[lane] = c0;
            q.queue_code[kWave + lane] = c1;
            wave_lds_sync();
        }
    }
}

// The ends of a wave's samples, after the workgroup's barrier.
template <typename Times>
__device__ __forceinline__ void end_list(const FillOut& out, const FillLds& q, const Times& times, int64_t first_ray,
                                         int pos0, const FillList& list) {
    const int lane = lane_id();
    if (list.head_end >= 0 && list.head_end <= list.pos && lane >= (pos0 & (kWave - 1))) {
        store_sample(out, times, first_ray, list.head_end - kWave, q.head[lane]);
    }
    if (list.block + lane < list.pos && list.block + lane >= pos0) {
        store_sample(out, times, first_ray, list.block, q.codes[lane]);
    }
}

// The part of a chunk's mask that its ray's limit leaves it; in_ray: the
// ray's samples before the chunk.
__device__ __forceinline__ uint64_t capped_mask(uint64_t m, int in_ray, int limit) {
    const int take = limit - in_ray;
    if (take <= 0) return 0ull;
    if (take < static_cast<int>(__popcll(m))) m &= (1ull << nth_set_bit(m, take)) - 1ull;
    return m;
}

// The samples of the stored chunks of one ray (lane j of `mine` holds chunk
// j's mask), each one checked: those at or past `capacity` are left out.
__device__ __forceinline__ int fill_chunks_checked(int64_t r, float t_near, float dt, int64_t start, int limit,
                                                   int64_t capacity, const FillOut& out, bool& overflow,
                                                   uint64_t mine) {
    const int lane = lane_id();
    int written = 0;
    for (uint64_t todo = ballot(mine != 0ull); todo != 0ull && written < limit; todo &= todo - 1ull) {
        const int j = static_cast<int>(__builtin_ctzll(todo));
        const uint64_t m = (static_cast<uint64_t>(static_cast<uint32_t>(
                                __builtin_amdgcn_readlane(static_cast<int>(mine >> 32), j)))
                            << 32) |
                           static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(mine), j));
        const int pc = static_cast<int>(__popcll(m));
        const int n_take = pc < limit - written ? pc : limit - written;
        const int rank = bits_below(m);
        if (((m >> lane) & 1ull) != 0ull && rank < n_take) {
            const int64_t pos = start + written + rank;
            if (pos >= 0 && pos < capacity) {
                const int k = j * kWave + lane;
                out.ray_indices[pos] = static_cast<int32_t>(r);
                out.t_starts[pos] = t_near + static_cast<float>(k) * dt;
                out.t_ends[pos] = t_near + static_cast<float>(k + 1) * dt;
            } else {
                overflow = true;
            }
        }
        written += n_take;
    }
    return written;
}

// per: rays per wave, at most kFillRaysMax and kFillGroups 64 / n_masks.
template <int LOOKUP, bool SKIP>
__global__ __launch_bounds__(kFillThreads) void fill_uniform_kernel(
    const float* __restrict__ rays_o, const float* __restrict__ rays_d,
    const int32_t* __restrict__ grid_id, int64_t n_rays, const uint32_t* __restrict__ bits,
    const uint8_t* __restrict__ skip, GridK g, ClipK c, StepK p, const int32_t* __restrict__ packed_info,
    int64_t capacity, int32_t* __restrict__ ray_indices, float* __restrict__ t_starts, float* __restrict__ t_ends,
    int32_t* __restrict__ status, const uint64_t* __restrict__ masks, int n_masks, int per) {
    __shared__ FillLds lds[kFillWaves];
    const int lane = lane_id();
    const int wave = uniform<int>(static_cast<int>(threadIdx.x) / kWave);
    const int64_t first = (xcd_grouped<16>(row_block(), row_blocks()) * kFillWaves + wave) * per;
    const int n_mine = static_cast<int>(max(min(static_cast<int64_t>(per), n_rays - first), int64_t{0}));
    FillLds& q = lds[wave];
    const FillOut out{ray_indices, t_starts, t_ends};
    // lane i: ray first + i
    int start = 0, limit = 0;
    if (lane < n_mine) {
        start = packed_info[2 * (first + lane)];
        limit = packed_info[2 * (first + lane) + 1];
    }
    // the wave's masks, chunk after chunk, ray after ray; all loaded before
    // anything is stored (one counter tracks a wave's loads and stores)
    const int n_flat = masks != nullptr ? n_mine * n_masks : 0;
    uint64_t mk[kFillGroups];
#pragma unroll
    for (int i = 0; i < kFillGroups; ++i) {
        const int f = i * kWave + lane;
        mk[i] = f < n_flat ? masks[first * n_masks + f] : 0ull;
    }
    RaySpan spans{};
    if (limit > 0) spans = ray_span<LOOKUP>(first + lane, rays_o, rays_d, grid_id, g, c, p);
    if (lane < kFillRaysMax) {
        q.t_near[lane] = spans.t_near;
        q.taken[lane] = 0;
    }
    wave_lds_sync();
    // the ray of entry f < 256 is f / n_masks: exact by this reciprocal
    const uint32_t inv = 65536u / static_cast<uint32_t>(max(n_masks, 1)) + 1u;
#pragma unroll
    for (int i = 0; i < kFillGroups; ++i) {
        const uint32_t f = static_cast<uint32_t>(i * kWave + lane);
        const int count = static_cast<int>(__popcll(mk[i]));
        if (count > 0) {
            __hip_atomic_fetch_add(&q.taken[(f * inv) >> 16], count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
        }
    }
    wave_lds_sync();
    const int stored = lane < n_mine ? q.taken[lane] : 0;
    const int before = wave_inclusive_sum(limit) - limit;
    const int pos0 = read_lane(start, 0), n_out = read_lane(before + limit, kWave - 1);
    // every ray's samples are those of its stored chunks (the first `limit`
    // of them), and they lie side by side inside the output
    const bool simple = ballot(lane < n_mine && (limit > stored || (limit > 0 && start != pos0 + before))) == 0ull &&
                        list_fits(pos0, n_out, capacity);
    const bool capped = ballot(limit < stored) != 0ull;
    FillList list = begin_list(pos0);
    const UniformTimes times{q.t_near, p.dt};
    bool overflow = false;
    if (simple) {
        int carried = 0;  // samples in earlier groups of the ray that group i begins with
        const int groups = (n_flat + kWave - 1) / kWave;
        for (int i = 0; i < groups; ++i) {
            uint64_t m = mk[0];
#pragma unroll
            for (int k = 0; k + 1 < kFillGroups; ++k) mk[k] = mk[k + 1];
            const uint32_t f = static_cast<uint32_t>(i * kWave + lane);
            const uint32_t ray = (f * inv) >> 16;
            const uint32_t code = (ray << kCodeRayShift) | ((f - ray * static_cast<uint32_t>(n_masks)) << kWaveLog2);
            if (capped) {  // keep of each chunk what its ray's limit leaves it
                const int count = static_cast<int>(__popcll(m));
                const int excl = wave_inclusive_sum(count) - count;
                const int ray_lane = static_cast<int>(ray) * n_masks - i * kWave;  // of the ray's first chunk
                const int base = lane_value(excl, max(ray_lane, 0));
                const int in_ray = ray_lane >= 0 ? excl - base : excl + carried;
                carried = read_lane(in_ray + count, kWave - 1);
                m = capped_mask(m, in_ray, lane_value(limit, static_cast<int>(min(ray, 63u))));
            }
            queue_chunks(out, q, times, m, code, i + 1 == groups, first, list);
        }
    }
    // rays going on past the stored chunks or not fitting the output, ray by
    // ray
    for (int i = 0; i < n_mine && !simple; ++i) {
        const int ray_limit = read_lane(limit, i);
        if (ray_limit == 0) continue;
        const int64_t r = first + i;
        const int64_t ray_start = read_lane(start, i);
        const RaySpan span = read_span(spans, i);
        const uint64_t mine = masks != nullptr && lane < n_masks ? masks[r * n_masks + lane] : 0ull;
        const int written = fill_chunks_checked(r, span.t_near, p.dt, ray_start, ray_limit, capacity, out, overflow,
                                                mine);
        if (written < ray_limit) {  // samples past the stored chunks: traverse from there
            march_ray_uniform<LOOKUP, true, SKIP>(r, span, bits, skip, g, p, ray_start, ray_limit, capacity,
                                                  ray_indices, t_starts, t_ends, overflow, nullptr, 0,
                                                  masks != nullptr ? n_masks : 0, written);
        }
    }
    if (overflow && status != nullptr) *status = NACC_ECAPACITY;
    __syncthreads();
    if (simple) end_list(out, q, times, first, pos0, list);
}

// Cone steps: the lattice is a recurrence in t, t_{k+1} = t_k +
// min(max(t_k c, dt), dt_max), so a lane walks a stretch of one ray.
// Candidates are taken kConeBatch at a time: the recurrence first (a few
// dependent FP32 operations per candidate), then the batch's grid words are
// all loaded before any is tested, so each lane keeps several loads in
// flight.  The count pass stores the occupancy bits of each chunk of 64
// candidates chunk-major (masks[chunk * n_rays + r]), and the fill pass
// replays them, running only the recurrence.
constexpr int kConeBatch = 8;
static_assert(kWave % kConeBatch == 0, "a batch must not straddle two chunks");

// The next kConeBatch cone steps from t: interval ends tb[0..kConeBatch] and
// how many of the batch's candidates lie inside the ray (a candidate is in
// while t_k < t_far and the step still advances t).
__device__ __forceinline__ int cone_steps(float t, float t_far, const StepK& p, float tb[kConeBatch + 1]) {
    tb[0] = t;
    int n_valid = kConeBatch;
#pragma unroll
    for (int u = 0; u < kConeBatch; ++u) {
        // min(max(t c, dt), dt_max) as one median (dt <= dt_max)
        const float step = __builtin_amdgcn_fmed3f(tb[u] * p.cone, p.dt, p.dt_max);
        tb[u + 1] = tb[u] + step;
        if (n_valid == kConeBatch && !(tb[u] < t_far && tb[u + 1] > tb[u])) n_valid = u;
    }
    return n_valid;
}

// Occupancy bits of a batch's candidates (bit u for candidate u < n_valid).
// All the batch's words (and one skip byte) are loaded before any is
// tested; every index is in range whatever the candidate.  Candidates
// inside a stretch cleared by the skip field are not looked up, and the
// batch's last candidate extends that stretch for the next batches.
template <int LOOKUP, bool SKIP>
__device__ __forceinline__ uint32_t cone_hits(const uint32_t* __restrict__ bits, const uint8_t* __restrict__ skip,
                                              const GridK& g, const SkipRay& sk, float& skip_end, uint32_t word0,
                                              const float o[3], const float d[3], const float tb[kConeBatch + 1],
                                              int n_valid) {
    float tm[kConeBatch];
    uint32_t todo = (1u << n_valid) - 1u;
#pragma unroll
    for (int u = 0; u < kConeBatch; ++u) {
        tm[u] = (tb[u] + tb[u + 1]) * 0.5f;
        if (SKIP && tm[u] < skip_end) todo &= ~(1u << u);
    }
    uint32_t hits = 0u;
    if (todo != 0u) {
        Probe q[kConeBatch];
        uint32_t w[kConeBatch];
#pragma unroll
        for (int u = 0; u < kConeBatch; ++u) {
            q[u] = probe<LOOKUP>(g, word0, o[0] + d[0] * tm[u], o[1] + d[1] * tm[u], o[2] + d[2] * tm[u]);
        }
#pragma unroll
        for (int u = 0; u < kConeBatch; ++u) w[u] = grid_word(grid_rsrc(bits, g), q[u].word);
        const int dist = SKIP ? static_cast<int>(skip[q[kConeBatch - 1].coarse]) : 0;
#pragma unroll
        for (int u = 0; u < kConeBatch; ++u) {
            if (((todo >> u) & 1u) != 0u && ((w[u] >> q[u].bit) & 1u) != 0u) hits |= 1u << u;
        }
        if (SKIP && n_valid == kConeBatch) {
            skip_end = fmaxf(skip_end, skip_end_at<LOOKUP>(g, sk, q[kConeBatch - 1], dist, tm[kConeBatch - 1]));
        }
    }
    return hits;
}

// Levels of a cascade segment's midpoints, bounded by cone_segment_live:
// every midpoint lies on `hi` or the level below it (`hi` alone where
// `one`); `wide`: on more levels, or not established.
struct SegLevels {
    int hi;
    bool one, wide;
};

__device__ __forceinline__ uint32_t cell_index(const GridK& g, float u0, float u1, float u2) {
    const uint32_t j0 = static_cast<uint32_t>(static_cast<int>(clamp_cell(u0, g.top)));
    const uint32_t j1 = static_cast<uint32_t>(static_cast<int>(clamp_cell(u1, g.top)));
    const uint32_t j2 = static_cast<uint32_t>(static_cast<int>(clamp_cell(u2, g.top)));
    return __umul24(j0, g.res2) + (__umul24(j1, static_cast<uint32_t>(g.res)) + j2);
}

// Occupancy bits of a segment's candidates (bit u for candidate u) from its
// first t, those from t_far on and past a stalled step cleared; cascades: a
// segment that is not `wide`.  The same cells as probe()'s with fewer
// operations: a cascade level scales by a power of two, which commutes with
// every rounding of ((x 2^-l) - lo) s, so one level costs the operations of a
// plain box with lo 2^l and s 2^-l, and two cost a comparison and three
// selections (wide_levels keeps the scales far from the ends of the exponent
// range).  Contraction: the fast cells first, then the exact ones where any
// lane needs them, four candidates at a time: all eight together hold 110
// registers, and half the waves fit (131,071 rays of 39 chunks: count 210 us;
// 137 us four at a time and with cells_within before them).  The other
// lookups hold eight in 62 registers (262,144 rays of a cascade: 129 us
// against 135 four at a time).
template <int LOOKUP>
__device__ __forceinline__ uint32_t segment_hits(__amdgpu_buffer_rsrc_t grs, const GridK& g, const StepK& p,
                                                 uint32_t word0, const SegLevels& lv, const float o[3],
                                                 const float d[3], float t, float t_far) {
    float lo_a = 0.0f, lo_b = 0.0f, s_a = 0.0f, s_b = 0.0f, thr = 0.0f;
    uint32_t w_a = word0, w_b = word0;
    if (LOOKUP == NACC_LOOKUP_CASCADE) {
        const int la = lv.one ? lv.hi : max(lv.hi - 1, 0);
        lo_a = ldexpf(g.lo[0], la);
        lo_b = ldexpf(g.lo[0], lv.hi);
        s_a = ldexpf(g.s[0], -la);
        s_b = ldexpf(g.s[0], -lv.hi);
        thr = ldexpf(g.base, la);
        w_a = static_cast<uint32_t>(la) * g.words;
        w_b = static_cast<uint32_t>(lv.hi) * g.words;
    }
    constexpr int kHitBatch = LOOKUP == NACC_LOOKUP_CONTRACT ? 4 : kConeBatch;
    uint32_t hits = 0u;
#pragma unroll 1
    for (int u0 = 0; u0 < kConeBatch; u0 += kHitBatch) {
        float tb[kHitBatch + 1];
        tb[0] = t;
#pragma unroll
        for (int u = 0; u < kHitBatch; ++u) {
            tb[u + 1] = tb[u] + __builtin_amdgcn_fmed3f(tb[u] * p.cone, p.dt, p.dt_max);
        }
        t = tb[kHitBatch];
        uint32_t cell[kHitBatch], w[kHitBatch];
        bool need[kHitBatch], any_need = false;
#pragma unroll
        for (int u = 0; u < kHitBatch; ++u) {
            const float tm = (tb[u] + tb[u + 1]) * 0.5f;
            const float x0 = o[0] + d[0] * tm, x1 = o[1] + d[1] * tm, x2 = o[2] + d[2] * tm;
            if (LOOKUP == NACC_LOOKUP_CASCADE) {
                const bool up = fmaxf(fmaxf(fabsf(x0), fabsf(x1)), fabsf(x2)) > thr;
                const float lo = up ? lo_b : lo_a, sc = up ? s_b : s_a;
                cell[u] = cell_index(g, (x0 - lo) * sc, (x1 - lo) * sc, (x2 - lo) * sc);
                w[u] = grid_word(grs, (up ? w_b : w_a) + (cell[u] >> 5));
            } else if (LOOKUP == NACC_LOOKUP_CONTRACT) {
                // see probe(); times 1 is exact where |x| is not contracted
                const float na = __builtin_amdgcn_sqrtf((x0 * x0 + x1 * x1) + x2 * x2);
                const float ia = __builtin_amdgcn_rcpf(na);
                const bool far = na > 1.0f;
                const float fa = far ? (2.0f - ia) * ia : 1.0f;
                const float v0 = (x0 * fa - g.lo[0]) * g.s[0];
                const float v1 = (x1 * fa - g.lo[1]) * g.s[1];
                const float v2 = (x2 * fa - g.lo[2]) * g.s[2];
                const float near =
                    fminf(fminf(fabsf(v0 - rintf(v0)), fabsf(v1 - rintf(v1))), fabsf(v2 - rintf(v2)));
                need[u] = (far && near <= g.contract_delta) || fabsf(na - 1.0f) <= 0x1p-20f;
                any_need = any_need || need[u];
                cell[u] = cell_index(g, v0, v1, v2);
            } else {
                cell[u] = cell_index(g, (x0 - g.lo[0]) * g.s[0], (x1 - g.lo[1]) * g.s[1], (x2 - g.lo[2]) * g.s[2]);
                w[u] = grid_word(grs, word0 + (cell[u] >> 5));
            }
        }
        if (LOOKUP == NACC_LOOKUP_CONTRACT) {
            if (ballot(any_need) != 0ull) {
#pragma unroll
                for (int u = 0; u < kHitBatch; ++u) {
                    if (need[u]) {
                        const float tm = (tb[u] + tb[u + 1]) * 0.5f;
                        float x0 = o[0] + d[0] * tm, x1 = o[1] + d[1] * tm, x2 = o[2] + d[2] * tm;
                        const float n = sqrtf((x0 * x0 + x1 * x1) + x2 * x2);
                        if (n > 1.0f) {
                            const float f = (2.0f - 1.0f / n) / n;
                            x0 = x0 * f;
                            x1 = x1 * f;
                            x2 = x2 * f;
                        }
                        cell[u] =
                            cell_index(g, (x0 - g.lo[0]) * g.s[0], (x1 - g.lo[1]) * g.s[1], (x2 - g.lo[2]) * g.s[2]);
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < kHitBatch; ++u) w[u] = grid_word(grs, word0 + (cell[u] >> 5));
        }
        // a stalled step repeats its t, which is then the last
        const float t_stop = fminf(t_far, t);
#pragma unroll
        for (int u = 0; u < kHitBatch; ++u) {
            const uint32_t bit = __builtin_amdgcn_ubfe(w[u], cell[u] & 31u, 1u);
            hits |= (tb[u] < t_stop ? bit : 0u) << (u0 + u);
        }
    }
    return hits;
}

// One ray, cone steps, one lane, traversing the grid: the fill pass when no
// count-pass workspace is given (the same samples as the chunk-parallel
// passes, for checking them and for callers that keep no workspace).
template <int LOOKUP, bool SKIP>
__device__ __forceinline__ void fill_ray_cone(
    int64_t r, const float* __restrict__ rays_o, const float* __restrict__ rays_d,
    const int32_t* __restrict__ grid_id, const uint32_t* __restrict__ bits,
    const uint8_t* __restrict__ skip, const GridK& g,
    const ClipK& c, const StepK& p, int64_t start, int limit, int64_t capacity,
    float* __restrict__ t_starts, float* __restrict__ t_ends, bool& overflow) {
    float o[3], d[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        o[i] = rays_o[3 * r + i];
        d[i] = rays_d[3 * r + i];
    }
    uint32_t word0;
    if (!grid_of_ray<LOOKUP>(grid_id, r, g, word0)) return;
    float t_near, t_far;
    if (!clip_ray(o, d, c, p.near_plane, p.far_plane, t_near, t_far)) return;
    SkipRay sk{};
    if (SKIP) sk = skip_ray(g, o, d, t_far);
    float skip_end = -INFINITY;  // candidates with midpoint below it are empty
    int count = 0;
    float t = t_near;
    for (int k0 = 0; k0 < kMaxCandidates && count < limit; k0 += kConeBatch) {
        float tb[kConeBatch + 1];
        const int n_valid = cone_steps(t, t_far, p, tb);
        const uint32_t hits =
            cone_hits<LOOKUP, SKIP>(bits, skip, g, sk, skip_end, word0, o, d, tb, n_valid) & ((1u << n_valid) - 1u);
#pragma unroll
        for (int u = 0; u < kConeBatch; ++u) {
            if (((hits >> u) & 1u) == 0u || count >= limit) continue;
            const int64_t pos = start + count;
            if (pos >= 0 && pos < capacity) {
                t_starts[pos] = tb[u];
                t_ends[pos] = tb[u + 1];
            } else {
                overflow = true;
            }
            ++count;
        }
        if (n_valid < kConeBatch) break;
        t = tb[kConeBatch];
    }
}

struct ConeHalo {
    float v;     // max_i s_i |d_i|: level-0 cells per unit t on the fastest axis
    float smax;  // max_i s_i
    float omax, dmax, dnorm;
    float onorm;  // |o|, rounded up
};

__device__ __forceinline__ ConeHalo cone_halo_ray(const GridK& g, const float o[3], const float d[3]) {
    ConeHalo k;
    k.v = fmaxf(fmaxf(g.s[0] * fabsf(d[0]), g.s[1] * fabsf(d[1])), g.s[2] * fabsf(d[2]));
    k.smax = fmaxf(fmaxf(g.s[0], g.s[1]), g.s[2]);
    k.omax = fmaxf(fmaxf(fabsf(o[0]), fabsf(o[1])), fabsf(o[2]));
    k.dmax = fmaxf(fmaxf(fabsf(d[0]), fabsf(d[1])), fabsf(d[2]));
    k.dnorm = sqrtf((d[0] * d[0] + d[1] * d[1]) + d[2] * d[2]) * (1.0f + 0x1p-18f);
    k.onorm = sqrtf((o[0] * o[0] + o[1] * o[1]) + o[2] * o[2]) * (1.0f + 0x1p-18f);
    return k;
}

// Where a segment of candidates whose midpoints lie in [ta, tb] is looked
// up: its centre (on its level, contracted) and `dev`, the bound of the cell
// coordinates' distance from the centre's on every axis.  False: no bound.
template <int LOOKUP>
__device__ __forceinline__ bool cone_segment_cells(const GridK& g, const float o[3], const float d[3],
                                                   const ConeHalo& k, float ta, float tb, SegLevels& lv, float x[3],
                                                   float& dev) {
    const float tc = (ta + tb) * 0.5f;
    const float h = (tb - ta) * 0.5f + fabsf(tb) * 0x1p-20f;  // half-extent, with the rounding of the t values
    float &x0 = x[0], &x1 = x[1], &x2 = x[2];
    x0 = o[0] + d[0] * tc;
    x1 = o[1] + d[1] * tc;
    x2 = o[2] + d[2] * tc;
    // the rounding of positions (a few ulps of the largest coordinate
    // reached, for both points) and of cell coordinates, generously
    const float slack_x = (k.omax + k.dmax * fabsf(tb) + 1.0f) * 0x1p-19f;
    const float cell_slack = static_cast<float>(g.res) * 0x1p-17f;
    bool open = false;  // the bound cannot be established
    if (LOOKUP == NACC_LOOKUP_CASCADE) {
        const float m = fmaxf(fmaxf(fabsf(x0), fabsf(x1)), fabsf(x2));
        const float dm = k.dmax * h + slack_x;
        const float m_lo = m - dm;
        const int l_hi = cascade_level(m + dm, g);
        const float below = ldexpf(g.base, l_hi - 1);  // the largest |x_i| of the level below
        lv.hi = l_hi;
        lv.one = l_hi == 0 || m_lo > below;
        lv.wide = !(lv.one || l_hi == 1 || m_lo > below * 0.5f) || !(dm < INFINITY) || g.wide_levels != 0;
        open = !lv.one;  // a midpoint may lie on another level
        x0 = ldexpf(x0, -l_hi);
        x1 = ldexpf(x1, -l_hi);
        x2 = ldexpf(x2, -l_hi);
        dev = ldexpf(k.v * h + k.smax * slack_x, -l_hi) + cell_slack;
    } else if (LOOKUP == NACC_LOOKUP_CONTRACT) {
        // The hardware square root and reciprocal (within a few ulps) serve
        // here: every quantity below is a bound that carries a margin far
        // above their error (2^-18 relative on |x|, L and the motion factor;
        // 2^-16 contracted units on the centre's position).
        const float n = __builtin_amdgcn_sqrtf((x0 * x0 + x1 * x1) + x2 * x2);
        // r_min bounds |x| from below over the segment; beyond radius r > 1
        // the contraction shrinks distances by at most (2 - 1/r)/r, and a
        // motion along the ray by at most (1 + 2|o|)/r^2: its radial part
        // shrinks by 1/r^2, its tangential part, at most |o||d|/r long, by
        // (2 - 1/r)/r < 2/r
        const float r_min = n * (1.0f - 0x1p-18f) - k.dnorm * h - 2.0f * slack_x;
        float lip = 1.0f, along = 1.0f;
        if (r_min > 1.0f) {
            const float ir = __builtin_amdgcn_rcpf(r_min);
            lip = ((2.0f - ir) * ir) * (1.0f + 0x1p-18f);
            along = fminf(lip, ((1.0f + 2.0f * k.onorm) * (ir * ir)) * (1.0f + 0x1p-18f));
        }
        if (n > 1.0f) {
            const float in = __builtin_amdgcn_rcpf(n);
            const float f = (2.0f - in) * in;
            x0 = x0 * f;
            x1 = x1 * f;
            x2 = x2 * f;
        }
        dev = k.smax * (along * k.dnorm * h + lip * 3.5f * slack_x + 3.5f * 0x1p-16f) + cell_slack;
    } else {
        dev = k.v * h + k.smax * slack_x + cell_slack;
    }
    return !open;
}

// Whether such a segment may hold samples (see above): false only when the
// centre's halo bit is clear and the bound holds.  Branch-free, so that the
// segments' halo words are all in flight together.
template <int LOOKUP>
__device__ __forceinline__ bool cone_segment_live(const GridK& g, __amdgpu_buffer_rsrc_t hrs, uint32_t grid,
                                                  const float o[3], const float d[3], const ConeHalo& k, float ta,
                                                  float tb, SegLevels& lv) {
    float x[3], dev;
    const bool bound = cone_segment_cells<LOOKUP>(g, o, d, k, ta, tb, lv, x, dev);
    const bool open = !bound || !(dev <= static_cast<float>(kHaloReach) * (1.0f - 0x1p-10f));
    const uint32_t hgrid = LOOKUP == NACC_LOOKUP_CASCADE ? static_cast<uint32_t>(lv.hi) : grid;
    const bool hb = halo_bit(hrs, g, hgrid * g.halo_words, x[0], x[1], x[2]);  // loaded in every case
    return open | hb;
}

// The cone-step lattice from the near plane, shared by every ray that
// starts there (rays from inside the clip box, or with no box at all, start
// at the near plane): t at every 8th candidate, computed once on the host
// in FP32 with the device's operations (each correctly rounded; the
// median of three is the clamp), and passed by value.  The recurrence only
// depends on t, so a chunk of any ray whose first t equals the table's
// entry continues along the table; the starts and count passes then read
// chunk and segment starts instead of walking them.  Left empty (n = 0) if
// the steps stall within the table (t + step == t), which the walks handle.
constexpr int kMaxMaskChunks = 64;  // one per lane of a wave
constexpr int kTableStride = kWave / kConeBatch;  // table entries per chunk
struct ConeTable {
    float t[kMaxMaskChunks * kTableStride + 1];
    int n;  // entries: n_masks 8 + 1, or 0
};

// Steps of the cone recurrence, t + clamp(t * cone, dt, dt_max) in FP32,
// from t while it is below `end`, at most `limit` of them: advances t and
// returns their number, or -1 if one stalls (t + step == t).  t only grows,
// so the three cases of the clamp follow each other; a loop each leaves only
// the operations of its own case in the serial chain (2,560 steps, mostly
// t + t * cone: 13 us with the clamp in every step, 6 us so).
// A NaN t * cone (0 times infinity) steps by dt, a NaN dt_max is no limit,
// as fmaxf and fminf have it.
int64_t cone_steps(float cone, float dt, float dt_max, double end, int64_t limit, float& t) {
    const float hi = std::isnan(dt_max) ? INFINITY : dt_max;
    const float lo = std::fmin(dt, hi);
    int64_t k = 0;
    float x = t;
    for (; k < limit && static_cast<double>(x) < end && !(x * cone > lo); ++k) {
        const float x1 = x + lo;
        if (!(x1 > x)) return -1;
        x = x1;
    }
    for (; k < limit && static_cast<double>(x) < end; ++k) {
        const float step = x * cone;
        if (!(step < hi)) break;
        const float x1 = x + step;
        if (!(x1 > x)) return -1;
        x = x1;
    }
    for (; k < limit && static_cast<double>(x) < end; ++k) {
        const float x1 = x + hi;
        if (!(x1 > x)) return -1;
        x = x1;
    }
    t = x;
    return k;
}

ConeTable cone_table(const StepK& p, int n_masks) {
    ConeTable tab;
    tab.n = 0;
    float t = p.near_plane;
    if (n_masks <= 0 || !std::isfinite(t)) return tab;
    const int n = n_masks * kTableStride + 1;
    for (int i = 0; i + 1 < n; ++i) {
        tab.t[i] = t;
        // stalls (or ends at infinity, as a stalled walk does): no table
        if (cone_steps(p.cone, p.dt, p.dt_max, INFINITY, kConeBatch, t) != kConeBatch) return tab;
    }
    tab.t[n - 1] = t;
    tab.n = n;
    return tab;
}

// Chunk-parallel cone marching, for calls without halo bits.  The recurrence
// itself is cheap (four FP32 operations per candidate) but serial; the grid
// lookups are not.  A
// pre-pass walks each ray's recurrence once, one lane per ray, and records
// t at the start of every chunk of 64 candidates; the count and fill passes
// then take one lane per (ray, chunk), so a launch has ~12 times as many
// independent lanes as rays to hide the lookup latency.  Tasks are ordered
// chunk-major (task = chunk * n_rays + ray): a wave's loads and stores of
// the per-chunk arrays are contiguous.  A ray longer than the stored chunks
// is finished by the task of its last stored chunk.
__global__ __launch_bounds__(kRaysPerBlock) void cone_starts_kernel(
    const float* __restrict__ rays_o, const float* __restrict__ rays_d, const int32_t* __restrict__ grid_id,
    int64_t n_rays, bool has_grid_id, GridK g, ClipK c, StepK p, int n_masks, float* __restrict__ chunk_t,
    float* __restrict__ t_far_out, int32_t* __restrict__ extra, ConeTable tab) {
    const int64_t r = static_cast<int64_t>(blockIdx.x) * kRaysPerBlock + threadIdx.x;
    if (r >= n_rays) return;
    float o[3], d[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        o[i] = rays_o[3 * r + i];
        d[i] = rays_d[3 * r + i];
    }
    float t_near = 0.0f, t_far = 0.0f;
    const int gid = has_grid_id ? grid_id[r] : 0;
    bool live = gid >= 0 && gid < g.n_grids;
    live = clip_ray(o, d, c, p.near_plane, p.far_plane, t_near, t_far) && live;
    t_far_out[r] = live ? t_far : -INFINITY;
    extra[r] = 0;
    float t = t_near;
    const bool tabled = tab.n > 0 && t_near == tab.t[0];  // starts at the near plane
    for (int j = 0; j < n_masks; ++j) {
        live = live && t < t_far;  // the chunk's first candidate exists
        chunk_t[static_cast<int64_t>(j) * n_rays + r] = live ? t : INFINITY;
        if (__builtin_amdgcn_ballot_w64(live && !tabled) == 0ull) {
            // the wave's live rays all follow the table (or have all
            // ended): the next chunk's start, past the ray's end too
            if (tabled) t = tab.t[kTableStride * (j + 1)];
        } else if (p.no_stall) {
            // every step advances, so the candidates inside the ray are a
            // prefix: the steps are taken without tests (past the ray's
            // end t runs on; the next chunk's test sees that)
#pragma unroll 8
            for (int u = 0; u < kWave; ++u) t = t + __builtin_amdgcn_fmed3f(t * p.cone, p.dt, p.dt_max);
        } else {
            // 64 steps without branches: a ray that ends keeps its last t
#pragma unroll 8
            for (int u = 0; u < kWave; ++u) {
                const float t1 = t + __builtin_amdgcn_fmed3f(t * p.cone, p.dt, p.dt_max);
                live = live && t < t_far && t1 > t;
                t = live ? t1 : t;
            }
        }
    }
}

// Occupancy bits of the 64 candidates of one chunk from its first t; `ended`
// tells whether the ray's candidates stop inside the chunk.
template <int LOOKUP>
__device__ __forceinline__ uint64_t cone_chunk_bits(const uint32_t* __restrict__ bits, const GridK& g, uint32_t word0,
                                                    const float o[3], const float d[3], float& t, float t_far,
                                                    const StepK& p, bool& ended) {
    SkipRay sk{};  // not read
    float skip_end = -INFINITY;
    uint64_t m = 0ull;
    ended = false;
#pragma unroll 1
    for (int b = 0; b < kWave / kConeBatch; ++b) {
        float tb[kConeBatch + 1];
        const int n_valid = cone_steps(t, t_far, p, tb);
        const uint32_t hits =
            cone_hits<LOOKUP, false>(bits, nullptr, g, sk, skip_end, word0, o, d, tb, n_valid) & ((1u << n_valid) - 1u);
        m |= static_cast<uint64_t>(hits) << (b * kConeBatch);
        if (n_valid < kConeBatch) {
            ended = true;
            break;
        }
        t = tb[kConeBatch];
    }
    return m;
}

constexpr int kTaskThreads = 256;

template <int LOOKUP>
__global__ __launch_bounds__(kTaskThreads) void count_cone_chunks_kernel(
    const float* __restrict__ rays_o, const float* __restrict__ rays_d, const int32_t* __restrict__ grid_id,
    int64_t n_rays, const uint32_t* __restrict__ bits, GridK g, StepK p,
    int n_masks, const float* __restrict__ chunk_t, const float* __restrict__ t_far_in,
    uint64_t* __restrict__ masks, int32_t* __restrict__ extra) {
    const int64_t task = static_cast<int64_t>(blockIdx.x) * kTaskThreads + threadIdx.x;
    if (task >= static_cast<int64_t>(n_masks) * n_rays) return;
    const int j = static_cast<int>(task / n_rays);
    const int64_t r = task - static_cast<int64_t>(j) * n_rays;
    float t = chunk_t[task];
    if (!(t < INFINITY)) {
        masks[task] = 0ull;
        return;
    }
    const float t_far = t_far_in[r];
    float o[3], d[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        o[i] = rays_o[3 * r + i];
        d[i] = rays_d[3 * r + i];
    }
    uint32_t word0;
    grid_of_ray<LOOKUP>(grid_id, r, g, word0);  // valid: the ray has candidates
    bool ended;
    masks[task] = cone_chunk_bits<LOOKUP>(bits, g, word0, o, d, t, t_far, p, ended);
    if (j == n_masks - 1 && !ended) {
        // past the stored chunks: count the rest of the ray here
        int count = 0;
        for (int k0 = n_masks * kWave; k0 < kMaxCandidates; k0 += kWave) {
            count += __popcll(cone_chunk_bits<LOOKUP>(bits, g, word0, o, d, t, t_far, p, ended));
            if (ended) break;
        }
        extra[r] = count;
    }
}

// Per-ray counts from the chunk masks (capped at max_per_ray) and the
// workgroup sums of the scan.
__global__ __launch_bounds__(kRaysPerBlock) void cone_counts_kernel(int64_t n_rays, int n_masks, int max_per_ray,
                                                                    const uint64_t* __restrict__ masks,
                                                                    const int32_t* __restrict__ extra,
                                                                    int32_t* __restrict__ packed_info,
                                                                    int64_t* __restrict__ block_sums) {
    const int64_t r = static_cast<int64_t>(blockIdx.x) * kRaysPerBlock + threadIdx.x;
    int n = 0;
    if (r < n_rays) {
        int64_t total = extra[r];
#pragma unroll 8
        for (int j = 0; j < n_masks; ++j) total += __popcll(masks[static_cast<int64_t>(j) * n_rays + r]);
        if (max_per_ray > 0) total = min(total, static_cast<int64_t>(max_per_ray));
        n = static_cast<int>(min(total, static_cast<int64_t>(kMaxCandidates)));
        packed_info[2 * r + 1] = n;
    }
    const int sum = wave_sum(n);  // <= 64 * 2^24 fits int32
    if (threadIdx.x == 0) block_sums[blockIdx.x] = sum;
}

template <int LOOKUP>
__global__ __launch_bounds__(kTaskThreads) void fill_cone_chunks_kernel(
    const float* __restrict__ rays_o, const float* __restrict__ rays_d, const int32_t* __restrict__ grid_id,
    int64_t n_rays, const uint32_t* __restrict__ bits, GridK g, StepK p,
    int n_masks, const float* __restrict__ chunk_t, const float* __restrict__ t_far_in,
    const uint64_t* __restrict__ masks, const int32_t* __restrict__ packed_info, int64_t capacity,
    float* __restrict__ t_starts, float* __restrict__ t_ends, int32_t* __restrict__ status) {
    const int64_t task = static_cast<int64_t>(blockIdx.x) * kTaskThreads + threadIdx.x;
    if (task >= static_cast<int64_t>(n_masks) * n_rays) return;
    const int j = static_cast<int>(task / n_rays);
    const int64_t r = task - static_cast<int64_t>(j) * n_rays;
    float t = chunk_t[task];
    if (!(t < INFINITY)) return;
    const int limit = packed_info[2 * r + 1];
    int idx = 0;  // samples of the ray before this chunk
    for (int q = 0; q < j; ++q) idx += __popcll(masks[static_cast<int64_t>(q) * n_rays + r]);
    if (idx >= limit) return;
    const int64_t start = packed_info[2 * r];
    const float t_far = t_far_in[r];
    bool overflow = false;
    auto emit = [&](float a, float b) {
        const int64_t pos = start + idx;
        if (pos >= 0 && pos < capacity) {
            t_starts[pos] = a;
            t_ends[pos] = b;
        } else {
            overflow = true;
        }
        ++idx;
    };
    const uint64_t m = masks[task];
    bool ended = false;
#pragma unroll 1
    for (int b = 0; b < kWave / kConeBatch && idx < limit; ++b) {
        float tb[kConeBatch + 1];
        const int n_valid = cone_steps(t, t_far, p, tb);
        const uint32_t hits = static_cast<uint32_t>(m >> (b * kConeBatch)) & ((1u << n_valid) - 1u);
#pragma unroll
        for (int u = 0; u < kConeBatch; ++u) {
            if (((hits >> u) & 1u) != 0u && idx < limit) emit(tb[u], tb[u + 1]);
        }
        if (n_valid < kConeBatch) {
            ended = true;
            break;
        }
        t = tb[kConeBatch];
    }
    if (j == n_masks - 1 && !ended && idx < limit) {
        // past the stored chunks: look the rest of the ray up again
        float o[3], d[3];
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            o[i] = rays_o[3 * r + i];
            d[i] = rays_d[3 * r + i];
        }
        uint32_t word0;
        grid_of_ray<LOOKUP>(grid_id, r, g, word0);
        SkipRay sk{};
        float skip_end = -INFINITY;
        for (int k0 = n_masks * kWave; k0 < kMaxCandidates && idx < limit; k0 += kConeBatch) {
            float tb[kConeBatch + 1];
            const int n_valid = cone_steps(t, t_far, p, tb);
            const uint32_t hits = cone_hits<LOOKUP, false>(bits, nullptr, g, sk, skip_end, word0, o, d, tb, n_valid) &
                                  ((1u << n_valid) - 1u);
#pragma unroll
            for (int u = 0; u < kConeBatch; ++u) {
                if (((hits >> u) & 1u) != 0u && idx < limit) emit(tb[u], tb[u + 1]);
            }
            if (n_valid < kConeBatch) break;
            t = tb[kConeBatch];
        }
    }
    if (overflow && status != nullptr) *status = NACC_ECAPACITY;
}

// ---------------------------------------------------------------------------
// Cone steps with halo bits (the skip buffer's, or built for the call).  A
// chunk's 64 candidates form 8 segments of kConeBatch; the count pass tests
// one halo bit per segment at its centre, and looks up, one segment per
// lane, those that may hold samples.  A segment's 8 occupancy bits are byte s
// of its chunk's mask (the mask of the plain passes).  The fill pass does not
// walk the recurrence again: its times are on the near-plane lattice, or
// follow from the t at the start of their segment, which is stored for rays
// that do not start at the near plane.
//
// A clear halo bit proves a segment empty when all its midpoints provably
// map within kHaloReach cells of the centre's cell in the grid the centre is
// looked up in: the midpoints lie within h of the centre in t (h half the
// segment's extent plus rounding), so within |d_i| h plus the rounding of
// positions on axis i; cascades also need every midpoint on the centre's
// level (its max |x_i| bracketed on both sides), and the contraction
// shrinks distances by at most L(r) = (2 - 1/r)/r beyond radius r >= 1
// (at most 1 everywhere).  Where the bound fails the segment is looked up.
// ---------------------------------------------------------------------------
constexpr int kSegsPerChunk = kWave / kConeBatch;
constexpr int kTaskWaves = kTaskThreads / kWave;
constexpr int kSegQueue = kWave * kSegsPerChunk;  // every segment of a wave's chunks

// Whether a chunk whose midpoints lie in [ta, tb] may hold samples, by the
// distance field of the skip buffer (box and cascade lookups): as
// cone_segment_live, with the coarse cells closer than the centre's distance
// in place of the halo's reach.
template <int LOOKUP>
__device__ __forceinline__ bool cone_chunk_live(const GridK& g, const uint8_t* __restrict__ dist, uint32_t word0,
                                                const float o[3], const float d[3], const ConeHalo& k, float ta,
                                                float tb) {
    const float tc = (ta + tb) * 0.5f;
    const float h = (tb - ta) * 0.5f + fabsf(tb) * 0x1p-20f;
    const float x0 = o[0] + d[0] * tc, x1 = o[1] + d[1] * tc, x2 = o[2] + d[2] * tc;
    const float slack_x = (k.omax + k.dmax * fabsf(tb) + 1.0f) * 0x1p-19f;
    const Probe q = probe<LOOKUP>(g, word0, x0, x1, x2);
    // the coarse cells less than D cells from the centre's are empty: every
    // fine cell up to 4 (D - 1) cells from the centre's
    const float reach = 4.0f * static_cast<float>(static_cast<int>(dist[q.coarse]) - 1) * (1.0f - 0x1p-10f);
    float dev = k.v * h + k.smax * slack_x;
    bool open = false;
    if (LOOKUP == NACC_LOOKUP_CASCADE) {
        const float dm = k.dmax * h + slack_x;
        const int l_hi = cascade_level(q.m + dm, g);
        open = l_hi != 0 && !(q.m - dm > ldexpf(g.base, l_hi - 1));
        dev = ldexpf(dev, -q.level);
    }
    return open || !(dev + static_cast<float>(g.res) * 0x1p-17f <= reach);
}

// The cells a segment's candidates can map to, from its centre and bound:
// all empty, all occupied, or undecided (also where they are more than two
// rows on an axis, or a row of them lies in two words).
enum class Cells { kEmpty, kOccupied, kUndecided };

__device__ __forceinline__ Cells cells_within(__amdgpu_buffer_rsrc_t grs, const GridK& g, uint32_t word0,
                                              const float x[3], float dev) {
    uint32_t a[3], b[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const float u = (x[i] - g.lo[i]) * g.s[i];
        a[i] = static_cast<uint32_t>(static_cast<int>(clamp_cell(u - dev, g.top)));
        b[i] = static_cast<uint32_t>(static_cast<int>(clamp_cell(u + dev, g.top)));
    }
    const uint32_t nz = b[2] - a[2];
    bool whole = b[0] - a[0] <= 1u && b[1] - a[1] <= 1u;
    uint32_t w[4], cell[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        cell[i] = __umul24(i < 2 ? a[0] : b[0], g.res2) +
                  (__umul24((i & 1) == 0 ? a[1] : b[1], static_cast<uint32_t>(g.res)) + a[2]);
        w[i] = grid_word(grs, word0 + (cell[i] >> 5));
        whole = whole && (cell[i] & 31u) + nz <= 31u;
    }
    uint32_t any = 0u, all = ~0u;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const uint32_t row = w[i] >> (cell[i] & 31u);
        any |= row;
        all &= row;
    }
    const uint32_t m = (2u << (nz & 31u)) - 1u;
    if (!whole) return Cells::kUndecided;
    return (any & m) == 0u ? Cells::kEmpty : (all & m) == m ? Cells::kOccupied : Cells::kUndecided;
}

// The LDS of the segment count for `rays` rays a workgroup.
constexpr int kSegmentRaysMax = kRaysPerBlock;
constexpr int kConeRayFloats = 20;  // 16-byte fields, 16 different ones in different banks
constexpr int kChunkQueue = kWave + kSegsPerChunk;
constexpr int kSegStack = 2 * kWave;
// A queued segment: its number (bits 0 to 2), chunk (3 to 8), ray (9 to 14),
// levels and whether its ray is not on the table.
constexpr uint32_t kSegOneLevel = 1u << 15, kSegWide = 1u << 16;
constexpr uint32_t kSegOwnLattice = 1u << 17;
constexpr int kSegLevelShift = 18;
struct ConeLds {
    int tab, masks, starts, seg_t, seg_id, near_t, near_end, near_id, chunks, bytes;  // byte offsets, after the rays
};
__host__ __device__ inline int mask_row_bytes(int n_masks) { return (n_masks | 1) * 8; }  // bytes a ray
__host__ __device__ inline ConeLds cone_lds(int rays, int n_masks, bool walks, bool ranges) {
    ConeLds l;
    l.masks = rays * kConeRayFloats * 4;
    l.tab = l.masks + rays * mask_row_bytes(n_masks);
    l.starts = l.tab + (n_masks * kTableStride + 1) * 4;
    l.seg_t = l.starts + (walks ? rays * (n_masks + 1) * 4 : 0);
    l.seg_id = l.seg_t + kTaskWaves * kSegStack * 4;
    l.near_t = l.seg_id + kTaskWaves * kSegStack * 4;
    const int near = ranges ? kTaskWaves * kSegStack * 4 : 0;
    l.near_end = l.near_t + near;
    l.near_id = l.near_end + near;
    l.chunks = l.near_id + near;
    l.bytes = l.chunks + kTaskWaves * kChunkQueue * 2;
    return l;
}

// In a ray's count of stored samples: the ray is not on the table.
constexpr uint32_t kOwnLattice = 1u << 31;

// Count pass of the cone steps with halo bits, one launch.  A workgroup takes
// `rays` consecutive rays, a quarter of them a wave.  Each wave works
// through three stages, 64 items at a time, one per lane: chunks of its rays
// that begin before the ray ends, kept if they may hold samples (by the
// halo bit of the chunk's centre under contraction, by the distance field
// otherwise; without one all are kept); the eight segments of the kept
// chunks, kept by their halo bits; and the candidates of the kept segments,
// looked up.  What a stage keeps goes on a stack in LDS, and a later stage
// runs as soon as it can fill the wave, so that every stage but the last
// of each wave runs with full lanes whatever the share of items kept.  The
// hits, a byte a segment, make the chunk masks in LDS; the first wave then
// counts each ray's samples and writes the masks that are not empty for the
// fill pass.
// Chunks and segments of a ray that starts at the near plane read their
// starts from the table; other rays' chunk starts are walked at the beginning,
// one ray per lane (`walks`: the lookup has a clip box, or there is no
// table), and their segment starts from them.  A stalled step repeats t:
// the lookups find no candidate there.
// Bound by VALU issue (84% of a 64-lane instruction per SIMD every 4 clocks on
// the cascades, 75% with the contraction).  262,144 rays of a cascade of 15
// chunks (92 segments inside the ray, 55 of kept chunks, 19 looked up, 10
// holding samples): 129 us, where a pass for the chunk starts, one lane per
// chunk with the wave's segments looked up together, and one for the counts
// took 7.5 + 166 + 11.  131,071 rays of 39 contracted chunks (42 segments
// near occupied cells, most of them decided by cells_within): 137 us, where
// the starts with culling, the scan of a task list, the list, the segments
// and the counts took 27 + 18 + 17 + 136 + 15.
template <int LOOKUP>
__global__ __launch_bounds__(kTaskThreads) void count_cone_kernel(
    const float* __restrict__ rays_o, const float* __restrict__ rays_d, const int32_t* __restrict__ grid_id,
    int64_t n_rays, const uint32_t* __restrict__ bits, const uint32_t* __restrict__ halo,
    const uint8_t* __restrict__ dist, GridK g, ClipK c, StepK p, int n_masks, int rays, int walks,
    int32_t* __restrict__ packed_info, int64_t* __restrict__ block_sums, uint64_t* __restrict__ masks,
    uint32_t* __restrict__ ray_stored, float* __restrict__ seg_t, float* __restrict__ t_more,
    float* __restrict__ t_far_out, uint64_t* __restrict__ sample_chunks, ConeTable tab) {
    extern __shared__ float4 lds4[];
    char* const lds = reinterpret_cast<char*>(lds4);
    constexpr bool kRanges = LOOKUP == NACC_LOOKUP_CONTRACT;
    const ConeLds l = cone_lds(rays, n_masks, walks != 0, kRanges);
    const int stride = mask_row_bytes(n_masks);
    float* const s_tab = reinterpret_cast<float*>(lds + l.tab);
    float* const s_starts = reinterpret_cast<float*>(lds + l.starts);
    const int lane = lane_id();
    const int wave = uniform<int>(static_cast<int>(threadIdx.x) / kWave);
    const int64_t first = static_cast<int64_t>(blockIdx.x) * rays;
    const __amdgpu_buffer_rsrc_t hrs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint32_t*>(halo), 0, static_cast<int>(g.halo_bytes), kBufferWord3);
    const __amdgpu_buffer_rsrc_t grs = grid_rsrc(bits, g);
    for (int i = threadIdx.x; i < tab.n; i += kTaskThreads) s_tab[i] = tab.t[i];
    for (int i = threadIdx.x; i < rays * stride / 8; i += kTaskThreads) {
        reinterpret_cast<uint64_t*>(lds + l.masks)[i] = 0ull;
    }
    // the rays, one per lane of the first wave
    bool own_lattice = false;
    float t_far = -INFINITY, t_end = INFINITY;  // t_end: t after the stored chunks, where the ray goes on
    float o[3] = {0.0f, 0.0f, 0.0f}, d[3] = {0.0f, 0.0f, 0.0f};
    uint32_t word0 = 0;
    const int64_t r = first + threadIdx.x;
    const bool mine = static_cast<int>(threadIdx.x) < rays && r < n_rays;
    if (static_cast<int>(threadIdx.x) < rays) {
        float t = 0.0f;
        bool tabled = true;
        if (mine) {
#pragma unroll
            for (int i = 0; i < 3; ++i) {
                o[i] = rays_o[3 * r + i];
                d[i] = rays_d[3 * r + i];
            }
            bool live = grid_of_ray<LOOKUP>(grid_id, r, g, word0);
            live = clip_ray(o, d, c, p.near_plane, p.far_plane, t, t_far) && live;
            if (!live) t_far = -INFINITY;
            tabled = !live || (tab.n > 0 && t == tab.t[0]);
            own_lattice = !tabled;
        }
        const ConeHalo k = cone_halo_ray(g, o, d);
        float4* const ray = lds4 + threadIdx.x * (kConeRayFloats / 4);
        ray[0] = make_float4(o[0], o[1], o[2], t_far);
        ray[1] = make_float4(d[0], d[1], d[2], __uint_as_float(word0));
        ray[2] = make_float4(k.v, k.omax, k.dmax, k.dnorm);
        ray[3] = make_float4(k.onorm, tabled ? 1.0f : 0.0f, __uint_as_float(word0 / g.words), 0.0f);
        if (tabled) {
            const float te = tab.n > 0 ? tab.t[kTableStride * n_masks] : INFINITY;
            if (te < t_far) t_end = te;
        }
        if (walks != 0 && __builtin_amdgcn_ballot_w64(!tabled) != 0ull) {
            float* const starts = s_starts + threadIdx.x * (n_masks + 1);
            for (int j = 0; j < n_masks; ++j) {
                starts[j] = t < t_far ? t : INFINITY;
#pragma unroll 8
                for (int u = 0; u < kWave; ++u) t = t + __builtin_amdgcn_fmed3f(t * p.cone, p.dt, p.dt_max);
            }
            starts[n_masks] = t < t_far ? t : INFINITY;
            if (!tabled && t < t_far) t_end = t;
        }
        if (mine) t_far_out[r] = t_far;
    }
    __syncthreads();

    uint16_t* const c_id = reinterpret_cast<uint16_t*>(lds + l.chunks) + wave * kChunkQueue;
    float* const q_t = reinterpret_cast<float*>(lds + l.seg_t) + wave * kSegStack;
    uint32_t* const q_id = reinterpret_cast<uint32_t*>(lds + l.seg_id) + wave * kSegStack;
    float* const r_t = reinterpret_cast<float*>(lds + l.near_t) + wave * kSegStack;
    float* const r_end = reinterpret_cast<float*>(lds + l.near_end) + wave * kSegStack;
    uint32_t* const r_id = reinterpret_cast<uint32_t*>(lds + l.near_id) + wave * kSegStack;
    const int per = rays / kTaskWaves;  // the wave's rays
    const int n_flat = per * n_masks;   // its chunks, ray by ray; f / n_masks by this reciprocal (f < 1,024)
    const uint32_t inv = 65536u / static_cast<uint32_t>(n_masks) + 1u;
    ConeHalo k;
    k.smax = fmaxf(fmaxf(g.s[0], g.s[1]), g.s[2]);
    int f0 = 0, n_chunks = 0, n_near = 0, n_segs = 0;  // chunks taken; entries of the stacks
    for (;;) {
        const bool listed = n_chunks == 0 && f0 >= n_flat;  // no more segments come
        if (n_segs >= kWave || (n_segs > 0 && n_near == 0 && listed)) {
            // look 64 segments up
            const int n = min(n_segs, kWave);
            n_segs -= n;
            const bool has = lane < n;
            const int i = n_segs + (has ? lane : 0);
            const float t0 = q_t[i];
            const uint32_t id = q_id[i];
            const int s = static_cast<int>(id & (kSegsPerChunk - 1));
            const int j = static_cast<int>((id >> 3) & 63u);
            const int rl = static_cast<int>((id >> 9) & 63u);
            const SegLevels lv{static_cast<int>(id >> kSegLevelShift), (id & kSegOneLevel) != 0u, (id & kSegWide) != 0u};
            const float4 a = lds4[rl * (kConeRayFloats / 4)], b = lds4[rl * (kConeRayFloats / 4) + 1];
            const float so[3] = {a.x, a.y, a.z}, sd[3] = {b.x, b.y, b.z};
            const float s_far = has ? a.w : -INFINITY;
            uint32_t hits;
            if (LOOKUP == NACC_LOOKUP_CASCADE && ballot(lv.wide) != 0ull) {
                SkipRay sk{};
                float skip_end = -INFINITY;
                float tb[kConeBatch + 1];
                const int n_valid = cone_steps(t0, s_far, p, tb);
                hits = cone_hits<LOOKUP, false>(bits, nullptr, g, sk, skip_end, __float_as_uint(b.w), so, sd, tb,
                                                n_valid) &
                       ((1u << n_valid) - 1u);
            } else {
                hits = segment_hits<LOOKUP>(grs, g, p, __float_as_uint(b.w), lv, so, sd, t0, s_far);
            }
            if (hits != 0u) {
                lds[l.masks + rl * stride + j * kSegsPerChunk + s] = static_cast<char>(hits);
                if ((id & kSegOwnLattice) != 0u) {
                    seg_t[(static_cast<int64_t>(j) * n_rays + first + rl) * kSegsPerChunk + s] = t0;
                }
            }
        } else if (kRanges && (n_near >= kWave || (n_near > 0 && listed))) {
            // 64 segments by the cells within their bounds
            const int n = min(n_near, kWave);
            n_near -= n;
            const bool has = lane < n;
            const int i = n_near + (has ? lane : 0);
            const float ta = r_t[i], te = r_end[i];
            const uint32_t id = r_id[i];
            const int rl = static_cast<int>((id >> 9) & 63u);
            const float4* const ray = lds4 + rl * (kConeRayFloats / 4);
            const float4 a = ray[0], b = ray[1], kc = ray[2], kd = ray[3];
            const float so[3] = {a.x, a.y, a.z}, sd[3] = {b.x, b.y, b.z};
            k.v = kc.x, k.omax = kc.y, k.dmax = kc.z, k.dnorm = kc.w, k.onorm = kd.x;
            SegLevels lv;
            float x[3], dev;
            const bool bound = cone_segment_cells<LOOKUP>(g, so, sd, k, ta, te, lv, x, dev);
            Cells cells = cells_within(grs, g, __float_as_uint(b.w), x, bound ? dev : 0.0f);
            // all candidates are samples only if all lie inside the ray (the
            // table's steps never stall)
            const bool inside = (p.no_stall != 0 || kd.y != 0.0f) && te <= a.w;
            if (!(bound && dev <= static_cast<float>(kHaloReach)) || (cells == Cells::kOccupied && !inside)) {
                cells = Cells::kUndecided;
            }
            if (has && cells == Cells::kOccupied) {
                const int j = static_cast<int>((id >> 3) & 63u), s = static_cast<int>(id & (kSegsPerChunk - 1));
                lds[l.masks + rl * stride + j * kSegsPerChunk + s] = static_cast<char>(0xff);
                if ((id & kSegOwnLattice) != 0u) {
                    seg_t[(static_cast<int64_t>(j) * n_rays + first + rl) * kSegsPerChunk + s] = ta;
                }
            }
            const bool left = has && cells == Cells::kUndecided;
            const uint64_t m = ballot(left);
            if (left) {
                const int pos = n_segs + bits_below(m);
                q_t[pos] = ta;
                q_id[pos] = id;
            }
            n_segs += static_cast<int>(__popcll(m));
        } else if (n_chunks >= kWave / kSegsPerChunk || (n_chunks > 0 && f0 >= n_flat)) {
            // the segments of 8 chunks
            const int n = min(n_chunks, kWave / kSegsPerChunk);
            n_chunks -= n;
            const int e = lane / kSegsPerChunk, s = lane % kSegsPerChunk;
            bool live = e < n;
            const uint32_t id = c_id[n_chunks + (live ? e : 0)];
            const int j = static_cast<int>(id & 63u);
            const int rl = static_cast<int>(id >> 6);
            const float4* const ray = lds4 + rl * (kConeRayFloats / 4);
            const float4 a = ray[0], b = ray[1], kc = ray[2], kd = ray[3];
            float ta = s_tab[kTableStride * j + s], te = s_tab[kTableStride * j + s + 1];
            if (walks != 0 && ballot(kd.y == 0.0f) != 0ull) {
                float t = s_starts[rl * (n_masks + 1) + j], t0 = t;
                for (int v = 0; v < kSegsPerChunk; ++v) {
                    if (v <= s) t0 = t;
#pragma unroll
                    for (int u = 0; u < kConeBatch; ++u) t = t + __builtin_amdgcn_fmed3f(t * p.cone, p.dt, p.dt_max);
                    if (kd.y == 0.0f && v == s) {
                        ta = t0;
                        te = t;
                    }
                }
            }
            const float so[3] = {a.x, a.y, a.z}, sd[3] = {b.x, b.y, b.z};
            k.v = kc.x, k.omax = kc.y, k.dmax = kc.z, k.dnorm = kc.w, k.onorm = kd.x;
            live = live && ta < a.w;
            SegLevels lv{0, true, false};
            live &= cone_segment_live<LOOKUP>(g, hrs, __float_as_uint(kd.z), so, sd, k, ta, te, lv);
            const uint64_t m = ballot(live);
            const int pos = (kRanges ? n_near : n_segs) + bits_below(m);
            const uint32_t seg = (id << 3) | static_cast<uint32_t>(s) | (kd.y == 0.0f ? kSegOwnLattice : 0u);
            if (kRanges) {
                if (live) {
                    r_t[pos] = ta;
                    r_end[pos] = te;
                    r_id[pos] = seg;
                }
                n_near += static_cast<int>(__popcll(m));
            } else {
                if (live) {
                    q_t[pos] = ta;
                    q_id[pos] = seg | (lv.one ? kSegOneLevel : 0u) | (lv.wide ? kSegWide : 0u) |
                                (static_cast<uint32_t>(lv.hi) << kSegLevelShift);
                }
                n_segs += static_cast<int>(__popcll(m));
            }
        } else if (f0 < n_flat) {
            // 64 chunks
            const int f = f0 + lane;
            bool live = f < n_flat;
            int rl = static_cast<int>((static_cast<uint32_t>(live ? f : 0) * inv) >> 16);
            const int j = live ? f - rl * n_masks : 0;
            rl += wave * per;
            f0 += kWave;
            const float4* const ray = lds4 + rl * (kConeRayFloats / 4);
            const float4 a = ray[0], b = ray[1], kc = ray[2], kd = ray[3];
            float ta = s_tab[kTableStride * j], te = s_tab[kTableStride * (j + 1)];
            if (walks != 0 && kd.y == 0.0f) {
                ta = s_starts[rl * (n_masks + 1) + j];
                te = s_starts[rl * (n_masks + 1) + j + 1];
            }
            const float so[3] = {a.x, a.y, a.z}, sd[3] = {b.x, b.y, b.z};
            k.v = kc.x, k.omax = kc.y, k.dmax = kc.z, k.dnorm = kc.w, k.onorm = kd.x;
            live = live && ta < a.w;
            if (LOOKUP == NACC_LOOKUP_CONTRACT) {
                SegLevels lv;
                live &= cone_segment_live<LOOKUP>(g, hrs, __float_as_uint(kd.z), so, sd, k, ta, te, lv);
            } else if (dist != nullptr) {
                live = live && cone_chunk_live<LOOKUP>(g, dist, __float_as_uint(b.w), so, sd, k, ta, te);
            }
            const uint64_t m = ballot(live);
            if (live) c_id[n_chunks + bits_below(m)] = static_cast<uint16_t>((rl << 6) | j);
            n_chunks += static_cast<int>(__popcll(m));
        } else {
            break;
        }
        wave_lds_sync();
    }
    __syncthreads();

    if (wave != 0) return;
    int n = 0;
    if (mine) {
        int64_t total = 0;
        uint64_t holding = 0ull;
        const uint64_t* const mm = reinterpret_cast<const uint64_t*>(lds + l.masks + threadIdx.x * stride);
#pragma unroll 4
        for (int j = 0; j < n_masks; ++j) {
            const uint64_t m = mm[j];
            if (m != 0ull) {  // the fill pass reads no others
                masks[static_cast<int64_t>(j) * n_rays + r] = m;
                holding |= 1ull << j;
            }
            total += __popcll(m);
        }
        sample_chunks[r] = holding;
        ray_stored[r] = static_cast<uint32_t>(total) | (own_lattice ? kOwnLattice : 0u);
        t_more[r] = t_end;
        if (t_end < INFINITY) {
            // past the stored chunks: count the rest of the ray here
            bool ended = false;
            float t = t_end;
            for (int k0 = n_masks * kWave; k0 < kMaxCandidates && !ended; k0 += kWave) {
                total += __popcll(cone_chunk_bits<LOOKUP>(bits, g, word0, o, d, t, t_far, p, ended));
            }
        }
        if (p.max_per_ray > 0) total = min(total, static_cast<int64_t>(p.max_per_ray));
        n = static_cast<int>(min(total, static_cast<int64_t>(kMaxCandidates)));
        packed_info[2 * r + 1] = n;
    }
    const int sum = wave_sum(n);  // <= 64 * 2^24 fits int32
    if (lane == 0) block_sums[blockIdx.x] = sum;
}

// Count pass of uniform steps through the box with halo bits.  A workgroup
// takes `rays` consecutive rays, a quarter of them a wave.  A wave's segments
// (of G candidates, the smallest its rays allow), ray after ray, are tested
// 64 at a time, one per lane: a clear halo bit leaves a segment out, a clear
// hole bit (holes may be nullptr) makes all its candidates samples, and what
// is left goes on a stack in LDS, from which 64 eighths of eight candidates
// each are looked up at a time, one per lane, the eight grid words in flight
// together.  All lanes work whatever the lengths of the rays and the share
// of segments left.  The hits make the rays' chunk masks in LDS, from which
// they are counted and stored.  Rays of more candidates than stored chunks
// are taken in windows of as many, the masks of the first one stored; rays
// too fast for segments (seg_log 0) look every candidate up.
// Bound by VALU issue (79% of a 64-lane instruction per SIMD every 4 clocks):
// 262,144 rays, 37 segments of 16 inside a ray, 21 near occupied cells: 131 us and 5 us for the hole bits
// (138 with a hole bit read for every segment; 162 without hole bits on these
// small blobs, a solid ball of 64 cells across gains more), 208 us with a wave
// per ray after ray, half of whose lanes tested no segment and a fifth looked no
// candidate up.
// SPREAD (more than one grid): of 64 runs a lane looks up one candidate of
// eight, so that neighbouring lanes read neighbouring cells, and a ballot
// holds eight runs' bytes; it reads a ray's data anew where the ray changes.
// With a run a lane every load touches as many cache lines as lanes, the same
// ones eight times over, and rays of many grids drive them out of the L1 and
// L2 in between.  262,144 rays in 64 grids of blobs: 407 -> 305 us a call, of 2%
// random cells 627 -> 427, in 2 grids 270 and 270, 339 and 297.  One grid stays
// in the L2: blobs 297 both ways, 2% random cells 321 and 295, but a thin shell
// 138 and 143, 0.02% random cells 107 and 112.
// CAP (max_per_ray > 0): the candidates of the rays are taken in turns, and a
// ray that holds the cap's number of samples after one takes part no more:
// what its later turns hold is cut off.  A turn is as long as the cap (no ray
// reaches it earlier) or has a round of the wave's segments, two where the
// wave has eight rays or more.  262,144 rays, cells at random (2%), cap 1: 320
// us a call without turns, 170 with; fine steps (8,660 candidates a ray), cap
// 16: 1,329 -> 676 us, a solid box 235 -> 163 us, a ball 368 -> 287 us (343 and
// 314 us with turns of one round; 8,192 rays, two a wave, a solid box 89 us
// with two rounds, 72 with one).
constexpr int kBoxRayFloats = 12;  // 16-byte fields, 16 different ones in different banks

__host__ __device__ inline int box_lds(int rays, int n_masks) {
    return rays * (kBoxRayFloats * 4 + mask_row_bytes(n_masks)) + kTaskWaves * kSegStack * 4;
}

template <bool CAP, bool SPREAD>
__global__ __launch_bounds__(kTaskThreads) void count_box_kernel(
    const float* __restrict__ rays_o, const float* __restrict__ rays_d, const int32_t* __restrict__ grid_id,
    int64_t n_rays, const uint32_t* __restrict__ bits, const uint32_t* __restrict__ halo,
    const uint32_t* __restrict__ holes, GridK g, ClipK c, StepK p, int n_masks, int rays,
    int32_t* __restrict__ packed_info, int64_t* __restrict__ block_sums, uint64_t* __restrict__ masks) {
    extern __shared__ float4 lds4[];
    __shared__ int wave_total[kTaskWaves];
    const int stride = mask_row_bytes(n_masks);
    char* const s_masks = reinterpret_cast<char*>(lds4) + rays * kBoxRayFloats * 4;
    const int lane = lane_id();
    const int wave = uniform<int>(static_cast<int>(threadIdx.x) / kWave);
    uint32_t* const q = reinterpret_cast<uint32_t*>(s_masks + rays * stride) + wave * kSegStack;
    const int64_t block = row_block(), first = block * rays;
    if (static_cast<int>(threadIdx.x) < rays) {  // in the first wave
        const int64_t r = first + threadIdx.x;
        RaySpan span{};
        if (r < n_rays) span = ray_span<NACC_LOOKUP_AABB>(r, rays_o, rays_d, grid_id, g, c, p);
        float4* const ray = lds4 + threadIdx.x * (kBoxRayFloats / 4);
        ray[0] = make_float4(span.o[0], span.o[1], span.o[2], span.t_near);
        ray[1] = make_float4(span.d[0], span.d[1], span.d[2], span.valid ? span.t_far : -INFINITY);
        ray[2] = make_float4(__uint_as_float(span.word0), __uint_as_float(span.grid * g.halo_words),
                             __int_as_float(span.valid ? seg_log(g, span, p) : 0), 0.0f);
    }
    __syncthreads();
    const int per = rays / kTaskWaves;  // the wave's rays, from ray0 on
    const int ray0 = wave * per;
    float t_near = 0.0f, t_far = -INFINITY;
    int own_log = 0;
    if (lane < per) {  // lane i: ray ray0 + i
        const float4* const ray = lds4 + (ray0 + lane) * (kBoxRayFloats / 4);
        t_near = ray[0].w;
        t_far = ray[1].w;
        own_log = __float_as_int(ray[2].z);
    }
    int log_g = 5;
    for (; log_g > kMinSegmentLog2 && ballot(own_log != 0 && own_log < log_g) != 0ull; --log_g) {
    }
    const int part_log = log_g - 3;  // eighths of a segment
    const int per_round = kWave >> part_log;
    // candidates of the ray, at most (the last t below t_far, with the
    // roundings of t and of this bound)
    const float bound = (((t_far - t_near) + (fabsf(t_far) + fabsf(t_near)) * 0x1p-22f) / p.dt) * (1.0f + 0x1p-20f) + 2.0f;
    int k_end = !(t_near < t_far) ? 0
                : bound < static_cast<float>(kMaxCandidates) ? static_cast<int>(bound)
                                                             : kMaxCandidates;
    const __amdgpu_buffer_rsrc_t grs = grid_rsrc(bits, g), hrs = halo_rsrc(halo, g), ors = halo_rsrc(holes, g);
    const int window = n_masks * kWave;
    const int turn_segs = per >= 8 ? 2 * kWave : kWave;
    const int turn = !CAP ? window
                          : min(window, max((min(p.max_per_ray, window) + kWave - 1) & ~(kWave - 1),
                                            max((turn_segs << log_g) / per, kWave)));
    // samples found so far of a ray, where there is a cap
    auto taken_of = [&](int rl) { return reinterpret_cast<int*>(lds4 + rl * (kBoxRayFloats / 4) + 2) + 3; };
    auto take = [&](int rl, int n) {
        __hip_atomic_fetch_add(taken_of(rl), n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WAVEFRONT);
    };
    const uint32_t inv = 65536u / static_cast<uint32_t>(n_masks) + 1u;  // i / n_masks, i < 1,024
    const int64_t wave_first = first + ray0;
    const int n_mine = static_cast<int>(max(min(static_cast<int64_t>(per), n_rays - wave_first), int64_t{0}));
    int count = 0;
    for (int kb = 0; kb < kMaxCandidates; kb += window) {
        for (int i = lane; i < per * (stride / 8); i += kWave) {
            reinterpret_cast<uint64_t*>(s_masks + ray0 * stride)[i] = 0ull;
        }
        int n_q = 0;  // entries of the stack
        for (int kw = kb; kw < kb + window; kw += turn) {
            wave_lds_sync();
            if (CAP && lane < per && taken_of(ray0 + lane)[0] >= p.max_per_ray) k_end = 0;
            const bool last = ballot(k_end > kw + turn) == 0ull || kw + turn >= kb + window;
            const int n_segs = (min(max(k_end - kw, 0), min(turn, kb + window - kw)) + (1 << log_g) - 1) >> log_g;
            const int before = wave_inclusive_sum(n_segs) - n_segs;
            const int total = read_lane(before + n_segs, kWave - 1);
            int f0 = 0;  // segments tested
            for (;;) {
                if (n_q >= per_round || (n_q > 0 && f0 >= total && last)) {
                    // look up 64 runs of eight candidates
                    const int n = min(n_q, per_round);
                    n_q -= n;
                    if constexpr (SPREAD) {
                        // eight runs a load, one after the other, so that
                        // neighbouring lanes read neighbouring cells
                        const int runs = n << part_log, run_mask = (1 << part_log) - 1;
                        int rl = -1;
                        float4 a = make_float4(0.0f, 0.0f, 0.0f, 0.0f), b = a;
                        uint32_t word0 = 0u;
                        uint32_t cell[kConeBatch], w[kConeBatch];
                        uint64_t inside[kConeBatch];
#pragma unroll
                        for (int u = 0; u < kConeBatch; ++u) {
                            const int run = u * (kWave / kConeBatch) + lane / kConeBatch;
                            const uint32_t id = q[n_q + min(run >> part_log, n - 1)];
                            const int r = static_cast<int>(id >> 16);
                            if (ballot(r != rl) != 0ull) {  // another ray, seldom
                                rl = r;
                                const float4* const ray = lds4 + rl * (kBoxRayFloats / 4);
                                a = ray[0];
                                b = ray[1];
                                word0 = __float_as_uint(ray[2].x);
                            }
                            const int byte = static_cast<int>(id & 0xffffu) + (run & run_mask);
                            const float k = static_cast<float>(kb + byte * kConeBatch + lane % kConeBatch);
                            const float t0 = a.w + k * p.dt, t1 = a.w + (k + 1.0f) * p.dt;
                            const float tm = (t0 + t1) * 0.5f;
                            const float x0 = a.x + b.x * tm, x1 = a.y + b.y * tm, x2 = a.z + b.z * tm;
                            cell[u] = cell_index(g, (x0 - g.lo[0]) * g.s[0], (x1 - g.lo[1]) * g.s[1],
                                                 (x2 - g.lo[2]) * g.s[2]);
                            w[u] = grid_word(grs, word0 + (cell[u] >> 5));
                            inside[u] = ballot(run < runs && t0 < b.w);
                        }
                        // lane i: the hits of run i
                        uint64_t m = 0ull;
#pragma unroll
                        for (int u = 0; u < kConeBatch; ++u) {
                            const uint64_t hit = inside[u] & ballot(((w[u] >> (cell[u] & 31u)) & 1u) != 0u);
                            if (lane / kConeBatch == u) m = hit;
                        }
                        const uint32_t hits = static_cast<uint32_t>(m >> (lane % kConeBatch * kConeBatch)) & 0xffu;
                        if (hits != 0u) {
                            const uint32_t id = q[n_q + (lane >> part_log)];
                            const int own = static_cast<int>(id >> 16);
                            s_masks[own * stride + static_cast<int>(id & 0xffffu) + (lane & run_mask)] =
                                static_cast<char>(hits);
                            if (CAP) take(own, __popc(hits));
                        }
                    } else {
                        const int e = lane >> part_log;
                        const bool has = e < n;
                        const uint32_t id = q[n_q + (has ? e : 0)];
                        const int rl = static_cast<int>(id >> 16);
                        const int byte = static_cast<int>(id & 0xffffu) + (lane & ((1 << part_log) - 1));
                        const float4* const ray = lds4 + rl * (kBoxRayFloats / 4);
                        const float4 a = ray[0], b = ray[1], w4 = ray[2];
                        const float k0 = static_cast<float>(kb + byte * kConeBatch);
                        const uint32_t word0 = __float_as_uint(w4.x);
                        float t[kConeBatch + 1];
#pragma unroll
                        for (int u = 0; u <= kConeBatch; ++u) t[u] = a.w + (k0 + static_cast<float>(u)) * p.dt;
                        uint32_t cell[kConeBatch], w[kConeBatch];
#pragma unroll
                        for (int u = 0; u < kConeBatch; ++u) {
                            const float tm = (t[u] + t[u + 1]) * 0.5f;
                            const float x0 = a.x + b.x * tm, x1 = a.y + b.y * tm, x2 = a.z + b.z * tm;
                            cell[u] =
                                cell_index(g, (x0 - g.lo[0]) * g.s[0], (x1 - g.lo[1]) * g.s[1], (x2 - g.lo[2]) * g.s[2]);
                            w[u] = grid_word(grs, word0 + (cell[u] >> 5));
                        }
                        uint32_t hits = 0u;
#pragma unroll
                        for (int u = 0; u < kConeBatch; ++u) {
                            const uint32_t bit = __builtin_amdgcn_ubfe(w[u], cell[u] & 31u, 1u);
                            hits |= (t[u] < b.w ? bit : 0u) << u;
                        }
                        if (has && hits != 0u) {
                            s_masks[rl * stride + byte] = static_cast<char>(hits);
                            if (CAP) take(rl, __popc(hits));
                        }
                    }
                } else if (f0 < total) {
                    // test 64 segments: segment f of the wave, the s-th of ray L
                    const int f = f0 + lane;
                    f0 += kWave;
                    int L = 0;
#pragma unroll
                    for (int step = kSegmentRaysMax / kTaskWaves / 2; step >= 1; step >>= 1) {
                        if (lane_value(before, L + step) <= f) L += step;
                    }
                    const int s = f - lane_value(before, L);
                    const int rl = ray0 + min(L, per - 1);
                    const int k = kw + (s << log_g);
                    const float4* const ray = lds4 + rl * (kBoxRayFloats / 4);
                    const float4 a = ray[0], b = ray[1], w4 = ray[2];
                    const bool valid = f < total && a.w + static_cast<float>(k) * p.dt < b.w;
                    const float tc = a.w + static_cast<float>(k + (1 << (log_g - 1))) * p.dt;
                    const uint32_t halo0 = __float_as_uint(w4.y);
                    const uint32_t cell = halo_cell(g, a.x + b.x * tc, a.y + b.y * tc, a.z + b.z * tc);
                    const bool open = __float_as_int(w4.z) == 0;
                    bool left = valid && (open | halo_bit(hrs, halo0, cell));
                    bool full = false;
                    if (holes != nullptr) {  // read for the segments left alone
                        if (left && !open) full = !halo_bit(ors, halo0, cell);
                        full = full && a.w + static_cast<float>(k + (1 << log_g) - 1) * p.dt < b.w;
                    }
                    left = left && !full;
                    const uint32_t byte = static_cast<uint32_t>(k - kb) >> 3;
                    char* const at = s_masks + rl * stride + byte;
                    if (full) {
                        if (log_g == 3) *reinterpret_cast<uint8_t*>(at) = 0xffu;
                        else if (log_g == 4) *reinterpret_cast<uint16_t*>(at) = 0xffffu;
                        else *reinterpret_cast<uint32_t*>(at) = ~0u;
                        if (CAP) take(rl, 1 << log_g);
                    }
                    const uint64_t m = ballot(left);
                    if (left) q[n_q + bits_below(m)] = (static_cast<uint32_t>(rl) << 16) | byte;
                    n_q += static_cast<int>(__popcll(m));
                } else {
                    break;
                }
                wave_lds_sync();
            }
            if (last) break;
        }
        if (lane < per) {
            const uint64_t* const mm = reinterpret_cast<const uint64_t*>(s_masks + (ray0 + lane) * stride);
#pragma unroll 4
            for (int j = 0; j < n_masks; ++j) count += static_cast<int>(__popcll(mm[j]));
        }
        if (kb == 0) {
            for (int i = lane; i < n_mine * n_masks; i += kWave) {
                const int rl = static_cast<int>((static_cast<uint32_t>(i) * inv) >> 16);
                masks[wave_first * n_masks + i] = *reinterpret_cast<const uint64_t*>(
                    s_masks + (ray0 + rl) * stride + (i - rl * n_masks) * 8);
            }
        }
        if (ballot(k_end > kb + window && !(CAP && count >= p.max_per_ray)) == 0ull) break;
        wave_lds_sync();
    }
    if (CAP) count = min(count, p.max_per_ray);
    if (lane < n_mine) packed_info[2 * (wave_first + lane) + 1] = count;
    const int sum = wave_sum(count);  // <= 16 * 2^24 fits int32
    if (lane == 0) wave_total[wave] = sum;
    __syncthreads();
    if (threadIdx.x == 0 && first < n_rays) {
        int64_t s = 0;
        for (int w = 0; w < kTaskWaves; ++w) s += wave_total[w];
        block_sums[block] = s;
    }
}

// Fill pass of the segment count.  A wave takes up to kFillRays consecutive
// rays, whose chunks holding samples (the count pass leaves their bits per
// ray) are its tasks, ray by ray, chunk by chunk, so in the order of their
// samples in the output.
// Rays that start at the near plane (and end within the stored chunks)
// share one lattice, whose times the workgroup expands from the table into
// LDS: their masks are listed and stored in whole blocks as in the uniform
// fill, a sample's times two LDS reads away.
// Other waves queue the segments that hold samples, 64 at a time: one lane
// per segment runs its 8 recurrence steps from the stored t at its start and
// puts its samples (t_start, t_end) into this wave's LDS slots in output
// order; then the wave stores the slots, 64 consecutive positions at a time
// (each segment's samples stored from its own lane scatter 4-byte writes
// over as many cache lines as lanes).  A ray longer than the stored chunks is
// finished past them by its lane.
// Bound by the write path: 262,144 rays of a cascade, 19.2 M samples, 56 us
// (4.1 TB/s) listed, 97 us by segments; 131,071 contracted rays, 13.0 M
// samples, 44 us and 71 us.  Not storing the segments' starts took 15 and 8
// us off the list (72 and 52 us): the count's scattered writes drain
// meanwhile.  8 rays a wave: the same; 4: 99 and 65 us.
constexpr int kFillSlots = kWave * kConeBatch;  // the samples of 64 segments at most
constexpr int kFillRays = 16;  // the code of a sample holds 4 bits of ray

struct SlotLds {
    int64_t e_pos[kWave];      // output position of an entry's first sample
    float t0[kFillSlots];  // the end is a step from the start
    int32_t e_slot[kWave];     // an entry's first slot
    int32_t e_ray[kWave];
    uint16_t q_id[kSegQueue];
    uint8_t entry[kFillSlots];  // the queue entry (of this round) a slot belongs to
};

union ConeFillLds {
    FillLds list;
    SlotLds slots;
};

// Floats of the lattice in LDS, and bytes of all.
__host__ __device__ inline int cone_fill_times(int n_masks) { return n_masks * kWave + 4; }
__host__ __device__ inline int cone_fill_lds(int n_masks) {
    return cone_fill_times(n_masks) * 4 + kTaskWaves * static_cast<int>(sizeof(ConeFillLds));
}

template <int LOOKUP>
__global__ __launch_bounds__(kTaskThreads, 6) void fill_cone_rays_kernel(
    const float* __restrict__ rays_o, const float* __restrict__ rays_d, const int32_t* __restrict__ grid_id,
    int64_t n_rays, const uint32_t* __restrict__ bits, GridK g, StepK p, int n_masks, int per,
    const float* __restrict__ t_more, const float* __restrict__ t_far_in, const uint64_t* __restrict__ masks,
    const uint32_t* __restrict__ ray_stored, const float* __restrict__ seg_t,
    const uint64_t* __restrict__ sample_chunks, const int32_t* __restrict__ packed_info, int64_t capacity,
    int32_t* __restrict__ ray_indices, float* __restrict__ t_starts, float* __restrict__ t_ends,
    int32_t* __restrict__ status, ConeTable tab) {
    extern __shared__ float4 lds4[];
    float* const s_times = reinterpret_cast<float*>(lds4);
    const int lane = lane_id();
    const int wave = uniform<int>(static_cast<int>(threadIdx.x) / kWave);
    ConeFillLds& lds = reinterpret_cast<ConeFillLds*>(s_times + cone_fill_times(n_masks))[wave];
    const int64_t first = (xcd_grouped<16>(blockIdx.x, gridDim.x) * kTaskWaves + wave) * per;
    // lane i: ray first + i
    const int64_t ray = first + lane;
    int limit = 0;
    int64_t start = 0;
    uint64_t nz = 0ull;
    uint32_t stored = 0u;
    float t_end = INFINITY;  // where the ray goes on past the stored chunks
    if (lane < per && ray < n_rays) {
        limit = packed_info[2 * ray + 1];
        start = packed_info[2 * ray];
        nz = sample_chunks[ray];
        stored = ray_stored[ray];
        t_end = t_more[ray];
    }
    if (limit <= 0) {
        limit = 0;
        nz = 0ull;
        t_end = INFINITY;
    }
    for (int i = threadIdx.x; i + 1 < tab.n; i += kTaskThreads) {
        float t = tab.t[i];
#pragma unroll
        for (int u = 0; u < kConeBatch; ++u) {
            s_times[i * kConeBatch + u] = t;
            t = t + __builtin_amdgcn_fmed3f(t * p.cone, p.dt, p.dt_max);
        }
        if (i + 2 == tab.n) s_times[(i + 1) * kConeBatch] = t;
    }
    __syncthreads();
    const int n_tasks = static_cast<int>(__popcll(nz));
    const int t_before = wave_inclusive_sum(n_tasks) - n_tasks;
    const int t_total = read_lane(t_before + n_tasks, kWave - 1);
    // the wave's samples are on the table, in its stored chunks, and lie side
    // by side inside the output
    const int before = wave_inclusive_sum(limit) - limit;
    const int pos0 = static_cast<int>(read_lane(static_cast<int>(start), 0));
    const int n_out = read_lane(before + limit, kWave - 1);
    const bool on_table = limit == 0 || (stored < kOwnLattice && !(t_end < INFINITY) &&
                                         static_cast<uint32_t>(limit) <= stored &&
                                         start == static_cast<int64_t>(pos0) + before);
    const bool simple = ballot(!on_table) == 0ull && list_fits(pos0, n_out, capacity);
    const FillOut out{ray_indices, t_starts, t_ends};
    const TableTimes times{s_times};
    FillList list = begin_list(pos0);
    bool overflow = false;
    const int start_lo = static_cast<int>(start), start_hi = static_cast<int>(start >> 32);
    const int nz_lo = static_cast<int>(nz), nz_hi = static_cast<int>(nz >> 32);
    int carried = 0;  // samples in earlier rounds of the ray that a round begins with
    for (int tb0 = 0; tb0 < t_total; tb0 += kWave) {
        // task i of the wave: the ray lane L whose tasks hold it, and its
        // (i - first task of L)-th chunk holding samples
        const int i = tb0 + lane;
        int L = 0;
#pragma unroll
        for (int step = kWave / 2; step >= 1; step >>= 1) {
            const int probe_lane = L + step;  // < 64
            if (lane_value(t_before, probe_lane) <= i) L = probe_lane;
        }
        const bool has_task = i < t_total;
        const uint64_t l_nz = (static_cast<uint64_t>(static_cast<uint32_t>(lane_value(nz_hi, L))) << 32) |
                              static_cast<uint32_t>(lane_value(nz_lo, L));
        const int l_first = lane_value(t_before, L);
        const int l_limit = lane_value(limit, L);
        const int64_t r = first + L;
        uint64_t m = 0ull;
        int j = 0;
        if (has_task) {
            j = nth_set_bit(l_nz, i - l_first);
            m = masks[static_cast<int64_t>(j) * n_rays + r];
        }
        // the ray's samples before the chunk
        const int count = static_cast<int>(__popcll(m));
        const int excl = wave_inclusive_sum(count) - count;
        const int ray_base = lane_value(excl, max(l_first - tb0, 0));
        const int in_ray = l_first >= tb0 ? excl - ray_base : excl + carried;
        carried = read_lane(in_ray + count, kWave - 1);
        if (simple) {
            queue_chunks(out, lds.list, times, capped_mask(m, in_ray, l_limit),
                         (static_cast<uint32_t>(L) << kCodeRayShift) | static_cast<uint32_t>(j << kWaveLog2),
                         tb0 + kWave >= t_total, first, list);
            continue;
        }
        SlotLds& z = lds.slots;
        const int64_t task = static_cast<int64_t>(j) * n_rays + r;
        const int base = in_ray;
        const int64_t l_start = (static_cast<int64_t>(lane_value(start_hi, L)) << 32) |
                                static_cast<uint32_t>(lane_value(start_lo, L));
        const float t_far = has_task ? t_far_in[r] : -INFINITY;
        const int l_own = lane_value(stored >= kOwnLattice ? 1 : 0, L);
        // segments holding samples that fall before the ray's limit
        uint32_t todo = 0u;
#pragma unroll
        for (int s = 0; s < kSegsPerChunk; ++s) {
            const bool holds = ((m >> (s * kConeBatch)) & 0xffull) != 0ull;
            const int idx = base + static_cast<int>(__popcll(m & ((1ull << (s * kConeBatch)) - 1ull)));
            if (holds && idx < l_limit) todo |= 1u << s;
        }
        const int n_items = __popc(todo);
        const int before = wave_inclusive_sum(n_items) - n_items;
        const int total = read_lane(before + n_items, kWave - 1);
        {
            int pos = before;
#pragma unroll
            for (int s = 0; s < kSegsPerChunk; ++s) {
                if (((todo >> s) & 1u) != 0u) {
                    z.q_id[pos] = static_cast<uint16_t>(lane | (s << kWaveLog2));
                    ++pos;
                }
            }
        }
        wave_lds_sync();
        const int m_lo = static_cast<int>(m), m_hi = static_cast<int>(m >> 32);
        const int task_lo = static_cast<int>(task), task_hi = static_cast<int>(task >> 32);
        // the stored starts of every round's segments (round k: queue entry
        // 64 k + lane; at most 8 rounds), all loaded before the first round
        // stores anything: one counter tracks a wave's loads and stores, so
        // a load issued after stores is waited for together with them
        float t_seg[kSegsPerChunk];
#pragma unroll
        for (int k = 0; k < kSegsPerChunk; ++k) {
            t_seg[k] = 0.0f;
            if (k * kWave < total) {
                const int q = k * kWave + lane;
                const bool has = q < total;
                const int id = has ? static_cast<int>(z.q_id[q]) : 0;
                const int src = id & (kWave - 1);
                const int64_t s_task = (static_cast<int64_t>(lane_value(task_hi, src)) << 32) |
                                       static_cast<uint32_t>(lane_value(task_lo, src));
                const int s_chunk = lane_value(j, src);
                const bool own = lane_value(l_own, src) != 0;
                if (has) {
                    const int s = id >> kWaveLog2;
                    t_seg[k] = own ? seg_t[s_task * kSegsPerChunk + s] : s_times[s_chunk * kWave + s * kConeBatch];
                }
            }
        }
        for (int qb = 0; qb < total; qb += kWave) {
            const int q = qb + lane;
            const bool has = q < total;
            const int id = has ? static_cast<int>(z.q_id[q]) : 0;
            const int src = id & (kWave - 1);
            const int s = id >> kWaveLog2;
            const float seg_t0 = t_seg[0];
#pragma unroll
            for (int k = 0; k + 1 < kSegsPerChunk; ++k) t_seg[k] = t_seg[k + 1];  // the next round's first
            // the queued segment's task, gathered from its lane (every lane
            // takes part in the permutes)
            const float s_far = lane_value(t_far, src);
            const int s_limit = lane_value(l_limit, src);
            const int s_base = lane_value(base, src);
            const int s_ray = lane_value(static_cast<int>(r), src);
            const int64_t s_start = (static_cast<int64_t>(lane_value(static_cast<int>(l_start >> 32), src)) << 32) |
                                    static_cast<uint32_t>(lane_value(static_cast<int>(l_start), src));
            const uint64_t s_m = (static_cast<uint64_t>(static_cast<uint32_t>(lane_value(m_hi, src))) << 32) |
                                 static_cast<uint32_t>(lane_value(m_lo, src));
            float tb[kConeBatch + 1];
            uint32_t hits = 0u;
            int first = 0;  // the segment's first sample within its ray
            if (has) {
                const int n_valid = cone_steps(seg_t0, s_far, p, tb);
                hits = static_cast<uint32_t>(s_m >> (s * kConeBatch)) & 0xffu & ((1u << n_valid) - 1u);
                first = s_base + static_cast<int>(__popcll(s_m & ((1ull << (s * kConeBatch)) - 1ull)));
            }
            const int n_out = has ? min(__popc(hits), max(s_limit - first, 0)) : 0;
            const int slot0 = wave_inclusive_sum(n_out) - n_out;
            const int n_slots = read_lane(slot0 + n_out, kWave - 1);
            if (has) {
                z.e_pos[lane] = s_start + first;
                z.e_slot[lane] = slot0;
                z.e_ray[lane] = s_ray;
                int k = 0;
#pragma unroll
                for (int u = 0; u < kConeBatch; ++u) {
                    if (((hits >> u) & 1u) != 0u && k < n_out) {
                        z.t0[slot0 + k] = tb[u];
                        z.entry[slot0 + k] = static_cast<uint8_t>(lane);
                        ++k;
                    }
                }
            }
            wave_lds_sync();
            for (int k = lane; k < n_slots; k += kWave) {
                const int e = z.entry[k];
                const float t0 = z.t0[k];
                const int64_t pos = z.e_pos[e] + (k - z.e_slot[e]);
                if (pos >= 0 && pos < capacity) {
                    t_starts[pos] = t0;
                    t_ends[pos] = t0 + __builtin_amdgcn_fmed3f(t0 * p.cone, p.dt, p.dt_max);
                    ray_indices[pos] = z.e_ray[e];
                } else {
                    overflow = true;
                }
            }
            wave_lds_sync();  // the queue and the slots are written again next round
        }
    }
    if (t_end < INFINITY) {
        // look the rest of the ray up again (rays of more than n_masks
        // chunks of candidates, rare)
        int idx = static_cast<int>(stored & ~kOwnLattice);
        const float t_far = t_far_in[ray];
        float t = t_end;
        if (idx < limit) {
            float o[3], d[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                o[c] = rays_o[3 * ray + c];
                d[c] = rays_d[3 * ray + c];
            }
            uint32_t word0;
            grid_of_ray<LOOKUP>(grid_id, ray, g, word0);
            SkipRay sk{};
            float skip_end = -INFINITY;
            for (int k0 = n_masks * kWave; k0 < kMaxCandidates && idx < limit; k0 += kConeBatch) {
                float tb[kConeBatch + 1];
                const int n_valid = cone_steps(t, t_far, p, tb);
                const uint32_t hits =
                    cone_hits<LOOKUP, false>(bits, nullptr, g, sk, skip_end, word0, o, d, tb, n_valid) &
                    ((1u << n_valid) - 1u);
#pragma unroll
                for (int u = 0; u < kConeBatch; ++u) {
                    if (((hits >> u) & 1u) != 0u && idx < limit) {
                        const int64_t pos = start + idx;
                        if (pos >= 0 && pos < capacity) {
                            t_starts[pos] = tb[u];
                            t_ends[pos] = tb[u + 1];
                            ray_indices[pos] = static_cast<int32_t>(ray);
                        } else {
                            overflow = true;
                        }
                        ++idx;
                    }
                }
                if (n_valid < kConeBatch) break;
                t = tb[kConeBatch];
            }
        }
    }
    if (overflow && status != nullptr) *status = NACC_ECAPACITY;
    __syncthreads();
    if (simple) end_list(out, lds.list, times, first, pos0, list);
}

template <int LOOKUP, bool SKIP>
__global__ __launch_bounds__(kRaysPerBlock) void fill_cone_kernel(
    const float* __restrict__ rays_o, const float* __restrict__ rays_d,
    const int32_t* __restrict__ grid_id, int64_t n_rays, const uint32_t* __restrict__ bits,
    const uint8_t* __restrict__ skip, GridK g, ClipK c, StepK p, const int32_t* __restrict__ packed_info,
    int64_t capacity, float* __restrict__ t_starts, float* __restrict__ t_ends, int32_t* __restrict__ status) {
    const int64_t r = static_cast<int64_t>(blockIdx.x) * kRaysPerBlock + threadIdx.x;
    if (r >= n_rays) return;
    const int limit = packed_info[2 * r + 1];
    if (limit == 0) return;
    bool overflow = false;
    // the ray indices are written by expand_rays_kernel, contiguously
    fill_ray_cone<LOOKUP, SKIP>(r, rays_o, rays_d, grid_id, bits, skip, g, c, p, packed_info[2 * r], limit, capacity,
                                t_starts, t_ends, overflow);
    if (overflow && status != nullptr) *status = NACC_ECAPACITY;
}

// ray_indices[start_r + i] = r for i < count_r: one wave per ray at a time,
// 64 consecutive slots per store (the lane-per-ray fill would scatter them).
constexpr int kExpandThreads = 256;

__global__ __launch_bounds__(kExpandThreads) void expand_rays_kernel(const int32_t* __restrict__ packed_info,
                                                                     int64_t n_rays, int64_t capacity,
                                                                     int32_t* __restrict__ ray_indices) {
    const int lane = lane_id();
    const int64_t waves = static_cast<int64_t>(gridDim.x) * (kExpandThreads / kWave);
    for (int64_t r = static_cast<int64_t>(blockIdx.x) * (kExpandThreads / kWave) + threadIdx.x / kWave; r < n_rays;
         r += waves) {
        const int64_t start = packed_info[2 * r];
        const int count = packed_info[2 * r + 1];
        for (int i = lane; i < count; i += kWave) {
            const int64_t pos = start + i;
            if (pos >= 0 && pos < capacity) ray_indices[pos] = static_cast<int32_t>(r);
        }
    }
}

__global__ void set_status_kernel(int32_t* status, int32_t value) { *status = value; }

// --------------------------------------------------------------------------
// Host side: validation and launch.
// --------------------------------------------------------------------------


// Longest [t_near, t_far) a ray can have: far - near, and (unless the
// lookup contracts space, which has no clip box) the clip box's diagonal.
double clip_span(const nacc_grid_desc& grid, const nacc_march_params& p) {
    double span = static_cast<double>(p.far_plane) - static_cast<double>(p.near_plane);
    if (grid.lookup != NACC_LOOKUP_CONTRACT) {
        const double scale = grid.lookup == NACC_LOOKUP_CASCADE ? std::ldexp(1.0, grid.n_grids - 1) : 1.0;
        double d2 = 0.0;
        for (int i = 0; i < 3; ++i) {
            const double e = (static_cast<double>(grid.hi[i]) - static_cast<double>(grid.lo[i])) * scale;
            d2 += e * e;
        }
        span = std::min(span, std::sqrt(d2));
    }
    return span;
}

// Upper bound of the lattice candidates of one ray (at most kMaxCandidates).
// Cone steps never shrink as t grows, so a ray entering later than the near
// plane covers its (at most span long) range in no more steps than the
// recurrence started at the near plane; two extra candidates absorb the
// rounding of the sums.
// Bounds of `limit` or more are returned as `limit`.
int64_t candidate_bound(const nacc_grid_desc& grid, const nacc_march_params& p, int64_t limit = kMaxCandidates) {
    const double span = clip_span(grid, p);
    if (!(span > 0.0)) return 0;
    if (!std::isfinite(span)) return limit;
    if (p.cone == 0.0f) {
        return std::min<int64_t>(limit, static_cast<int64_t>(std::ceil(span / p.dt)) + 2);
    }
    float t = p.near_plane;
    const int64_t k = cone_steps(p.cone, p.dt, p.dt_max, static_cast<double>(p.near_plane) + span, limit, t);
    return k < 0 ? limit : std::min<int64_t>(limit, k + 2);
}

// Workgroups per group of kRaysPerBlock rays in the uniform-step count
// kernel: batches that make fewer than 16,384 waves (two for every place on
// the chip) are spread over more workgroups, so that each wave walks fewer
// rays one after the other; results do not depend on it.  1,021 rays in 256
// waves 15 us, in 1,021 waves 6.7 us; a call for 16,384 rays 92 us with
// 1,024 waves, 69 us with 8,192; for 65,536 rays 114 and 109 us with 4,096
// and 16,384, no gain from more.
constexpr int64_t kCountWaves = 16384;

int march_split(int64_t groups, int waves) {
    int split = 1;
    while (split * waves < kRaysPerBlock && split < 16 && groups * split * waves < kCountWaves &&
           2 * split * groups <= kMaxParts) {
        split *= 2;
    }
    return split;
}

// Rays per workgroup of the counts by segments: 64, or 32 where their masks
// would leave too few workgroups to a CU (contraction, 600,000 rays of 40
// chunks: 611 us a call with 64, 584 with 32; 15 chunks, 262,144 rays: the
// count 130 us with 64, 137 with 32, 160 with 16), and fewer for small
// batches, so that every CU has eight workgroups.
int segment_rays(int64_t n_rays, int n_masks) {
    int rays = n_masks > 24 ? 32 : kSegmentRaysMax;
    while (rays > kTaskWaves && n_rays < static_cast<int64_t>(rays) * 2048) rays /= 2;
    return rays;
}

// Workspace of the marching calls: the per-workgroup sums of the scan, then
// n_masks 64-bit occupancy masks per ray, one per chunk of 64 candidates,
// written by the count pass and replayed by the fill pass.  n_masks covers
// the longest possible ray (up to kMaxMaskChunks chunks).
// Cone steps add, for the chunk-parallel passes: t at the start of every
// chunk (chunk-major, +inf past the ray's candidates), each ray's t_far
// (-inf: no samples) and its hits past the stored chunks.
struct Layout {
    int64_t sums_bytes;
    int n_masks;
    int64_t chunk_t_off, t_far_off, extra_off;  // cone steps only (0 otherwise)
    int64_t stored_off, seg_t_off;              // cone steps, segment passes
    int64_t holding_off;                        // cone steps, segment passes: chunks holding samples
    int64_t halo_off, holes_off;                // halo and hole bits built by the count pass (0: none)
    int64_t bytes;
};

int64_t align256(int64_t b) { return ((b + 255) / 256) * 256; }

// Whether a count pass without a skip buffer builds halo bits of its own
// (halo.h, 4.5 us up to a few 128^3 grids, 23 us for 64 of them) in the
// workspace, so as to look up only the candidates near occupied cells.
// Uniform steps gain from about 16,384 rays on (128^3, a ball: 109 -> 68 us a
// call at 32,768 rays, 478 -> 262 us at 262,144; even at 16,384; 2% of the
// cells at random: 105 -> 87 and 331 -> 321 us; 262,144 rays in 64 grids of
// blobs 502 -> 305 us, of 0.4% random cells 355 -> 313 us).  The one loss known
// is that of 64 grids of 2% random cells, whose halo bits are nearly all set:
// 400 -> 427 us, the 23 us of building them.  Cone steps
// gain from the smallest batches on (they also lose a separate expansion of
// the ray indices; cascades 94 -> 55 us at 256 rays, 434 -> 175 us at
// 262,144; contraction 135 -> 63 and 1,281 -> 258 us) unless a few rays are
// spread over many grids.
bool builds_halo(int64_t n_rays, int n_masks, const nacc_grid_desc& grid, const nacc_march_params& p) {
    if (n_masks == 0) return false;
    const int64_t words = halo_words(grid.res) * grid.n_grids;
    if (p.cone > 0.0f) return words <= 65536 + 16 * n_rays;
    return grid.lookup == NACC_LOOKUP_AABB && n_rays >= 16384 + words / 4;
}

// Whether uniform steps through the box build hole bits, with a skip buffer
// too: 5 us for a 128^3 grid.  They shorten the count where there are solid
// parts (small blobs, 262,144 rays: 162 -> 138 us) and lengthen it where there
// are none (a thin shell in each of 64 grids, 262,144 rays: 178 us a call
// without them, 251 with).
bool builds_holes(int64_t n_rays, int n_masks, const nacc_grid_desc& grid, const nacc_march_params& p) {
    return n_masks > 0 && p.cone == 0.0f && grid.lookup == NACC_LOOKUP_AABB &&
           n_rays >= 16384 + 2 * halo_words(grid.res) * grid.n_grids;
}

Layout workspace_layout(int64_t n_rays, const nacc_grid_desc& grid, const nacc_march_params& p) {
    Layout l;
    // the workgroup sums, then the scan's scratch
    const int64_t nb = num_blocks(n_rays);
    l.n_masks = 0;
    if (p.dt > 0.0f) {
        const int64_t k = candidate_bound(grid, p, int64_t{kMaxMaskChunks} * kWave);
        l.n_masks = static_cast<int>((k + kWave - 1) / kWave);
    }
    const int64_t split = std::max<int64_t>(kRaysPerBlock / segment_rays(n_rays, l.n_masks), march_split(nb, 1));
    l.sums_bytes = align256((nb * split + scan_scratch_values(nb * split)) * static_cast<int64_t>(sizeof(int64_t)));
    l.bytes = l.sums_bytes + align256(n_rays * l.n_masks * static_cast<int64_t>(sizeof(uint64_t)));
    l.chunk_t_off = l.t_far_off = l.extra_off = l.stored_off = l.seg_t_off = 0;
    l.holding_off = 0;
    if (p.cone > 0.0f) {
        l.chunk_t_off = l.bytes;
        l.t_far_off = l.chunk_t_off + align256(n_rays * l.n_masks * static_cast<int64_t>(sizeof(float)));
        l.extra_off = l.t_far_off + align256(n_rays * static_cast<int64_t>(sizeof(float)));
        l.stored_off = l.extra_off + align256(n_rays * static_cast<int64_t>(sizeof(int32_t)));
        l.seg_t_off = l.stored_off + align256(n_rays * static_cast<int64_t>(sizeof(uint32_t)));
        l.holding_off =
            l.seg_t_off + align256(n_rays * l.n_masks * kSegsPerChunk * static_cast<int64_t>(sizeof(float)));
        l.bytes = l.holding_off + align256(n_rays * static_cast<int64_t>(sizeof(uint64_t)));
    }
    l.halo_off = l.holes_off = 0;
    if (builds_halo(n_rays, l.n_masks, grid, p)) {
        l.halo_off = l.bytes;
        l.bytes += align256(halo_words(grid.res) * 4 * grid.n_grids);
    }
    if (builds_holes(n_rays, l.n_masks, grid, p)) {
        l.holes_off = l.bytes;
        l.bytes += align256(halo_words(grid.res) * 4 * grid.n_grids);
    }
    return l;
}

struct ConeWork {
    uint64_t* masks;      // [n_masks][n_rays]
    float* chunk_t;       // [n_masks][n_rays]
    float* t_far;         // [n_rays]
    int32_t* extra;       // [n_rays]
    uint32_t* ray_stored;  // [n_rays]: samples in the stored chunks, and kOwnLattice
    float* seg_t;         // [n_masks][n_rays][kSegsPerChunk]: t at the start of segments holding
                          // samples, for rays not on the table
    uint64_t* sample_chunks;  // [n_rays]: bits of the chunks holding samples
    int n_masks;
};

ConeWork cone_work(void* workspace, const Layout& l) {
    char* b = static_cast<char*>(workspace);
    ConeWork w;
    w.masks = reinterpret_cast<uint64_t*>(b + l.sums_bytes);
    w.chunk_t = reinterpret_cast<float*>(b + l.chunk_t_off);
    w.t_far = reinterpret_cast<float*>(b + l.t_far_off);
    w.extra = reinterpret_cast<int32_t*>(b + l.extra_off);
    w.ray_stored = reinterpret_cast<uint32_t*>(b + l.stored_off);
    w.seg_t = reinterpret_cast<float*>(b + l.seg_t_off);
    w.sample_chunks = reinterpret_cast<uint64_t*>(b + l.holding_off);
    w.n_masks = l.n_masks;
    return w;
}

// Halo bits of a skip buffer (see halo_offset).
const uint32_t* halo_of(const uint8_t* skip, const GridK& g) {
    return skip == nullptr ? nullptr
                           : reinterpret_cast<const uint32_t*>(skip + halo_offset(g.res, g.n_grids));
}

template <int LOOKUP, bool SKIP, int WAVES>
void launch_count_uniform(const uint8_t* skip, int64_t nb, hipStream_t s, const float* o,
                          const float* d, const int32_t* gid, int64_t n, const uint32_t* bits, const GridK& g,
                          const ClipK& c, const StepK& p, int32_t* packed, int64_t* sums, uint64_t* masks,
                          int n_masks) {
    const int split = march_split(nb, WAVES);
    hipLaunchKernelGGL((count_uniform_kernel<LOOKUP, SKIP, WAVES>), dim3(static_cast<unsigned>(nb * split)),
                       dim3(WAVES * kWave), 0, s, o, d, gid, n, bits, skip, g, c, p, packed, sums, masks,
                       n_masks, split);
}

// Rays per wave of the uniform fill: as many as its LDS holds (longer lists,
// fewer stores that are not whole blocks), fewer for small batches, so that
// every SIMD has two waves.
int fill_rays(int64_t n, int n_masks) {
    int per = kFillRaysMax;
    while (per > 1 && (per * n_masks > kFillGroups * kWave || n < static_cast<int64_t>(per) * 2048)) per /= 2;
    return per;
}

template <int LOOKUP, bool SKIP>
void launch_fill_uniform(const uint8_t* skip, int64_t nb, hipStream_t s, const float* o, const float* d,
                         const int32_t* gid, int64_t n, const uint32_t* bits, const GridK& g, const ClipK& c,
                         const StepK& p, const int32_t* packed, int64_t capacity, int32_t* ri, float* ts, float* te,
                         int32_t* status, const uint64_t* masks, int n_masks) {
    const int per = fill_rays(n, n_masks);
    const int64_t rays = static_cast<int64_t>(per) * kFillWaves;
    hipLaunchKernelGGL((fill_uniform_kernel<LOOKUP, SKIP>), grid_rows((n + rays - 1) / rays, kFillThreads),
                       dim3(kFillThreads), 0, s, o, d, gid, n, bits, skip, g, c, p, packed, capacity, ri, ts, te,
                       status, masks, n_masks, per);
}

unsigned task_blocks(int n_masks, int64_t n_rays) {
    return static_cast<unsigned>((static_cast<int64_t>(n_masks) * n_rays + kTaskThreads - 1) / kTaskThreads);
}

template <int LOOKUP>
void launch_count_cone(const ConeWork& cw, const uint8_t* skip, const uint32_t* halo, int64_t nb, hipStream_t s,
                       const float* o, const float* d, const int32_t* gid, int64_t n, const uint32_t* bits,
                       const GridK& g, const ClipK& c, const StepK& p, int32_t* packed, int64_t* sums, uint64_t*,
                       int) {
    const ConeTable tab = cone_table(p, cw.n_masks);
    if (halo != nullptr) {
        const int rays = segment_rays(n, cw.n_masks);
        const bool walks = LOOKUP != NACC_LOOKUP_CONTRACT || tab.n == 0;
        hipLaunchKernelGGL((count_cone_kernel<LOOKUP>), dim3(static_cast<unsigned>((n + rays - 1) / rays)),
                           dim3(kTaskThreads), cone_lds(rays, cw.n_masks, walks, LOOKUP == NACC_LOOKUP_CONTRACT).bytes, s, o, d, gid, n, bits, halo,
                           skip, g, c, p, cw.n_masks, rays, walks ? 1 : 0, packed, sums, cw.masks, cw.ray_stored,
                           cw.seg_t, cw.chunk_t, cw.t_far, cw.sample_chunks, tab);
        return;
    }
    hipLaunchKernelGGL(cone_starts_kernel, dim3(nb), dim3(kRaysPerBlock), 0, s, o, d, gid, n,
                       gid != nullptr && LOOKUP != NACC_LOOKUP_CASCADE, g, c, p, cw.n_masks, cw.chunk_t, cw.t_far,
                       cw.extra, tab);
    if (cw.n_masks > 0) {
        hipLaunchKernelGGL((count_cone_chunks_kernel<LOOKUP>), dim3(task_blocks(cw.n_masks, n)), dim3(kTaskThreads), 0,
                           s, o, d, gid, n, bits, g, p, cw.n_masks, cw.chunk_t, cw.t_far, cw.masks, cw.extra);
    }
    hipLaunchKernelGGL(cone_counts_kernel, dim3(nb), dim3(kRaysPerBlock), 0, s, n, cw.n_masks, p.max_per_ray, cw.masks,
                       cw.extra, packed, sums);
}

void launch_count_box(const uint32_t* halo, const uint32_t* holes, int64_t, hipStream_t s, const float* o,
                      const float* d, const int32_t* gid, int64_t n, const uint32_t* bits, const GridK& g,
                      const ClipK& c, const StepK& p, int32_t* packed, int64_t* sums, uint64_t* masks, int n_masks) {
    const int rays = segment_rays(n, n_masks);
    const bool cap = p.max_per_ray > 0, spread = g.n_grids > 1;
    hipLaunchKernelGGL(cap ? (spread ? count_box_kernel<true, true> : count_box_kernel<true, false>)
                           : (spread ? count_box_kernel<false, true> : count_box_kernel<false, false>),
                       grid_rows((n + rays - 1) / rays, kTaskThreads), dim3(kTaskThreads), box_lds(rays, n_masks),
                       s, o, d, gid, n, bits, halo, holes, g, c, p, n_masks, rays, packed, sums, masks);
}

template <int LOOKUP, bool SKIP, typename... A>
void launch_count_waves(A&&... a) {
    switch (tuning().march_waves_per_group) {
        case 1: launch_count_uniform<LOOKUP, SKIP, 1>(a...); break;
        case 2: launch_count_uniform<LOOKUP, SKIP, 2>(a...); break;
        case 8: launch_count_uniform<LOOKUP, SKIP, 8>(a...); break;
        case 16: launch_count_uniform<LOOKUP, SKIP, 16>(a...); break;
        default: launch_count_uniform<LOOKUP, SKIP, 4>(a...); break;
    }
}

// Rays per wave of the cone fill, fewer for small batches, so that every SIMD
// has two waves.
int cone_fill_rays(int64_t n) {
    int per = kFillRays;
    while (per > 1 && n < static_cast<int64_t>(per) * 2048) per /= 2;
    return per;
}

template <int LOOKUP, bool SKIP>
void launch_fill_cone(const uint8_t* skip, bool segments, const ConeWork* cw, int64_t nb, hipStream_t s,
                      const float* o, const float* d, const int32_t* gid, int64_t n, const uint32_t* bits,
                      const GridK& g, const ClipK& c, const StepK& p, const int32_t* packed, int64_t capacity,
                      int32_t* ri, float* ts, float* te, int32_t* status, const uint64_t*, int) {
    if (cw != nullptr && cw->n_masks > 0 && segments) {
        // the segment count's masks, segment starts and chunks holding
        // samples, ray-major (the ray indices written with the samples)
        const int per = cone_fill_rays(n);
        const int64_t per_block = static_cast<int64_t>(kTaskWaves) * per;
        const unsigned blocks = static_cast<unsigned>((n + per_block - 1) / per_block);
        hipLaunchKernelGGL((fill_cone_rays_kernel<LOOKUP>), dim3(blocks), dim3(kTaskThreads),
                           cone_fill_lds(cw->n_masks), s, o, d, gid, n, bits, g, p, cw->n_masks, per, cw->chunk_t,
                           cw->t_far, cw->masks, cw->ray_stored, cw->seg_t, cw->sample_chunks, packed, capacity, ri, ts,
                           te, status, cone_table(p, cw->n_masks));
        return;
    }
    if (cw != nullptr && cw->n_masks > 0) {  // replay the count pass's chunks, one lane per chunk
        hipLaunchKernelGGL((fill_cone_chunks_kernel<LOOKUP>), dim3(task_blocks(cw->n_masks, n)), dim3(kTaskThreads), 0,
                           s, o, d, gid, n, bits, g, p, cw->n_masks, cw->chunk_t, cw->t_far, cw->masks, packed,
                           capacity, ts, te, status);
    } else {  // traversal, one lane per ray
        hipLaunchKernelGGL((fill_cone_kernel<LOOKUP, SKIP>), dim3(nb), dim3(kRaysPerBlock), 0, s, o, d, gid, n, bits,
                           skip, g, c, p, packed, capacity, ts, te, status);
    }
    const int64_t blocks = std::min<int64_t>((n + kExpandThreads / kWave - 1) / (kExpandThreads / kWave), 256 * 64);
    hipLaunchKernelGGL(expand_rays_kernel, dim3(static_cast<unsigned>(blocks)), dim3(kExpandThreads), 0, s, packed, n,
                       capacity, ri);
}

template <int LOOKUP>
using Lookup = std::integral_constant<int, LOOKUP>;

// `halo`: the halo bits the call marches by (the skip buffer's, or built in
// the workspace), or nullptr.  The box lookup's uniform steps and every
// lookup's cone steps use them; the skip buffer's distances serve the
// uniform steps of the other lookups.
template <int LOOKUP, typename... A>
void dispatch_count(const uint8_t* skip, const uint32_t* halo, const uint32_t* holes, const ConeWork* cw, A&&... a) {
    if (cw != nullptr) {
        launch_count_cone<LOOKUP>(*cw, skip, halo, a...);
    } else if (LOOKUP == NACC_LOOKUP_AABB && halo != nullptr) {
        launch_count_box(halo, holes, a...);
    } else if (LOOKUP != NACC_LOOKUP_AABB && skip != nullptr) {
        launch_count_waves<LOOKUP, true>(skip, a...);
    } else {
        launch_count_waves<LOOKUP, false>(nullptr, a...);
    }
}

// `segments` (cone steps): the count pass marched by halo bits.
template <int LOOKUP, typename... A>
void dispatch_fill(const uint8_t* skip, bool cone, bool segments, const ConeWork* cw, A&&... a) {
    if (cone && skip != nullptr) {
        launch_fill_cone<LOOKUP, true>(skip, segments, cw, a...);
    } else if (cone) {
        launch_fill_cone<LOOKUP, false>(nullptr, segments, cw, a...);
    } else if (LOOKUP != NACC_LOOKUP_AABB && skip != nullptr) {
        launch_fill_uniform<LOOKUP, true>(skip, a...);
    } else {
        launch_fill_uniform<LOOKUP, false>(nullptr, a...);
    }
}

const uint8_t* usable_skip(const uint8_t* skip, const nacc_grid_desc& grid) {
    if (skip == nullptr || grid.res % 4 != 0) return nullptr;
    return skip;
}

// Count, scan and starts of one marching call, given the scan sums and (for
// uniform steps, nullable) the chunk masks or (cone steps) the cone
// workspace.
int march_count_launch(const float* rays_o, const float* rays_d, const int32_t* grid_id, int64_t n_rays,
                       const uint32_t* grid_bits, const uint8_t* grid_skip, const nacc_grid_desc* grid,
                       const nacc_march_params* params, int32_t* packed_info, int64_t* total, int64_t* sums,
                       uint64_t* masks, int n_masks, const ConeWork* cw, uint32_t* own_halo, uint32_t* own_holes,
                       hipStream_t s) {
    GridK g;
    ClipK c;
    StepK p;
    make_constants(*grid, *params, g, c, p);
    const int64_t nb = num_blocks(n_rays);
    const uint8_t* skip = usable_skip(grid_skip, *grid);
    int st = NACC_OK;
    bool by_segments = false;
    if (nb > 0) {
        const uint32_t* halo = halo_of(skip, g);
        const bool own = halo == nullptr && own_halo != nullptr;
        if (own || own_holes != nullptr) {
            launch_halo(grid_bits, g.res, g.n_grids, own ? own_halo : nullptr, own_holes, s);
            st = check_launch("march halo");
            if (st != NACC_OK) return st;
            if (own) halo = own_halo;
        }
        if (n_masks == 0) halo = nullptr;  // no candidates: nothing to look up
        by_segments = halo != nullptr && (cw != nullptr || grid->lookup == NACC_LOOKUP_AABB);
        auto run = [&](auto lookup) {
            dispatch_count<decltype(lookup)::value>(skip, halo, own_holes, cw, nb, s, rays_o, rays_d, grid_id, n_rays, grid_bits,
                                                    g, c, p, packed_info, sums, masks, n_masks);
        };
        switch (grid->lookup) {
            case NACC_LOOKUP_AABB: run(Lookup<NACC_LOOKUP_AABB>{}); break;
            case NACC_LOOKUP_CASCADE: run(Lookup<NACC_LOOKUP_CASCADE>{}); break;
            default: run(Lookup<NACC_LOOKUP_CONTRACT>{}); break;
        }
        st = check_launch("march count");
        if (st != NACC_OK) return st;
    }
    if (nb == 0) {
        scan_exclusive(sums, 0, total, nullptr, s);
        return check_launch("march scan");
    }
    // rays of a sum
    const int part_rays = by_segments     ? segment_rays(n_rays, n_masks)
                          : cw != nullptr ? kRaysPerBlock
                                          : kRaysPerBlock / march_split(nb, tuning().march_waves_per_group);
    launch_starts(sums, (n_rays + part_rays - 1) / part_rays, __builtin_ctz(static_cast<unsigned>(part_rays)), n_rays,
                  packed_info, total, s);
    return check_launch("march starts");
}

}  // namespace

bool nacc::march_follows_waves(int64_t n_rays, const nacc_grid_desc& grid, const nacc_march_params& params,
                               bool has_skip) {
    if (params.cone > 0.0f) return false;
    const Layout l = workspace_layout(n_rays, grid, params);
    return grid.lookup != NACC_LOOKUP_AABB || l.n_masks == 0 || !(has_skip || l.halo_off != 0);
}

extern "C" {

int64_t nacc_march_workspace_size(int64_t n_rays, const nacc_grid_desc* grid, const nacc_march_params* params) {
    clear_error();
    if (n_rays < 0 || grid == nullptr || params == nullptr) return -1;
    if (validate(nullptr, nullptr, 0, nullptr, grid, params) != NACC_OK) return -1;
    return workspace_layout(n_rays, *grid, *params).bytes;
}

int64_t nacc_march_max_samples_per_ray(const nacc_grid_desc* grid, const nacc_march_params* params) {
    clear_error();
    if (grid == nullptr || params == nullptr) {
        set_error(NACC_EINVAL, "grid and params must be non-NULL");
        return -1;
    }
    const nacc_march_params& p = *params;
    if (!(std::isfinite(p.dt) && p.dt > 0.0f) || !(p.cone >= 0.0f) || std::isnan(p.near_plane) ||
        std::isnan(p.far_plane)) {
        set_error(NACC_EINVAL, "invalid marching parameters");
        return -1;
    }
    int64_t bound = candidate_bound(*grid, p);
    if (p.max_per_ray > 0) bound = std::min<int64_t>(bound, p.max_per_ray);
    return bound;
}

int nacc_march_count(const float* rays_o, const float* rays_d, const int32_t* grid_id, int64_t n_rays,
                     const uint32_t* grid_bits, const uint8_t* grid_skip, const nacc_grid_desc* grid,
                     const nacc_march_params* params,
                     int32_t* packed_info, int64_t* total, void* workspace, size_t workspace_bytes,
                     void* stream) {
    clear_error();
    int st = validate(rays_o, rays_d, n_rays, grid_bits, grid, params);
    if (st != NACC_OK) return st;
    NACC_REQUIRE(total != nullptr, NACC_EINVAL, "total must be non-NULL");
    NACC_REQUIRE(n_rays == 0 || packed_info != nullptr, NACC_EINVAL, "packed_info must be non-NULL");
    const Layout lay = workspace_layout(n_rays, *grid, *params);
    const int64_t need = lay.bytes;
    NACC_REQUIRE(need == 0 || workspace != nullptr, NACC_EINVAL, "workspace must be non-NULL");
    NACC_REQUIRE(static_cast<int64_t>(workspace_bytes) >= need, NACC_ESHAPE,
                 "workspace of %zu bytes, need %lld", workspace_bytes, static_cast<long long>(need));
    uint64_t* masks = lay.n_masks > 0 ? reinterpret_cast<uint64_t*>(static_cast<char*>(workspace) + lay.sums_bytes)
                                      : nullptr;
    ConeWork cw_store{};
    const ConeWork* cw = nullptr;
    if (params->cone > 0.0f) {
        cw_store = cone_work(workspace, lay);
        cw = &cw_store;
    }
    uint32_t* own_halo =
        lay.halo_off != 0 ? reinterpret_cast<uint32_t*>(static_cast<char*>(workspace) + lay.halo_off) : nullptr;
    uint32_t* own_holes =
        lay.holes_off != 0 ? reinterpret_cast<uint32_t*>(static_cast<char*>(workspace) + lay.holes_off) : nullptr;
    return march_count_launch(rays_o, rays_d, grid_id, n_rays, grid_bits, grid_skip, grid, params, packed_info,
                              total, static_cast<int64_t*>(workspace), masks, lay.n_masks, cw, own_halo, own_holes,
                              as_stream(stream));
}

int nacc_march_fill(const float* rays_o, const float* rays_d, const int32_t* grid_id, int64_t n_rays,
                    const uint32_t* grid_bits, const uint8_t* grid_skip, const nacc_grid_desc* grid,
                    const nacc_march_params* params,
                    const int32_t* packed_info, const void* workspace, size_t workspace_bytes, int64_t capacity,
                    int32_t* ray_indices, float* t_starts, float* t_ends, int32_t* status, void* stream) {
    clear_error();
    int st = validate(rays_o, rays_d, n_rays, grid_bits, grid, params);
    if (st != NACC_OK) return st;
    NACC_REQUIRE(capacity >= 0 && capacity <= INT32_MAX, NACC_ECAPACITY,
                 "capacity = %lld out of [0, 2^31-1]", static_cast<long long>(capacity));
    NACC_REQUIRE(n_rays == 0 || packed_info != nullptr, NACC_EINVAL, "packed_info must be non-NULL");
    NACC_REQUIRE(capacity == 0 || (ray_indices != nullptr && t_starts != nullptr && t_ends != nullptr),
                 NACC_EINVAL, "sample outputs must be non-NULL");
    GridK g;
    ClipK c;
    StepK p;
    make_constants(*grid, *params, g, c, p);
    hipStream_t s = as_stream(stream);
    if (status != nullptr) {
        hipLaunchKernelGGL(set_status_kernel, dim3(1), dim3(1), 0, s, status, static_cast<int32_t>(NACC_OK));
        st = check_launch("march status");
        if (st != NACC_OK) return st;
    }
    const int64_t nb = num_blocks(n_rays);
    if (nb == 0) return NACC_OK;
    const bool cone = params->cone > 0.0f;
    const uint8_t* skip = usable_skip(grid_skip, *grid);
    const Layout lay = workspace_layout(n_rays, *grid, *params);
    NACC_REQUIRE(workspace == nullptr || static_cast<int64_t>(workspace_bytes) >= lay.bytes, NACC_ESHAPE,
                 "workspace of %zu bytes, need %lld", workspace_bytes, static_cast<long long>(lay.bytes));
    const uint64_t* masks =
        workspace != nullptr && lay.n_masks > 0
            ? reinterpret_cast<const uint64_t*>(static_cast<const char*>(workspace) + lay.sums_bytes)
            : nullptr;
    ConeWork cw_store{};
    const ConeWork* cw = nullptr;
    if (cone && workspace != nullptr) {
        cw_store = cone_work(const_cast<void*>(workspace), lay);
        cw = &cw_store;
    }
    // as the count pass decided: by the skip buffer's halo bits or its own
    const bool segments = skip != nullptr || lay.halo_off != 0;
    auto run = [&](auto lookup) {
        dispatch_fill<decltype(lookup)::value>(skip, cone, segments, cw, nb, s, rays_o, rays_d, grid_id, n_rays,
                                               grid_bits, g, c, p, packed_info, capacity, ray_indices, t_starts,
                                               t_ends, status, masks, lay.n_masks);
    };
    switch (grid->lookup) {
        case NACC_LOOKUP_AABB: run(Lookup<NACC_LOOKUP_AABB>{}); break;
        case NACC_LOOKUP_CASCADE: run(Lookup<NACC_LOOKUP_CASCADE>{}); break;
        default: run(Lookup<NACC_LOOKUP_CONTRACT>{}); break;
    }
    return check_launch("march fill");
}

}  // extern "C"
