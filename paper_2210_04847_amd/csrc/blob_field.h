// The synthetic Gaussian-blob field's device code (test and benchmark input,
// standing in for the user's radiance field), shared by the field kernels
// and the fused inference kernel, which must evaluate it bit for bit alike.
//
// The coefficient table holds, per blob, (c_x, c_y, c_z, k, peak) with
// k = -log2(e) / (2 std^2), so each blob costs one exp2 on the hardware
// transcendental unit; the 9 + 3 colour coefficients follow the blobs, then
// the flags word (1.0f: the scene is defined in contracted coordinates).
#pragma once

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

namespace nacc {
namespace blob {

constexpr int kBlobStride = 5;
constexpr float kLog2e = 1.4426950408889634f;

inline int64_t table_floats(int32_t n_blobs, int32_t n_sets) {
    return static_cast<int64_t>(n_sets) * n_blobs * kBlobStride + 13;
}

__device__ __forceinline__ float exp2_fast(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ float add_blob(const float* __restrict__ e, float x0, float x1, float x2, float acc) {
    const float dx = x0 - e[0];
    const float dy = x1 - e[1];
    const float dz = x2 - e[2];
    const float d2 = fmaf(dz, dz, fmaf(dy, dy, dx * dx));
    return fmaf(e[4], exp2_fast(d2 * e[3]), acc);
}

__device__ __forceinline__ void eval_field(const float* __restrict__ table, int n_blobs, int set, float x0, float x1,
                                           float x2, float& sigma) {
    const float* blob = table + static_cast<int64_t>(set) * n_blobs * kBlobStride;
    float acc = 0.0f;
#pragma unroll 4
    for (int b = 0; b < n_blobs; ++b) acc = add_blob(blob + kBlobStride * b, x0, x1, x2, acc);
    sigma = acc;
}

// The blobs that may contribute to a chunk of samples lying within `reach`
// of point c (both in scene coordinates, every lane the same), one bit each
// for blobs [64 i, 64 i + 64) of the set.  A blob is left out when its term
// is +0 at every such point: the exponent k d^2 of its exp2 is below -160
// there, where the hardware's result is 0, and its peak is finite, so that
// adding the product leaves the sum as it is.  `reach` carries the rounding
// of the positions; the distance to c is lowered by 2^-16 of itself for its
// own rounding, and -160 leaves 2^11 below the smallest subnormal, 2^-149.
// (32 blobs of 0.03 to 0.1 in a box of 3, 640,000 rays of one view, 64 rays a
// workgroup: 844 -> 734 us.)
__device__ __forceinline__ uint64_t near_blobs(const float* __restrict__ blob, int n_blobs, int i, float c0, float c1,
                                               float c2, float reach) {
    const int b = 64 * i + static_cast<int>(__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)));
    bool near = false;
    if (b < n_blobs) {
        const float* e = blob + static_cast<int64_t>(kBlobStride) * b;
        const float dx = c0 - e[0], dy = c1 - e[1], dz = c2 - e[2];
        const float dist = __builtin_amdgcn_sqrtf(fmaf(dz, dz, fmaf(dy, dy, dx * dx)));
        const float gap = dist * (1.0f - 0x1p-16f) - reach;
        near = !(gap > 0.0f && gap * gap * e[3] < -160.0f && fabsf(e[4]) < INFINITY);
    }
    return __builtin_amdgcn_ballot_w64(near);
}

// eval_field over the blobs near the chunk alone (see near_blobs), in the
// same order: the same bits.
__device__ __forceinline__ float eval_near(const float* __restrict__ blob, int n_blobs, float c0, float c1, float c2,
                                           float reach, float x0, float x1, float x2) {
    float acc = 0.0f;
    for (int i = 0; 64 * i < n_blobs; ++i) {
        const float* group = blob + static_cast<int64_t>(kBlobStride) * 64 * i;
        uint64_t todo = near_blobs(blob, n_blobs, i, c0, c1, c2, reach);
        // four at a time, so that their scalar loads are in flight together
        while (__builtin_popcountll(todo) >= 4) {
            const float* e[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                e[k] = group + kBlobStride * __builtin_ctzll(todo);
                todo &= todo - 1ull;
            }
#pragma unroll
            for (int k = 0; k < 4; ++k) acc = add_blob(e[k], x0, x1, x2, acc);
        }
        for (; todo != 0ull; todo &= todo - 1ull) {
            acc = add_blob(group + kBlobStride * __builtin_ctzll(todo), x0, x1, x2, acc);
        }
    }
    return acc;
}

__device__ __forceinline__ void eval_rgb(const float* __restrict__ cc, float x0, float x1, float x2, float& r,
                                         float& g, float& b) {
    const float z0 = fmaf(cc[0], x0, fmaf(cc[1], x1, fmaf(cc[2], x2, cc[9])));
    const float z1 = fmaf(cc[3], x0, fmaf(cc[4], x1, fmaf(cc[5], x2, cc[10])));
    const float z2 = fmaf(cc[6], x0, fmaf(cc[7], x1, fmaf(cc[8], x2, cc[11])));
    r = 1.0f / (1.0f + exp2_fast(-z0 * kLog2e));
    g = 1.0f / (1.0f + exp2_fast(-z1 * kLog2e));
    b = 1.0f / (1.0f + exp2_fast(-z2 * kLog2e));
}

// Sample midpoint, FP32, no fused multiply-add (matches the positions of the
// tests).
__device__ __forceinline__ float midpoint_coord(float o, float d, float t0, float t1) {
#pragma clang fp contract(off)
    const float tm = (t0 + t1) * 0.5f;
    return o + d * tm;
}

// Scene coordinates of a world point when the scene is defined in
// contracted space: beyond the unit ball, x -> (2 - 1/|x|) x / |x|.
__device__ __forceinline__ void to_scene(bool contract, float& x0, float& x1, float& x2) {
    if (!contract) return;
    const float n2 = fmaf(x2, x2, fmaf(x1, x1, x0 * x0));
    if (n2 > 1.0f) {
        const float n = sqrtf(n2);
        const float f = (2.0f - 1.0f / n) / n;
        x0 *= f;
        x1 *= f;
        x2 *= f;
    }
}

}  // namespace blob
}  // namespace nacc
