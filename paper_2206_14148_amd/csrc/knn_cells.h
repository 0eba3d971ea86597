// Cells over the points' bounding box, shared by the low-dimensional search kernels: which cell a
// coordinate falls into and between which bounds its points then lie.
#pragma once
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "knn_config.h"

namespace knn {

namespace {

// floats <-> unsigned keys with the same order (for atomicMin / atomicMax)
__device__ __forceinline__ unsigned ordered_bits(float f) {
    const unsigned u = __float_as_uint(f);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}
__device__ __forceinline__ float ordered_value(unsigned k) {
    return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

template <int D>
struct SeedGrid {
    float mn[D], inv_w[D], w[D], slack[D];
    int G;
};

template <int D>
__device__ __forceinline__ SeedGrid<D> seed_grid(const unsigned* __restrict__ hdr, int G) {
    SeedGrid<D> g;
    g.G = G;
#pragma unroll
    for (int t = 0; t < D; ++t) {
        const float mn = ordered_value(hdr[1 + t]);
        const float mx = ordered_value(hdr[1 + kPbMaxD + t]);
        float rg = mx - mn;
        if (!(rg > 1e-30f)) rg = 1.f;  // all points share this coordinate: one cell holds them
        g.mn[t] = mn;
        g.inv_w[t] = (float)G / rg;
        g.w[t] = rg / (float)G;
        // A point whose computed cell number is c lies in mn + [c w, (c + 1) w] up to the
        // roundings of (x - mn) * inv_w, of w and of the two ends: under 16 ulps of the
        // magnitudes involved; the slack is twice that.
        g.slack[t] = 0x1p-19f * (fabsf(mn) + fabsf(mx) + rg);
    }
    return g;
}

// cell number along axis t, the same expression for points and queries (queries outside the
// box land in the nearest cell)
template <int D>
__device__ __forceinline__ int seed_cell(const SeedGrid<D>& g, int t, float x) {
    const float u = (x - g.mn[t]) * g.inv_w[t];
    return (int)fminf(fmaxf(u, 0.f), (float)(g.G - 1));  // NaN -> 0
}

}  // namespace

}  // namespace knn
