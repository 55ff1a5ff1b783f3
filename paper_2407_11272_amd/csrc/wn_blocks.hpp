// Blocks of voxels with Chebyshev nodes: shared by the caps' far field (wn_cycle.hip) and the
// boundary edges' adjoint (wn_edge_bwd.hip).
#pragma once

#include "wn_cycle.hpp"

namespace wn {
namespace {

// Points at least this many times the longer of the edges v_0 v_1 and v_0 v_2 away from
// v_0 use a triangle's far forms: the squares' differences lose at most three bits there, of a
// triangle's share of W that is at most 0.01, and its half angle is below 0.07, where
// three terms of the arctangent are off by 1e-9.
constexpr float kFar = 2.0f;

constexpr int kBlockSide = 16, kBlockRows = 4, kCoarse = 4, kFine = 8;
constexpr int64_t kBlockPoints = 1 << 18;
constexpr int kMaxSplits = 8;
constexpr int64_t kSplitWaves = 24576;
constexpr float kFarError = 4.0e-8f, kCoarseError = 1.0e-9f;

__device__ __forceinline__ float centre(const PointSrc &ps, int d, int i) {
    return __builtin_fmaf((float)i + 0.5f, ps.h[d], ps.lo[d]);
}

// Node j of n voxels, in voxels from the first: the voxels themselves where they are few.
__device__ __forceinline__ float node_at(int order, int size, int j) {
    constexpr float kCheb4[4] = {0.92387953251128674f, 0.38268343236508977f, -0.38268343236508977f, -0.92387953251128674f};
    constexpr float kCheb8[8] = {0.98078528040323045f,  0.83146961230254524f,  0.55557023301960222f,
                                 0.19509032201612827f,  -0.19509032201612827f, -0.55557023301960222f,
                                 -0.83146961230254524f, -0.98078528040323045f};
    if (size <= order) return (float)j;
    const float x = order == kCoarse ? kCheb4[j & 3] : kCheb8[j];
    return 0.5f * (float)(size - 1) * (1.0f + x);
}

// Weight at x of the value at node j.
__device__ __forceinline__ float node_weight(int order, int size, float x, int j) {
    const double xj = node_at(order, size, j);
    double num = 1.0, den = 1.0;
    for (int k = 0; k < min(order, size); ++k) {
        const double xk = node_at(order, size, k);
        if (k != j) num *= (double)x - xk, den *= xj - xk;
    }
    return (float)(num / den);
}

// A block's box, and which triangles are far from it.
struct Block {
    float lo[3], hi[3], a, inv_a;

    __device__ __forceinline__ Block(const CycMesh &m, const int (&i0)[3]) {
        a = 0.0f;
        for (int d = 0; d < 3; ++d) {
            lo[d] = centre(m.ps, d, i0[d]);
            hi[d] = centre(m.ps, d, i0[d] + m.grid.size[d] - 1);
            a = fmaxf(a, 0.5f * (hi[d] - lo[d]));
        }
        inv_a = 1.0f / a;
    }
    // tight: a factor on the errors allowed.
    // Slot v: no triangle (0), far (1), far enough for the coarse nodes (2), or near (-1).
    // (Products and explicit multiply-adds only: both kernels come to the same answer.)
    __device__ __forceinline__ int kind(const float4 v, float tight = 1.0f) const {
        const float x = fmaxf(fmaxf(lo[0] - v.x, v.x - hi[0]), 0.0f), y = fmaxf(fmaxf(lo[1] - v.y, v.y - hi[1]), 0.0f),
                    z = fmaxf(fmaxf(lo[2] - v.z, v.z - hi[2]), 0.0f);
        const float d2 = __builtin_fmaf(z, z, __builtin_fmaf(y, y, x * x));
        const float e2 = v.w * (1.0f / (kFar * kFar));
        const float D = fast_sqrt(d2) - fast_sqrt(e2);  // v_0's distance less an edge
        const float t = D * inv_a, rho = t + fast_sqrt(__builtin_fmaf(t, t, 1.0f));
        const float r2 = rho * rho, r4 = r2 * r2, r8 = r4 * r4;
        if (!(v.w >= 0.0f)) return 0;
        if (!(d2 >= 1.01f * v.w && D > 0.0f && 0.04f * e2 <= tight * kFarError * (D * D) * r8)) return -1;
        return 0.04f * e2 <= tight * kCoarseError * (D * D) * r4 ? 2 : 1;
    }
};

template <typename Int>
__device__ __forceinline__ void block_origin(const CycMesh &m, Int b, int (&i0)[3]) {
    const int yz = m.grid.n[1] * m.grid.n[2];
    const int bx = (int)(b / yz), r = (int)(b - (Int)bx * yz), by = r / m.grid.n[2];
    i0[0] = (m.xb0 + bx) * m.grid.size[0];
    i0[1] = by * m.grid.size[1];
    i0[2] = (r - by * m.grid.n[2]) * m.grid.size[2];
}

__device__ __forceinline__ int64_t block_count(const CycMesh &m) {
    return (int64_t)(m.xb1 - m.xb0 + 1) * m.grid.n[1] * m.grid.n[2];
}

}  // namespace
}  // namespace wn
