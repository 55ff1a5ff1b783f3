// Adjoint for dL/dV from the mesh's boundary edges.
//
// The solid angle of a face depends on its edges alone: moving a vertex changes it by
// line integrals along the face's edges (the Biot-Savart form of dOmega), and the two
// faces at an inner edge run along it in opposite directions.  So in
//     dL/dV = sum over faces of dL/dT
// the inner edges cancel, and what is left is the sum over the boundary edges of
// wn_cycle.hip: for an edge from u to v, with A = u - q, B = v - q, E = v - u,
//     dW/du = -(A x E) / (4 pi |A| (|A| |B| + A . B)),
//     dW/dv = -(A x E) / (4 pi |B| (|A| |B| + A . B)).
// A closed mesh has no such edge and no gradient (Section 2.4 of arXiv 2407.11272 notes
// that it vanishes).
//
// One lane owns an edge and keeps six sums, sum(g J P) for either end: A x E = P x E with P the
// part of A at right angles to E and J the rest, so the cross product waits until the sums are complete.  Points come
// through LDS, 256 to a tile, tiles dealt to S splits in turn, as in the all-pairs adjoint (the same
// calls on point ranges give the same bits as one call).
//
// The all-pairs adjoint is bound by its arithmetic over all faces; here it is 40 VALU instructions and 3
// transcendentals per (edge, point), issued at 1.1 VALU per CU and clock in the point kernel and 0.73 over blocks
// (the all-pairs kernels: 1.5): few waves and idle lanes are the rest.  Measured, whole
// adjoint: 7706 faces with 1154 boundary edges on 96 x 88 x 97 points, 10.0 -> 1.08 ms point by point,
// 0.72 ms with nodes (k_edge_blocks); 9140 faces, 2.6 % of them missing, on 43 x 32 x 17 points, 519 -> 118 us.  The error
// against 64 bits falls too (1.3e-6 -> 1e-7 in the first): fewer terms, and none that cancel.
#include <algorithm>

#include "wn_blocks.hpp"

namespace wn {

namespace {

constexpr int kEdgeWaves = 16384;  // one-wave workgroups of the point kernel
constexpr int kTile = kBwdTile;
constexpr int64_t kEdgeBlockPoints = 1 << 19;  // 64^3: 208 us with and without the nodes, too few blocks

// Splits of B edges over the tiles of the points, a pure function of the sizes: about
// kEdgeWaves waves of (64 edges, split), all with the same number of tiles.
__device__ __forceinline__ int edge_splits(int B, int tiles) {
    const int64_t blocks = B > 64 ? (B + 63) / 64 : 1;
    const int per = max((int)((tiles * blocks + kEdgeWaves - 1) / kEdgeWaves), (tiles + 4095) / 4096);
    return max(1, (tiles + per - 1) / max(1, per));
}

// A boundary edge from u to v, and its sums over points, in units of about its length: lengths
// are multiplied by `s`, a power of two that brings |E| to [1, 2).  A coordinate times s is exact, so
// u - q in these units is one multiply-add, and no product depends on the mesh's scale.  (An edge
// shorter than 2^-30 of the distances to the points is taken in units of that, or the squares of
// the distances would leave FP32's range.)
struct Edge {
    float s, u[3], v[3], E[3], f[3], l, L2;  // f = E / |E|^2, l = |E|; L2 = |E|^2 in the mesh's units

    __device__ __forceinline__ Edge(const CycMesh &m, const int2 id) {
        const float *pu = m.V + 3 * (int64_t)id.x, *pv = m.V + 3 * (int64_t)id.y;
        double x[3], l2 = 0.0, far = 0.0;
        const int n[3] = {m.n0, m.ps.n1, m.ps.n2};
        for (int d = 0; d < 3; ++d) {
            x[d] = (double)pv[d] - pu[d];
            l2 += x[d] * x[d];
            const double a = (double)m.ps.lo[d] - pu[d];
            far += fmax(fabs(a), fabs(a + (double)n[d] * m.ps.h[d]));
        }
        const double len = sqrt(l2);
        s = (float)ldexp(1.0, -min(max(ilogb(fmax(len, 0x1p-30 * far)), -100), 100));
        for (int d = 0; d < 3; ++d) {
            u[d] = s * pu[d];
            v[d] = s * pv[d];
            E[d] = (float)(x[d] * s);
            f[d] = l2 > 0.0 ? (float)(x[d] / (l2 * s)) : 0.0f;
        }
        l = (float)(len * s);
        L2 = (float)l2;
    }
    // Its start in the mesh's units, and the square of the distance from which it may be far (wn_blocks.hpp).
    __device__ __forceinline__ float4 start() const {
        const float x = 1.0f / s;
        return make_float4(x * u[0], x * u[1], x * u[2], kFar * kFar * L2);
    }
    // What a point adds: k J P for either end (ku, kv the factors of P).
    struct Term {
        float p[3], ku, kv;
    };
    // A point close to either end or to the edge's line.  |B| and P are formed from the nearer end,
    // as they vanish with the distance to it.  The term is left out where the point is a vertex, or is on
    // the edge up to the rounding of P (at most 4 x 2^-24 of the distance to the end that it is formed from:
    // R, E and P are rounded; what a rounds to is along E).
    __device__ __forceinline__ Term near_term(const float4 q) const {
        float a[3], b[3];
        for (int d = 0; d < 3; ++d) {
            const float x = d == 0 ? q.x : d == 1 ? q.y : q.z;
            a[d] = __builtin_fmaf(-x, s, u[d]);
            b[d] = __builtin_fmaf(-x, s, v[d]);
        }
        const bool from_v = dot3(b[0], b[1], b[2], b[0], b[1], b[2]) < dot3(a[0], a[1], a[2], a[0], a[1], a[2]);
        Term t;
        for (int d = 0; d < 3; ++d) a[d] = from_v ? b[d] : a[d];
        const float x = dot3(a[0], a[1], a[2], f[0], f[1], f[2]);
        for (int d = 0; d < 3; ++d) t.p[d] = __builtin_fmaf(-x, E[d], a[d]);
        const float d2 = dot3(t.p[0], t.p[1], t.p[2], t.p[0], t.p[1], t.p[2]);
        const float ul = from_v ? x * l - l : x * l, vl = from_v ? x * l : x * l + l;
        const float A2 = __builtin_fmaf(ul, ul, d2), B2 = __builtin_fmaf(vl, vl, d2), AB = __builtin_fmaf(ul, vl, d2);
        const float ia = __builtin_amdgcn_rsqf(A2), ib = __builtin_amdgcn_rsqf(B2);
        const float mn = (A2 * ia) * (B2 * ib) + __builtin_fabsf(AB);
        const bool between = AB < 0.0f;
        const float den = between ? d2 * (l * l) : mn;
        const bool ok = fminf(fminf(A2, B2), den) >= kFltMin && !(between && d2 <= 0x1p-44f * (from_v ? B2 : A2));
        const float k = (between ? mn * q.w : q.w) * __builtin_amdgcn_rcpf(den);
        t.ku = ok ? k * ia : 0.0f;
        t.kv = ok ? k * ib : 0.0f;
        return t;
    }
    // Any other point's; where `den` comes out below kNear it is near_term's to form.
    __device__ __forceinline__ Term term(const float4 q, float &den) const {
        const float x = __builtin_fmaf(-q.x, s, u[0]), y = __builtin_fmaf(-q.y, s, u[1]), z = __builtin_fmaf(-q.z, s, u[2]);
        const float a = dot3(x, y, z, f[0], f[1], f[2]);  // A = a E + P
        const float px = __builtin_fmaf(-a, E[0], x), py = __builtin_fmaf(-a, E[1], y), pz = __builtin_fmaf(-a, E[2], z);
        // (1e-37 keeps the squares of the distances from 0)
        const float d2 = __builtin_fmaf(pz, pz, __builtin_fmaf(py, py, __builtin_fmaf(px, px, 1.0e-37f)));
        const float ul = a * l, vl = ul + l;
        const float A2 = __builtin_fmaf(ul, ul, d2), B2 = __builtin_fmaf(vl, vl, d2), AB = __builtin_fmaf(ul, vl, d2);
        const float ia = __builtin_amdgcn_rsqf(A2), ib = __builtin_amdgcn_rsqf(B2);
        const float mn = (A2 * ia) * (B2 * ib) + __builtin_fabsf(AB);
        // 1 / (|A| |B| + A . B); between the ends, where that cancels, through
        // (|A| |B|)^2 - (A . B)^2 = |P|^2 |E|^2
        const bool between = AB < 0.0f;
        den = between ? d2 * (l * l) : mn;
        const float k = (between ? mn * q.w : q.w) * __builtin_amdgcn_rcpf(den);
        return Term{{px, py, pz}, k * ia, k * ib};
    }
    // Adds g J P at the n points (x, y, z, g) for either end, four at a time; those up to the next
    // multiple of four are there, without weight.  Points that are close to the edge of any lane are taken by
    // near_term: with kHold the four terms wait for the test (107 registers), else they are added as they
    // come and a group of eight with such a point is taken again by near_term, which holds for every point.
    // k_edge_bwd holds them: adjoints of 1000 to 5000 faces below 2^19 voxels take 0 to 7 % less than without,
    // 326 us for 351 at 4983 faces of 72 x 38 x 76.  k_edge_blocks, which has a block's state to keep as well,
    // needs 95 registers without and 116 with it, and is no faster with it.
    template <bool kHold>
    __device__ __forceinline__ void add(const float4 *pts, int n, float (&su)[3], float (&sv)[3]) const {
        constexpr int kGroup = kHold ? 4 : 8;
#pragma unroll 1
        for (int i0 = 0; i0 < n; i0 += kGroup) {
            float least = INFINITY;
            if constexpr (kHold) {
                Term t[4];
                float den[4];
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    t[j] = term(pts[i0 + j], den[j]);
                    least = fminf(least, den[j]);
                }
                if (__builtin_expect(__builtin_amdgcn_ballot_w64(least < kNear) != 0ull, 0)) {
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        if (den[j] < kNear) t[j] = near_term(pts[i0 + j]);
                }
#pragma unroll
                for (int j = 0; j < 4; ++j) add_term(t[j], su, sv);
                continue;
            }
            const int i1 = min(n, i0 + kGroup);
            float bu[3], bv[3];
#pragma unroll
            for (int d = 0; d < 3; ++d) bu[d] = su[d], bv[d] = sv[d];
#pragma unroll 1
            for (int i = i0; i < i1; i += 4)
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    float den;
                    const Term t = term(pts[i + j], den);
                    least = fminf(least, den);
                    add_term(t, su, sv);
                }
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(least < kNear) == 0ull, 1)) continue;
#pragma unroll
            for (int d = 0; d < 3; ++d) su[d] = bu[d], sv[d] = bv[d];
#pragma unroll 1
            for (int i = i0; i < i1; ++i) add_term(near_term(pts[i]), su, sv);
        }
    }
    static __device__ __forceinline__ void add_term(const Term &t, float (&su)[3], float (&sv)[3]) {
#pragma unroll
        for (int d = 0; d < 3; ++d) {
            su[d] = __builtin_fmaf(t.ku, t.p[d], su[d]);
            sv[d] = __builtin_fmaf(t.kv, t.p[d], sv[d]);
        }
    }
    // Points within 1/128 (and up to 1/64, by direction) of the edge's length of an end, or 1/8 of it of the
    // edge between them: beyond, |B| is off by at most 3e-5, and 1e-6 from a tenth of the length on.
    static constexpr float kNear = 0x1p-6f;
};

// state: float2 (sum, compensation) [S][6][B].  Grid: waves; wave w takes edge block
// w mod blocks of the split w / blocks.  dL/dW that is not finite is noted (with
// no edge at all the points are only looked at): every vertex gets NaN then, as from the
// all-pairs sum.
__global__ __launch_bounds__(64) void k_edge_bwd(const char *table, int64_t nQ, int64_t t0, int64_t t1,
                                                 const float *__restrict__ dLdW, float2 *__restrict__ state) {
    __shared__ float4 pts[kTile];
    const CycMesh &m = *reinterpret_cast<const CycMesh *>(table + reinterpret_cast<const CycHead *>(table)->meshes);
    if (m.st->go) return;
    const int B = __builtin_amdgcn_readfirstlane(m.st->n_rec);
    const int blocks = B > 64 ? (B + 63) / 64 : 1;
    const int tiles = (int)((nQ + kTile - 1) / kTile), S = edge_splits(B, tiles);
    const int lane = threadIdx.x;
    const PointSrc ps = m.ps;
    bool odd = false;
    for (int w = blockIdx.x; w < blocks * S; w += gridDim.x) {
        const int s = w / blocks, block = w - s * blocks;
        // the split's first tile in the range
        int t = (int)t0 - (int)t0 % S + s;
        if (t < (int)t0) t += S;
        if (t >= (int)t1) continue;
        const int e = block * 64 + lane;
        const bool live = e < B;
        const int2 id = B > 0 ? m.edge[live ? e : B - 1] : make_int2(0, 0);
        const Edge edge(m, id);
        for (; t < (int)t1; t += S) {
            const int q0 = t * kTile;
            const int nt = (int)min((int64_t)kTile, nQ - q0);
            __syncthreads();
#pragma unroll 1
            for (int k = 0; k < kTile / 64; ++k) {
                const int j = lane + 64 * k;
                float x, y, z, g = 0.0f;  // past the last point: that point again, without weight
                ps.get(q0 + min(j, nt - 1), x, y, z);
                if (j < nt) g = dLdW[q0 + j];
                odd = odd || !(__builtin_fabsf(g) < INFINITY);
                pts[j] = make_float4(x, y, z, g);
            }
            __syncthreads();
            if (B == 0) continue;
            float su[3] = {0.0f, 0.0f, 0.0f}, sv[3] = {0.0f, 0.0f, 0.0f};
            edge.add<true>(pts, kTile, su, sv);
            if (live) {
                float2 *row = state + (int64_t)s * 6 * B + e;
                const float ts[6] = {su[0], su[1], su[2], sv[0], sv[1], sv[2]};
                float2 x[6];
#pragma unroll
                for (int i = 0; i < 6; ++i) x[i] = t < S ? make_float2(0.0f, 0.0f) : row[(int64_t)i * B];
#pragma unroll
                for (int i = 0; i < 6; ++i) {
                    neumaier_add(x[i].x, x[i].y, ts[i]);
                    row[(int64_t)i * B] = x[i];
                }
            }
        }
    }
    if (__builtin_amdgcn_ballot_w64(odd) && lane == 0) atomicOr(&m.st->odd, 1);
}

// Large grids.  An edge's J P is smooth away from it, so a block of voxels acts on a far edge
// through its nodes: the block's dL/dW, weighted with what each node gives to each voxel, summed
// per node (the transpose of the caps' interpolation).  The errors allowed are a tenth of the
// field's: they are relative to a gradient here.
constexpr float kEdgeTight = 0.1f;
constexpr int kParts = 8;

// A value that is the same in every lane, as a scalar.
__device__ __forceinline__ float uniform(float x) {
    return __uint_as_float((unsigned)__builtin_amdgcn_readfirstlane((int)__float_as_uint(x)));
}

// Node sums of dL/dW, a workgroup per block from `first` on: [block][coarse, fine].
__global__ __launch_bounds__(kBlock) void k_edge_nodes(const char *table, int first, const float *__restrict__ dLdW,
                                                       float *__restrict__ node) {
    static_assert(kBlock == kBlockSide * kBlockSide, "a thread per (y, z)");
    __shared__ float T[3][kBlockSide][kFine], C[3][kFine][kCoarse];
    __shared__ float Y[kFine][kBlockSide][kBlockSide], Z[kFine][kFine][kBlockSide], S[kFine][kFine][kFine];
    const CycMesh &m = *reinterpret_cast<const CycMesh *>(table + reinterpret_cast<const CycHead *>(table)->meshes);
    if (m.st->go) return;
    const CycBlocks &g = m.grid;
    const int tid = threadIdx.x, ty = tid / kBlockSide, tz = tid % kBlockSide;
    for (int e = tid; e < 3 * kBlockSide * kFine; e += kBlock) {
        const int d = e / (kBlockSide * kFine), i = e / kFine % kBlockSide, j = e % kFine;
        T[d][i][j] = i < g.size[d] && j < g.fine[d] ? node_weight(kFine, g.size[d], (float)i, j) : 0.0f;
    }
    if (tid < 3 * kFine * kCoarse) {
        const int d = tid / (kFine * kCoarse), i = tid / kCoarse % kFine, j = tid % kCoarse;
        C[d][i][j] = i < g.fine[d] && j < g.coarse[d]
                         ? node_weight(kCoarse, g.size[d], node_at(kFine, g.size[d], i), j)
                         : 0.0f;
    }
    __syncthreads();
    int i0[3];
    const int b = first + (int)blockIdx.x;
    block_origin(m, b, i0);
    const int iy = i0[1] + ty, iz = i0[2] + tz;
    const bool in = ty < g.size[1] && tz < g.size[2] && iy < m.ps.n1 && iz < m.ps.n2;
    float v[kFine];
#pragma unroll
    for (int j = 0; j < kFine; ++j) v[j] = 0.0f;
    bool odd = false;
    for (int x = 0; x < g.size[0] && i0[0] + x < m.n0; ++x) {
        const float w = in ? dLdW[((int64_t)(i0[0] + x) * m.ps.n1 + iy) * m.ps.n2 + iz] : 0.0f;
        odd = odd || !(__builtin_fabsf(w) < INFINITY);
#pragma unroll
        for (int j = 0; j < kFine; ++j) v[j] = __builtin_fmaf(T[0][x][j], w, v[j]);
    }
    if (__builtin_amdgcn_ballot_w64(odd) && (tid & 63) == 0) atomicOr(&m.st->odd, 1);
#pragma unroll
    for (int j = 0; j < kFine; ++j) Y[j][ty][tz] = v[j];
    __syncthreads();
    for (int e = tid; e < kFine * kFine * kBlockSide; e += kBlock) {
        const int j0 = e / (kFine * kBlockSide), j1 = e / kBlockSide % kFine, z = e % kBlockSide;
        float a = 0.0f;
        for (int y = 0; y < kBlockSide; ++y) a = __builtin_fmaf(Y[j0][y][z], T[1][y][j1], a);
        Z[j0][j1][z] = a;
    }
    __syncthreads();
    const int nc = g.coarse[0] * g.coarse[1] * g.coarse[2], nf = g.fine[0] * g.fine[1] * g.fine[2];
    float *out = node + (int64_t)b * (nc + nf);
    for (int e = tid; e < kFine * kFine * kFine; e += kBlock) {
        const int j0 = e / (kFine * kFine), j1 = e / kFine % kFine, j2 = e % kFine;
        float a = 0.0f;
        for (int z = 0; z < kBlockSide; ++z) a = __builtin_fmaf(Z[j0][j1][z], T[2][z][j2], a);
        S[j0][j1][j2] = a;
        if (j0 < g.fine[0] && j1 < g.fine[1] && j2 < g.fine[2]) out[nc + (j0 * g.fine[1] + j1) * g.fine[2] + j2] = a;
    }
    __syncthreads();
    if (tid < nc) {
        const int k0 = tid / (g.coarse[1] * g.coarse[2]), r = tid % (g.coarse[1] * g.coarse[2]);
        const int k1 = r / g.coarse[2], k2 = r % g.coarse[2];
        float a = 0.0f;
        for (int j0 = 0; j0 < kFine; ++j0) {
            float a0 = 0.0f;
            for (int j1 = 0; j1 < kFine; ++j1) {
                float a1 = 0.0f;
                for (int j2 = 0; j2 < kFine; ++j2) a1 = __builtin_fmaf(S[j0][j1][j2], C[2][j2][k2], a1);
                a0 = __builtin_fmaf(a1, C[1][j1][k1], a0);
            }
            a = __builtin_fmaf(a0, C[0][j0][k0], a);
        }
        out[tid] = a;
    }
}

// A wave per 64 edges and split; split s takes the parts s, s + S, ... of the blocks (an eighth of the fine
// nodes and of the voxels each, all coarse nodes in one of them): far edges at the coarse or
// the fine nodes, near ones at the voxels (lanes without such an edge wait).  With whole blocks
// the waves that had near edges took 864 us.
// kRange: the call takes the parts [x0, x1) of a sequence, and a split goes on from its sums in `state`; else all
// of them (an instance of its own: 1.5 % of the adjoint).
// state: float2 [S][6][B].  Bound by 40 VALU and 3 transcendentals per (edge, point), a part of them in lanes that
// wait: 1154 edges on 96 x 88 x 97 voxels take 621 to 700 us, all points one by one 1024.
template <bool kRange>
__global__ __launch_bounds__(64) void k_edge_blocks(const char *table, const float *__restrict__ dLdW,
                                                    const float *__restrict__ node, int S, int x0, int x1,
                                                    float2 *__restrict__ state) {
    __shared__ float4 pts[kTile];
    const CycMesh &m = *reinterpret_cast<const CycMesh *>(table + reinterpret_cast<const CycHead *>(table)->meshes);
    if (m.st->go) return;
    const int B = __builtin_amdgcn_readfirstlane(m.st->n_rec), groups = (B + 63) / 64;
    const CycBlocks &g = m.grid;
    const int nc = g.coarse[0] * g.coarse[1] * g.coarse[2], nf = g.fine[0] * g.fine[1] * g.fine[2];
    const int voxels = g.size[0] * g.size[1] * g.size[2], blocks = g.n[0] * g.n[1] * g.n[2];
    const int lane = threadIdx.x;
    for (int64_t w = blockIdx.x; w < (int64_t)groups * S; w += gridDim.x) {
        const int split = (int)(w / groups), e = (int)(w - (int64_t)split * groups) * 64 + lane;
        const int first = kRange && split < x0 ? split + (x0 - split + S - 1) / S * S : split;
        if (kRange && first >= x1) continue;
        const bool live = e < B;
        const int2 id = m.edge[live ? e : B - 1];
        const Edge edge(m, id);
        float s[6], c[6];
#pragma unroll
        for (int i = 0; i < 6; ++i) s[i] = c[i] = 0.0f;
        if (kRange && split < x0 && live)
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                const float2 x = state[((int64_t)split * 6 + i) * B + e];
                s[i] = x.x, c[i] = x.y;
            }
        for (int x = first; x < (kRange ? x1 : blocks * kParts); x += S) {
            const int b = x / kParts, part = x - b * kParts;
            int i0[3];
            block_origin(m, b, i0);
            Block box(m, i0);
            for (int d = 0; d < 3; ++d) box.lo[d] = uniform(box.lo[d]);  // (three registers less)
            const int kind = live ? box.kind(edge.start(), kEdgeTight) : 0;
            const float *at = node + (int64_t)b * (nc + nf);
#pragma unroll 1
            for (int want = 2; want >= -1; --want) {
                if (want == 0 || !__builtin_amdgcn_ballot_w64(kind == want)) continue;
                const int n = want == 2 ? nc : want == 1 ? nf : voxels, order = want == 2 ? kCoarse : kFine;
                const int *side = want == 2 ? g.coarse : want == 1 ? g.fine : g.size;
                // (the coarse nodes are few: one part has them all)
                const int first = want == 2 ? (part == b % kParts ? 0 : n) : n * part / kParts;
                const int end = want == 2 ? n : n * (part + 1) / kParts;
                for (int t0 = first; t0 < end; t0 += kTile) {
                    const int here = min(kTile, end - t0);
                    __syncthreads();
#pragma unroll 1
                    for (int k = lane; k < (here + 3) / 4 * 4; k += 64) {
                        const int x = t0 + min(k, here - 1), a = x / (side[1] * side[2]), r = x - a * side[1] * side[2];
                        const int j = r / side[2], l = r - j * side[2];
                        if (want > 0) {
                            pts[k] = make_float4(__builtin_fmaf(node_at(order, g.size[0], a), m.ps.h[0], box.lo[0]),
                                                 __builtin_fmaf(node_at(order, g.size[1], j), m.ps.h[1], box.lo[1]),
                                                 __builtin_fmaf(node_at(order, g.size[2], l), m.ps.h[2], box.lo[2]),
                                                 k < here ? at[(want == 2 ? 0 : nc) + x] : 0.0f);
                        } else {
                            const int ix = i0[0] + a, iy = i0[1] + j, iz = i0[2] + l;
                            const bool in = k < here && ix < m.n0 && iy < m.ps.n1 && iz < m.ps.n2;
                            // (beyond the grid: a voxel of it, without weight)
                            pts[k] = make_float4(centre(m.ps, 0, min(ix, m.n0 - 1)), centre(m.ps, 1, min(iy, m.ps.n1 - 1)),
                                                 centre(m.ps, 2, min(iz, m.ps.n2 - 1)),
                                                 in ? dLdW[((int64_t)ix * m.ps.n1 + iy) * m.ps.n2 + iz] : 0.0f);
                        }
                    }
                    __syncthreads();
                    if (kind == want) {
                        float su[3] = {0.0f, 0.0f, 0.0f}, sv[3] = {0.0f, 0.0f, 0.0f};
                        edge.add<false>(pts, here, su, sv);
#pragma unroll
                        for (int i = 0; i < 3; ++i) {
                            neumaier_add(s[i], c[i], su[i]);
                            neumaier_add(s[3 + i], c[3 + i], sv[i]);
                        }
                    }
                }
            }
        }
        if (live)
#pragma unroll
            for (int i = 0; i < 6; ++i) state[((int64_t)split * 6 + i) * B + e] = make_float2(s[i], c[i]);
    }
}

// dL/dW of a point range, for the calls that complete its blocks.
__global__ __launch_bounds__(kBlock) void k_edge_keep(const char *table, const float *__restrict__ dLdW, int64_t n,
                                                      float *__restrict__ kept) {
    const CycMesh &m = *reinterpret_cast<const CycMesh *>(table + reinterpret_cast<const CycHead *>(table)->meshes);
    if (m.st->go) return;  // (the all-pairs sums use that space)
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        kept[i] = dLdW[i];
}

// Notes a term of vertex v (three floats) in the largest of its terms.
__device__ __forceinline__ void note_term(const CycMesh &m, int32_t v, const float *x) {
    uint32_t bits = 0;
    for (int d = 0; d < 3; ++d)
        if (__builtin_fabsf(x[d]) < INFINITY) bits = max(bits, __float_as_uint(__builtin_fabsf(x[d])));
    if (bits) atomicMax(&m.most[v], bits);
}

// One wave per edge: its six sums over the splits (lane l the splits l, l + 64, ... in
// order, then the lanes in pairs), and the gradients of its two ends.
__global__ __launch_bounds__(kBlock) void k_edge_reduce(const char *table, int64_t nQ, int splits,
                                                        const float2 *__restrict__ state, float *__restrict__ G) {
    const CycMesh &m = *reinterpret_cast<const CycMesh *>(table + reinterpret_cast<const CycHead *>(table)->meshes);
    if (m.st->go) return;
    const int64_t B = m.st->n_rec, S = splits > 0 ? splits : edge_splits((int)B, (int)((nQ + kTile - 1) / kTile));
    const int lane = threadIdx.x & 63;
    for (int64_t e = (int64_t)blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6); e < B;
         e += (int64_t)gridDim.x * (kBlock / 64)) {
        float s[6], c[6];
#pragma unroll
        for (int i = 0; i < 6; ++i) s[i] = c[i] = 0.0f;
        for (int64_t k = lane; k < S; k += 64) {
            float2 x[6];
#pragma unroll
            for (int i = 0; i < 6; ++i) x[i] = state[(k * 6 + i) * B + e];
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                neumaier_add(s[i], c[i], x[i].x);
                c[i] += x[i].y;
            }
        }
#pragma unroll
        for (int o = 1; o < 64; o <<= 1)
#pragma unroll
            for (int i = 0; i < 6; ++i) {
                const float os = __shfl_xor(s[i], o), oc = __shfl_xor(c[i], o);
                const float a = (lane & o) ? os : s[i], b = (lane & o) ? s[i] : os;  // lower lane first
                const float t = a + b;
                const float big = __builtin_fabsf(a) >= __builtin_fabsf(b) ? a : b;
                const float small = __builtin_fabsf(a) >= __builtin_fabsf(b) ? b : a;
                c[i] = (c[i] + oc) + ((big - t) + small);
                s[i] = t;
            }
        if (lane == 0) {
            const int2 id = m.edge[e];
            const float *pu = m.V + 3 * (int64_t)id.x, *pv = m.V + 3 * (int64_t)id.y;
            const double E[3] = {(double)pv[0] - pu[0], (double)pv[1] - pu[1], (double)pv[2] - pu[2]};
            const float scale = Edge(m, id).s;
            const double f = -0.07957747154594767 * scale * scale;  // -1 / (4 pi), and P J is in the edge's units
#pragma unroll
            for (int end = 0; end < 2; ++end) {
                const double P[3] = {(double)s[3 * end] + c[3 * end], (double)s[3 * end + 1] + c[3 * end + 1],
                                     (double)s[3 * end + 2] + c[3 * end + 2]};
                G[6 * e + 3 * end + 0] = (float)(f * (P[1] * E[2] - P[2] * E[1]));
                G[6 * e + 3 * end + 1] = (float)(f * (P[2] * E[0] - P[0] * E[2]));
                G[6 * e + 3 * end + 2] = (float)(f * (P[0] * E[1] - P[1] * E[0]));
                note_term(m, end ? id.y : id.x, G + 6 * e + 3 * end);
            }
        }
    }
}

// The terms of dL/dV: the two ends of each boundary edge (G), or, for a mesh that took the
// all-pairs sum, every corner (T).  They are added per vertex as 64-bit integers, so that the sum
// does not depend on the order, on a scale of the vertex's own: with n terms in all and the vertex's of at
// most 2^e the unit is 2^(e - 61) n, rounded up to a power of two, 1e-13 of its largest term for 1e5
// terms (on one scale for the mesh a vertex beside one whose terms are 1e13 times larger got 0).
struct Terms {
    const float *x;  // three floats per term
    int64_t n;
    bool edges;
};

__device__ __forceinline__ Terms terms_of(const CycMesh &m, const float *G, const float *T) {
    if (m.st->go) return Terms{T, 3 * m.nF, false};
    return Terms{G, 2 * (int64_t)m.st->n_rec, true};
}

// Power of two that a term of vertex v is multiplied by.
__device__ __forceinline__ int term_shift(const CycMesh &m, int64_t n, int64_t v) {
    int bits = 0;
    while (bits < 40 && ((int64_t)1 << bits) < n) ++bits;
    const int e = (int)(m.most[v] >> 23) - 126;  // |term| < 2^e
    return 61 - bits - e;
}

// The vertex of term i.
__device__ __forceinline__ int32_t term_vertex(const CycMesh &m, bool edges, int64_t i) {
    if (edges) {
        const int2 e = m.edge[i >> 1];
        return (i & 1) ? e.y : e.x;
    }
    const int32_t v = m.F[i];
    return (v < 0 || (int64_t)v >= m.nV) ? 0 : v;
}

// Largest corner gradients (the edges' are noted as they are formed).
__global__ __launch_bounds__(kBlock) void k_corner_max(const char *table, const float *__restrict__ T) {
    const CycMesh &m = *reinterpret_cast<const CycMesh *>(table + reinterpret_cast<const CycHead *>(table)->meshes);
    if (m.st->go == 0) return;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < 3 * m.nF; i += (int64_t)gridDim.x * blockDim.x)
        note_term(m, term_vertex(m, false, i), T + 3 * i);
}

__global__ __launch_bounds__(kBlock) void k_add_terms(const char *table, const float *__restrict__ G,
                                                      const float *__restrict__ T) {
    const CycMesh &m = *reinterpret_cast<const CycMesh *>(table + reinterpret_cast<const CycHead *>(table)->meshes);
    const Terms t = terms_of(m, G, T);
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < t.n; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t v = term_vertex(m, t.edges, i);
        const int shift = term_shift(m, t.n, v);
        for (int d = 0; d < 3; ++d) {
            const float x = t.x[3 * i + d];
            if (__builtin_fabsf(x) < INFINITY)
                atomicAdd(reinterpret_cast<unsigned long long *>(&m.grad[3 * (int64_t)v + d]),
                          (unsigned long long)__double2ll_rn(ldexp((double)x, shift)));
            else
                m.used[v] = 2;
        }
    }
}

__global__ __launch_bounds__(kBlock) void k_write_grad(const char *table, float *__restrict__ dLdV) {
    const CycMesh &m = *reinterpret_cast<const CycMesh *>(table + reinterpret_cast<const CycHead *>(table)->meshes);
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 3 * m.nV) return;
    const int32_t used = m.used[i / 3];
    const int shift = term_shift(m, m.st->go ? 3 * m.nF : 2 * (int64_t)m.st->n_rec, i / 3);
    // dL/dW that is not finite reaches every vertex of a face
    const bool odd = used == 2 || (used == 1 && m.st->go == 0 && m.st->odd);
    dLdV[i] = odd ? NAN : (float)ldexp((double)m.grad[i], -shift);
}

}  // namespace

hipError_t launch_edge_bwd(const char *table, int64_t nQ, int64_t t0, int64_t t1, const float *dLdW, float2 *state,
                           hipStream_t s) {
    k_edge_bwd<<<kEdgeWaves, 64, 0, s>>>(table, nQ, t0, t1, dLdW, state);
    return hipGetLastError();
}

EdgeBlocks edge_blocks(const CycBlocks &g, int64_t nF, int64_t nQ, char *space, size_t bytes) {
    EdgeBlocks e{};
    if (g.order == 0 || nQ < kEdgeBlockPoints) return e;
    const int64_t blocks = (int64_t)g.n[0] * g.n[1] * g.n[2];
    const size_t node = align_up(4 * (size_t)cyc_node_floats(CycBlocks{g.order, {g.size[0], g.size[1], g.size[2]},
                                                                       {g.n[0], g.n[1], g.n[2]},
                                                                       {g.coarse[0], g.coarse[1], g.coarse[2]},
                                                                       {g.fine[0], g.fine[1], g.fine[2]}, 1},
                                                             g.n[0]));
    const size_t kept = align_up(4 * (size_t)nQ);
    if (node + kept >= bytes) return e;
    const int64_t splits = std::min<int64_t>(blocks, (int64_t)((bytes - node - kept) / (48 * (size_t)nF)));
    if (splits < std::min<int64_t>(blocks, 64)) return e;
    e.splits = (int)splits;
    e.state = reinterpret_cast<float2 *>(space);
    e.kept = reinterpret_cast<float *>(space + bytes / 256 * 256 - kept);
    e.node = reinterpret_cast<float *>(reinterpret_cast<char *>(e.kept) - node);
    return e;
}

hipError_t launch_edge_keep(const char *table, const float *dLdW, int64_t p0, int64_t n, const EdgeBlocks &e,
                            hipStream_t s) {
    k_edge_keep<<<1024, kBlock, 0, s>>>(table, dLdW + p0, n, e.kept + p0);
    return hipGetLastError();
}

hipError_t launch_edge_blocks(const char *table, const CycBlocks &g, int64_t plane, int64_t p0, int64_t p1, int64_t nQ,
                              const float *dLdW, const EdgeBlocks &e, hipStream_t s) {
    // layers of blocks along x that are complete with so many points
    auto complete = [&](int64_t points) { return points >= nQ ? g.n[0] : (int)(points / (plane * g.size[0])); };
    const int layer = g.n[1] * g.n[2], b0 = complete(p0) * layer, b1 = complete(p1) * layer;
    if (b1 == b0) return hipSuccess;
    k_edge_nodes<<<(unsigned)(b1 - b0), kBlock, 0, s>>>(table, b0, dLdW, e.node);
    (p1 - p0 < nQ ? k_edge_blocks<true> : k_edge_blocks<false>)<<<kEdgeWaves, 64, 0, s>>>(
        table, dLdW, e.node, e.splits, b0 * kParts, b1 * kParts, e.state);
    return hipGetLastError();
}

hipError_t launch_edge_reduce(const char *table, int64_t nQ, int splits, const float2 *state, float *G, hipStream_t s) {
    k_edge_reduce<<<1024, kBlock, 0, s>>>(table, nQ, splits, state, G);
    return hipGetLastError();
}

hipError_t launch_edge_gather(const char *table, int64_t nV, const float *G, const float *T, float *dLdV,
                              hipStream_t s) {
    k_corner_max<<<256, kBlock, 0, s>>>(table, T);
    k_add_terms<<<256, kBlock, 0, s>>>(table, G, T);
    k_write_grad<<<(unsigned)((3 * nV + kBlock - 1) / kBlock), kBlock, 0, s>>>(table, dLdV);
    return hipGetLastError();
}

}  // namespace wn
