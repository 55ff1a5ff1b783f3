// Forward by the boundary of the mesh; see wn_cycle.hpp for the identity.
//
// Steps, each a launch over all meshes of a call:
//   begin   clear the chains and the crossing counts (kept in W);
//   faces   chain every half-edge by its undirected edge; crossings of the small faces
//           with the columns of voxels, and the voxels close to them;
//   mark    half-edges whose undirected edge does not cancel: the mesh's boundary;
//   caps    (one workgroup per mesh) join the boundary edges to loops, fill each loop with
//           a zigzag strip of triangles;
//   slabs   crossings of the large faces and the caps;
//   columns winding number of M - C at every voxel from the crossings above it, and the
//           list of voxels close to a face;
//   sum     solid angles of the caps at every voxel, W and occupancy;
//   near    the direct sum at the listed voxels.
// A mesh that the path does not suit (an edge used three times the same way, a
// boundary longer than the face count or with too many edges at a vertex, caps that cost
// more than the faces, coordinates out of range, a strip stream that does not name every
// face once) sets `go` and the all-pairs kernels, launched after `sum`, run for it;
// otherwise they leave at once.  More voxels than the list holds are
// marked, and the all-pairs kernels run for the marked ones.
#include "wn_blocks.hpp"

#include <algorithm>
#include <cmath>

namespace wn {

namespace {

constexpr int kChainLimit = 1024;   // half-edges looked at per chain before giving up
constexpr int kDegreeLimit = 1024;  // boundary edges looked at per vertex; fewer for long boundaries (degree_limit)
constexpr float kCoordMax = 1.0e9f; // coordinates beyond this (or not finite) go direct

__device__ __forceinline__ const CycMesh *meshes_of(const char *table) {
    return reinterpret_cast<const CycMesh *>(table + reinterpret_cast<const CycHead *>(table)->meshes);
}

template <int64_t CycMesh::*First>
__device__ __forceinline__ const CycMesh *find_mesh(const char *table, int64_t u) {
    const CycHead *h = reinterpret_cast<const CycHead *>(table);
    const CycMesh *m = meshes_of(table);
    int lo = 0, hi = h->n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (m[mid].*First <= u)
            lo = mid;
        else
            hi = mid - 1;
    }
    return m + lo;
}

__device__ __forceinline__ int32_t face_vertex(const CycMesh &m, int64_t h) {
    const int32_t v = m.F[h];
    return (v < 0 || (int64_t)v >= m.nV) ? 0 : v;  // as the packs replace them
}

// Half-edge h = 3 f + j runs from corner j to corner j + 1 of face f.
__device__ __forceinline__ void half_edge(const CycMesh &m, int64_t h, int32_t &u, int32_t &v) {
    const int64_t f = h / 3;
    const int j = (int)(h - 3 * f);
    u = face_vertex(m, h);
    v = face_vertex(m, 3 * f + (j == 2 ? 0 : j + 1));
}

// Crossing counts live in the W array until the columns are summed: a bias that keeps them
// positive, and the top bit for "close to a face".
constexpr uint32_t kCountBias = 0x40000000u, kCloseBit = 0x80000000u;

__device__ void clear_unit(const CycMesh &m, int64_t u) {
    for (int64_t i = u * kCycClear + threadIdx.x; i < (u + 1) * kCycClear; i += kCycUnit) {
        if (i < m.buckets) m.head[i] = -1;
        if (m.W && i < m.nV) m.hout[i] = m.hin[i] = -1;
        if (m.strips && i < m.nF) m.count[i] = 0;
        if (m.W && i < m.P) reinterpret_cast<uint32_t *>(m.W)[m.p0 + i] = kCountBias;
        if (m.W && 32 * i < m.P) m.mark[i] = 0u;
        if (i < (int64_t)m.bins * m.bins) {
            m.bin[i] = -1;
            m.bin_n[i] = 0;
        }
        if (!m.W && i < m.nV) {
            m.used[i] = 0;
            m.most[i] = 0u;
        }
        if (!m.W && i < 3 * m.nV) m.grad[i] = 0;
        if (i == 0) *m.st = CycState{};
    }
}

__global__ __launch_bounds__(kCycUnit) void k_cyc_begin_one(CycMesh m, CycHead h, char *table) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        *reinterpret_cast<CycHead *>(table) = h;
        *reinterpret_cast<CycMesh *>(table + h.meshes) = m;
        if (m.hdr) {
            m.hdr->bad_index = 0;
            m.hdr->cursor = 0ull;
        }
    }
    clear_unit(m, blockIdx.x);
}

__global__ __launch_bounds__(kCycUnit) void k_cyc_clear(char *table) {
    CycHead *h = reinterpret_cast<CycHead *>(table);
    if (blockIdx.x == 0 && threadIdx.x == 0) h->cursor = 0ull;
    for (int64_t u = blockIdx.x; u < h->u_clear; u += gridDim.x) {
        const CycMesh &m = *find_mesh<&CycMesh::u_clear>(table, u);
        clear_unit(m, u - m.u_clear);
    }
}

// ------------------------------------------------------------------ crossings

// Voxels closer to a triangle than this share of its extent are listed: there
// the side of the triangle, and with it the jump of its solid angle, is near the rounding
// of FP32 (about 4e-7 of the extent), and the all-pairs sum's own error grows as 1e-7
// extent / distance.
constexpr double kClose = 2.0e-4;

// What edge (p, q) adds to the winding of its triangle's projection about (x, y): the
// signed crossing with the ray towards +x.  The same for every face that uses the edge but
// for the sign, so the windings of a closed surface's faces cancel exactly, whatever the
// rounding.
__device__ __forceinline__ int edge_crossing(double px, double py, double qx, double qy, double x, double y) {
    const bool up = py <= y && qy > y, down = qy <= y && py > y;
    if (!(up || down)) return 0;
    const double lx = up ? px : qx, ly = up ? py : qy, ux = up ? qx : px, uy = up ? qy : py;
    const double t = (x - lx) * (uy - ly);
    return __builtin_fma(ux - lx, y - ly, -t) > 0.0 ? (up ? 1 : -1) : 0;
}

__device__ __forceinline__ float axis_centre(const PointSrc &ps, int d, int i) {
    return __builtin_fmaf((float)i + 0.5f, ps.h[d], ps.lo[d]);
}

// Cells whose centres may be a coordinate: more (a grid whose cells are far below the rounding of its place) are
// not looked at one by one.
constexpr int kCentreCells = 1024;

// Cells [a, b] of an axis whose centres may lie in [lo, hi] (all of them, and perhaps a
// neighbour: the slack covers the rounding of the centres), within [first, last].
__device__ __forceinline__ void cell_range(const CycMesh &m, int d, double lo, double hi, int first, int last, int &a,
                                           int &b) {
    const double z = m.ps.lo[d], inv = m.inv_h[d], slack = m.slack[d];
    a = (int)fmin(fmax(ceil((lo - z) * inv - 0.5 - slack), (double)first), (double)last + 1.0);
    b = (int)fmax(fmin(floor((hi - z) * inv - 0.5 + slack), (double)last), (double)first - 1.0);
}

// A float as an unsigned integer of the same order; larger than 0 for every number.
__device__ __forceinline__ uint32_t ordered(float x) {
    const uint32_t b = __float_as_uint(x);
    return (b >> 31) ? ~b : b | 0x80000000u;
}
__device__ __forceinline__ float from_ordered(uint32_t k) {
    return __uint_as_float((k >> 31) ? k & 0x7fffffffu : ~k);
}

// The bins' squares: the box of the vertices with a margin wider than any face's eps, so a point outside
// meets no face.
struct Bins {
    double lo[2], inv[2];

    __device__ __forceinline__ explicit Bins(const CycMesh &m) {
        double a[3], b[3], most = 0.0;
        for (int d = 0; d < 3; ++d) {
            a[d] = -(double)from_ordered(m.st->box[3 + d]);
            b[d] = (double)from_ordered(m.st->box[d]);
            most = fmax(most, b[d] - a[d]);
        }
        const double margin = 1.0e-3 * most + 1.0e-30;
        for (int d = 0; d < 2; ++d) {
            lo[d] = a[d] - margin;
            inv[d] = (double)m.bins / (b[d] - a[d] + 2.0 * margin);
        }
    }
    __device__ __forceinline__ double at(int d, double x) const { return floor((x - lo[d]) * inv[d]); }
};

// A triangle (a, b, c) for the columns of voxels: N, its range, and the cells it may meet.
struct RasterFace {
    double ax, ay, az, bx, by, bz, cx, cy, cz, nx, ny, nz, inv, zmin, zmax, eps, nn;
    float lab, lbc, lca;  // eps times the edges' lengths in the x-y plane
    int i0, i1, j0, j1;

    __device__ __forceinline__ void set(const CycMesh &m, const float *a, const float *b, const float *c) {
        ax = a[0], ay = a[1], az = a[2], bx = b[0], by = b[1], bz = b[2], cx = c[0], cy = c[1], cz = c[2];
        const double e1x = bx - ax, e1y = by - ay, e1z = bz - az, e2x = cx - ax, e2y = cy - ay, e2z = cz - az;
        nx = e1y * e2z - e1z * e2y, ny = e1z * e2x - e1x * e2z, nz = e1x * e2y - e1y * e2x;
        inv = 1.0 / nz;
        zmin = fmin(fmin(az, bz), cz), zmax = fmax(fmax(az, bz), cz);
        const double x0 = fmin(fmin(ax, bx), cx), x1 = fmax(fmax(ax, bx), cx);
        const double y0 = fmin(fmin(ay, by), cy), y1 = fmax(fmax(ay, by), cy);
        eps = kClose * sqrt((x1 - x0) * (x1 - x0) + (y1 - y0) * (y1 - y0) + (zmax - zmin) * (zmax - zmin));
        nn = sqrt(nx * nx + ny * ny + nz * nz) * eps;
        const float e = (float)eps * 1.01f;
        lab = e * length(bx - ax, by - ay), lbc = e * length(cx - bx, cy - by), lca = e * length(ax - cx, ay - cy);
        if (m.bins) {
            const Bins b(m);
            const double top = m.bins - 1.0;
            i0 = (int)fmin(fmax(b.at(0, x0 - eps), 0.0), top), i1 = (int)fmin(fmax(b.at(0, x1 + eps), 0.0), top);
            j0 = (int)fmin(fmax(b.at(1, y0 - eps), 0.0), top), j1 = (int)fmin(fmax(b.at(1, y1 + eps), 0.0), top);
            return;
        }
        cell_range(m, 0, x0 - eps, x1 + eps, m.i_first, m.i_last, i0, i1);
        cell_range(m, 1, y0 - eps, y1 + eps, 0, m.ps.n1 - 1, j0, j1);
    }
    static __device__ __forceinline__ float length(double x, double y) { return fast_sqrt((float)(x * x + y * y)); }
    // Whether (x, y) is inside, or within eps of, the triangle's projection (a superset near
    // its corners; a projection that is a mere line keeps its own strip).
    __device__ __forceinline__ bool over(double x, double y) const {
        const double t = nz < 0.0 ? -1.0 : 1.0;
        return t * ((bx - ax) * (y - ay) - (x - ax) * (by - ay)) >= -lab &&
               t * ((cx - bx) * (y - by) - (x - bx) * (cy - by)) >= -lbc &&
               t * ((ax - cx) * (y - cy) - (x - cx) * (ay - cy)) >= -lca;
    }
    __device__ __forceinline__ int64_t columns() const {
        return i1 < i0 || j1 < j0 ? 0 : (int64_t)(i1 - i0 + 1) * (j1 - j0 + 1);
    }
    // Bin (i, j) of a list of points: the crossing is counted at the points below it.
    __device__ __forceinline__ void points(const CycMesh &m, int sign, int i, int j) const {
        uint32_t *count = reinterpret_cast<uint32_t *>(m.W);
        int32_t after;
        for (int32_t at = m.bin[(int64_t)i * m.bins + j]; at >= 0; at = after) {
            const float *q = m.ps.Q + 3 * (int64_t)at;
            const double x = q[0], y = q[1], z = q[2];
            after = m.after[at];
            const double off = nx * (ax - x) + ny * (ay - y);
            const int w = edge_crossing(ax, ay, bx, by, x, y) + edge_crossing(bx, by, cx, cy, x, y) +
                          edge_crossing(cx, cy, ax, ay, x, y);
            if (w != 0 && z < fmin(fmax(az + off * inv, zmin), zmax)) atomicAdd(&count[at], (uint32_t)(sign * w));
            if (z >= zmin - eps && z <= zmax + eps && fabs(off + nz * (az - z)) <= 1.01 * nn && over(x, y))
                atomicOr(&count[at], kCloseBit);
        }
    }
    // Column (i, j): the crossing is counted at the last voxel below it (a column is summed
    // from the top), and the voxels within eps are marked.
    __device__ __forceinline__ void column(const CycMesh &m, int sign, int i, int j) const {
        if (m.bins) {
            points(m, sign, i, j);
            return;
        }
        const int n2 = m.ps.n2;
        const int64_t base = ((int64_t)i * m.ps.n1 + j) * n2;
        const int first = base >= m.p0 ? 0 : (int)(m.p0 - base < n2 ? m.p0 - base : n2);  // voxels of this slice
        const int last = (int)(m.p0 + m.P - base < n2 ? m.p0 + m.P - base : n2) - 1;
        if (first > last) return;
        uint32_t *count = reinterpret_cast<uint32_t *>(m.W) + base;
        const double x = axis_centre(m.ps, 0, i), y = axis_centre(m.ps, 1, j);
        const double off = nx * (ax - x) + ny * (ay - y);  // N . (a - (x, y, a.z))
        const int w = edge_crossing(ax, ay, bx, by, x, y) + edge_crossing(bx, by, cx, cy, x, y) +
                      edge_crossing(cx, cy, ax, ay, x, y);
        if (w != 0) {
            const double zf = fmin(fmax(az + off * inv, zmin), zmax);  // also a vertical sliver's NaN
            int k = (int)fmin(fmax((zf - m.ps.lo[2]) * m.inv_h[2] - 0.5, 0.0), (double)n2);
            while (k < n2 && (double)axis_centre(m.ps, 2, k) < zf) ++k;
            while (k > 0 && !((double)axis_centre(m.ps, 2, k - 1) < zf)) --k;
            k = min(k - 1, last);
            if (k >= first) atomicAdd(&count[k], (uint32_t)(sign * w));
        }
        if (!over(x, y)) return;
        double lo = zmin - eps, hi = zmax + eps;
        if (fabs(nz) * (hi - lo) > 2.0e-3 * nn) {  // |N . (a - q)| <= |N| eps
            const double zc = az + off * inv, dz = nn * fabs(inv);
            lo = fmax(lo, zc - dz);
            hi = fmin(hi, zc + dz);
        } else if (fabs(off + nz * (az - lo)) > 1.01 * nn) {
            return;
        }
        int ka, kb;
        cell_range(m, 2, lo, hi, first, last, ka, kb);
        for (int k = ka; k <= kb; ++k) atomicOr(&count[k], kCloseBit);
    }
};

// Columns that a face's own lanes take; more are left to the raster list, 64 per entry or as many more as the
// triangle's share of the list asks for: the list has room for a share for each, so it never overflows.
constexpr int kOwnColumns = 64;
constexpr int kListShare = 32768;  // entries for the faces beyond one each, and entries for the caps

__device__ __forceinline__ int face_share(const CycMesh &m) { return 1 + kListShare / (int)m.nF; }

// Entries of a triangle with so many columns (more than 0), and the columns of each.
__device__ __forceinline__ int list_entries(int64_t columns, int share) { return (int)min((columns + 63) / 64, (int64_t)share); }
__device__ __forceinline__ int64_t list_columns(int64_t columns, int share) {
    const int n = list_entries(columns, share);
    return (columns + 64 * (int64_t)n - 1) / (64 * n) * 64;
}

// Puts a triangle on the raster list.  Called by the lanes of a wave together (any of them): one atomic for
// all, since thousands queue up at its address (the caps of 1364 boundary edges took 58 us with one
// each, 55 with one per wave).  Returns how many entries of 64 columns were asked for before (the counter's upper
// half; it may wrap).
__device__ __forceinline__ unsigned add_slabs(const CycMesh &m, int32_t id, int64_t columns, int share) {
    const int n = list_entries(columns, share);
    const int wide = (int)min((columns + 63) / 64, (int64_t)1 << 20);
    const int lane = threadIdx.x & 63;
    unsigned long long asking = __builtin_amdgcn_ballot_w64(true);
    const int leader = __builtin_ctzll(asking);
    unsigned before = 0, total = 0, total_wide = 0;
    for (; asking; asking &= asking - 1ull) {
        const int l = __builtin_ctzll(asking);
        const unsigned x = (unsigned)__builtin_amdgcn_readlane(n, l);
        if (l < lane) before += x;
        total += x;
        total_wide += (unsigned)__builtin_amdgcn_readlane(wide, l);
    }
    unsigned long long at = 0;
    if (lane == leader) at = atomicAdd(&m.st->n_slab, (unsigned long long)total_wide << 32 | total);
    const unsigned first = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)at, leader) + before;
    for (int k = 0; k < n; ++k) m.slab[first + k] = make_int2(id, k);
    return (unsigned)__builtin_amdgcn_readlane((int)(at >> 32), leader);
}

// The bucket of an undirected edge (l < u): a multiplicative hash.
__device__ __forceinline__ int64_t edge_bucket(const CycMesh &m, int32_t l, int32_t u) {
    const uint64_t x = ((uint64_t)(uint32_t)l << 32 | (uint32_t)u) * 0x9E3779B97F4A7C15ull;
    return (int64_t)((x >> 32) & (uint64_t)(m.buckets - 1));
}

// Point lists.  Packs the record stream, and takes the box of the vertices.
__global__ __launch_bounds__(kCycUnit) void k_cyc_box(const char *table) {
    __shared__ uint32_t s_box[6];
    const CycMesh &m = *meshes_of(table);
    const int64_t i = (int64_t)blockIdx.x * kCycUnit + threadIdx.x;
    if (threadIdx.x < 6) s_box[threadIdx.x] = 0u;
    __syncthreads();
    if (i < m.nR) pack_record(i, m.V, m.nV, m.F, m.nF, m.R, m.recs, m.hdr, m.R ? m.count : nullptr, &m.st->go);
    if (i < m.nV)
        for (int d = 0; d < 3; ++d) {
            const float x = m.V[3 * i + d];
            if (__builtin_fabsf(x) <= kCoordMax) {  // (a face corner beyond that makes the mesh go direct)
                atomicMax(&s_box[d], ordered(x));
                atomicMax(&s_box[3 + d], ordered(-x));
            }
        }
    __syncthreads();
    if (threadIdx.x < 6 && s_box[threadIdx.x]) atomicMax(&m.st->box[threadIdx.x], s_box[threadIdx.x]);
}

// Points of a bin that are too many (all faces that meet it go through them one by one).
constexpr int kBinMax = 64;

__global__ __launch_bounds__(kCycUnit) void k_cyc_bin(const char *table) {
    const CycMesh &m = *meshes_of(table);
    const int64_t i = (int64_t)blockIdx.x * kCycUnit + threadIdx.x;
    if (i >= m.P) return;
    const float x = m.ps.Q[3 * i], y = m.ps.Q[3 * i + 1], z = m.ps.Q[3 * i + 2];
    if (!(__builtin_fabsf(x) <= kCoordMax && __builtin_fabsf(y) <= kCoordMax && __builtin_fabsf(z) <= kCoordMax)) {
        atomicOr(reinterpret_cast<uint32_t *>(m.W) + i, kCloseBit);  // the direct sum
        return;
    }
    const Bins b(m);
    const double bx = b.at(0, x), by = b.at(1, y);
    if (!(bx >= 0.0 && by >= 0.0 && bx < (double)m.bins && by < (double)m.bins)) return;
    const int64_t at = (int64_t)bx * m.bins + (int64_t)by;
    if (atomicAdd(&m.bin_n[at], 1) >= kBinMax) {
        atomicMax(&m.st->go, 2);
        return;
    }
    m.after[i] = atomicExch(&m.bin[at], (int32_t)i);
}

// Eight lanes per face: three chain its half-edges, all share its columns.  Bound by the
// latency of the loads and of the FP64 chain per column, so the lanes go to more faces and
// columns at a time rather than to a face's whole range.
// kPack: workgroups beyond the faces' pack the record stream.
template <bool kPack>
__global__ __launch_bounds__(kCycUnit) void k_cyc_faces(const char *table) {
    constexpr int kFaces = kCycUnit / kCycFaceLanes;
    const CycHead *h = reinterpret_cast<const CycHead *>(table);
    if (kPack && blockIdx.x >= h->u_face) {
        const CycMesh &m = *meshes_of(table);
        const int64_t r = ((int64_t)blockIdx.x - h->u_face) * kCycUnit + threadIdx.x;
        if (r < m.nR)
            pack_record(r, m.V, m.nV, m.F, m.nF, m.R, m.recs, m.hdr, m.R ? m.count : nullptr, &m.st->go);
        return;
    }
    const int part = threadIdx.x % kCycFaceLanes;
    for (int64_t u = blockIdx.x; u < h->u_face; u += gridDim.x) {
        const CycMesh &m = *find_mesh<&CycMesh::u_face>(table, u);
        const int64_t f = (u - m.u_face) * kFaces + threadIdx.x / kCycFaceLanes;
        uint32_t bits = 0;
        if (f < m.nF) {
            int32_t id[3];
            float p[3][3];
            for (int j = 0; j < 3; ++j) {
                id[j] = face_vertex(m, 3 * f + j);
                for (int c = 0; c < 3; ++c) {
                    p[j][c] = m.V[3 * (int64_t)id[j] + c];
                    bits = max(bits, __float_as_uint(__builtin_fabsf(p[j][c])));
                }
            }
            if (part < 3) {
                const int32_t a = part == 0 ? id[0] : part == 1 ? id[1] : id[2];
                const int32_t b = part == 0 ? id[1] : part == 1 ? id[2] : id[0];
                int4 x = make_int4(-1, -1, -1, 0);  // a degenerate edge bounds nothing
                if (a != b) {
                    x.y = min(a, b);
                    x.z = max(a, b);
                    x.w = a > b;
                    x.x = atomicExch(&m.head[edge_bucket(m, x.y, x.z)], (int32_t)(3 * f + part));
                }
                m.ent[3 * f + part] = x;
            }
            if (!m.W) {
                // a face whose vertex is a query point contributes nothing there, so its
                // edges do not cancel its neighbours': the all-pairs sum takes such a mesh
                if (part < 3) {
                    const int32_t v = part == 0 ? id[0] : part == 1 ? id[1] : id[2];
                    m.used[v] = 1;
                    bool same = bits <= __float_as_uint(kCoordMax);  // else the mesh goes direct
                    for (int d = 0; d < 3 && same; ++d) {
                        const float x = part == 0 ? p[0][d] : part == 1 ? p[1][d] : p[2][d];
                        int a, b;
                        cell_range(m, d, x, x, 0, (d == 0 ? m.n0 : d == 1 ? m.ps.n1 : m.ps.n2) - 1, a, b);
                        bool hit = b - a > kCentreCells;
                        for (int k = a - 1; k <= b + 1 && !hit; ++k) hit = axis_centre(m.ps, d, k) == x;
                        same = hit;
                    }
                    if (same) atomicMax(&m.st->go, 2);
                }
            } else if (bits <= __float_as_uint(kCoordMax) && !(m.bins && m.st->go)) {  // else the mesh goes direct
                RasterFace r;
                r.set(m, p[0], p[1], p[2]);
                const int64_t n = r.columns();
                if (n > kOwnColumns) {
                    // (many large faces on a list of points are better summed)
                    if (part == 0 && add_slabs(m, (int32_t)f, n, face_share(m)) > (unsigned)m.slab_cap && m.bins)
                        atomicMax(&m.st->go, 2);
                } else {
                    const int nj = r.j1 - r.j0 + 1;
                    for (int c = part; c < (int)n; c += kCycFaceLanes) {
                        const int i = c / nj;
                        r.column(m, 1, r.i0 + i, r.j0 + c - i * nj);
                    }
                }
            }
        }
        for (int o = 32; o > 0; o >>= 1) bits = max(bits, (uint32_t)__shfl_xor((int)bits, o));
        if ((threadIdx.x & 63) == 0 && bits) atomicMax(&m.st->max_bits, bits);
    }
}

// One thread per half-edge: the uses of an undirected edge in its two directions cancel; the first
// half-edge of the direction that is left over stands for it.
__global__ __launch_bounds__(kCycUnit) void k_cyc_mark(const char *table) {
    __shared__ int32_t wave_n[kCycUnit / 64];
    const CycHead *h = reinterpret_cast<const CycHead *>(table);
    for (int64_t u = blockIdx.x; u < h->u_half; u += gridDim.x) {
        const CycMesh &m = *find_mesh<&CycMesh::u_half>(table, u);
        const int64_t unit = u - m.u_half, e = unit * kCycUnit + threadIdx.x;
        bool keep = false;
        if (e < 3 * m.nF) {
            const int4 x = m.ent[e];
            if (x.y != -1) {
                int net = 0, steps = 0;
                bool first = true;
                for (int32_t k = m.head[edge_bucket(m, x.y, x.z)]; k >= 0; ++steps) {
                    if (steps == kChainLimit) {
                        atomicMax(&m.st->go, 2);
                        break;
                    }
                    const int4 y = m.ent[k];
                    if (y.y == x.y && y.z == x.z) {  // the same edge
                        const bool same = y.w == x.w;
                        net += same ? 1 : -1;
                        first = first && !(same && k < (int32_t)e);
                    }
                    k = y.x;
                }
                keep = net > 0 && first;
                if (net > 1) atomicMax(&m.st->go, 2);
            }
            if (m.strips && e < m.nF && m.count[e] != 1) atomicMax(&m.st->go, 2);
        }
        const unsigned long long mask = __builtin_amdgcn_ballot_w64(keep);
        const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
        if (lane == 0) wave_n[wave] = __popcll(mask);
        __syncthreads();
        int base = 0, total = 0;
        for (int w = 0; w < kCycUnit / 64; ++w) {
            if (w < wave) base += wave_n[w];
            total += wave_n[w];
        }
        if (keep) m.list[unit * kCycUnit + base + __popcll(mask & ((1ull << lane) - 1ull))] = (int32_t)e;
        if (threadIdx.x == 0) m.blk[2 * unit] = total;
        __syncthreads();
    }
}

__device__ TriRec tri_record(const RasterFace &f) {
    TriRec t;
    const double d1[3] = {f.bx - f.ax, f.by - f.ay, f.bz - f.az}, d2[3] = {f.cx - f.ax, f.cy - f.ay, f.cz - f.az};
    auto dot = [](const double *x, const double *y) { return x[0] * y[0] + x[1] * y[1] + x[2] * y[2]; };
    t.v[0] = (float)f.ax, t.v[1] = (float)f.ay, t.v[2] = (float)f.az;
    for (int k = 0; k < 3; ++k) {
        t.d[0][k] = (float)(2.0 * d1[k]);
        t.d[1][k] = (float)(2.0 * d2[k]);
    }
    t.d[0][3] = (float)dot(d1, d1);
    t.d[1][3] = (float)dot(d2, d2);
    t.n[0] = (float)f.nx, t.n[1] = (float)f.ny, t.n[2] = (float)f.nz;
    t.g = (float)dot(d1, d2);
    t.far = kFar * kFar * fmaxf(t.d[0][3], t.d[1][3]);
    return t;
}

constexpr int kCapListed = 1 << 30;  // in cpos: the triangle's columns are on the raster list
constexpr int kWaveColumns = 2048;   // columns that one wave takes

// The triangle that cap record x completes (its place in the strip is at least 2), wound as the caps
// are: the zigzag turns every second one.  False for a degenerate one.
__device__ __forceinline__ bool set_cap(const CycMesh &m, int x, RasterFace &f) {
    const int32_t a = m.cvid[x - 2], u = m.cvid[x - 1], v = m.cvid[x];
    if (a == u || u == v || v == a) return false;
    const bool turn = m.cpos[x] & 1;
    f.set(m, m.V + 3 * (int64_t)a, m.V + 3 * (int64_t)(turn ? v : u), m.V + 3 * (int64_t)(turn ? u : v));
    return true;
}

constexpr int kCapThreads = 1024;
constexpr int kUnitLanes = 16;  // lanes that collect the boundary edges of a unit of 256 half-edges: mostly a few
constexpr int kCapLds = 4096;  // a boundary of at most so many edges is worked on in LDS

// Exclusive sum over the workgroup; `total` gets the sum of all.
__device__ __forceinline__ unsigned long long block_scan(unsigned long long x, unsigned long long *red,
                                                         unsigned long long &total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    unsigned long long s = x;
    for (int o = 1; o < 64; o <<= 1) {
        const unsigned long long y = __shfl_up(s, o);
        if (lane >= o) s += y;
    }
    if (lane == 63) red[wave] = s;
    __syncthreads();
    unsigned long long before = 0;
    total = 0;
    for (int w = 0; w < kCapThreads / 64; ++w) {
        if (w < wave) before += red[w];
        total += red[w];
    }
    __syncthreads();
    return before + s - x;
}

// Place of a loop's vertex r (of k) in its zigzag strip p0, p1, p(k-1), p2, p(k-2), ...
__device__ __forceinline__ int zigzag(int r, int k) { return r == 0 ? 0 : (r <= k / 2 ? 2 * r - 1 : 2 * (k - r)); }

// Boundary edges that an edge looks at before the mesh goes direct: with B edges on one workgroup, at most
// 2^25 / 1024 dependent loads per thread and search.
__device__ __forceinline__ int degree_limit(int B) { return min(kDegreeLimit, max(16, (1 << 25) / B)); }

// What the path and the all-pairs sum take, in units of 0.01 ps per voxel, measured on open sheets, ribbons, fans
// and patches: a face of the all-pairs sum without and with a strip order; a cap record summed one by one, of a
// triangle, of another short loop, of a long one (in FP64); in blocks one that is far (as those of short loops
// mostly are), and what one of a long loop adds where it is close (a workgroup takes it for 1024 voxels, so few
// workgroups leave the chip idle); joining, per edge and call; a column that a cap triangle may meet.  Where
// the caps cost more the mesh goes direct: a fan of 5000 faces (5000 edges in one loop) on 64^3 takes 3.37 ms by
// its boundary and 1.63 by its faces, a ribbon of 10000 faces two quads wide 5.7 and 3.1; the ribbon on 128^3
// 13.0 and 25, 1000 patches of eight faces on 64^3 1.7 and 2.5.
constexpr double kFaceCost = 122.0, kStripCost = 88.0, kJoinCost = 3.0e6, kColumnCost = 700.0;
constexpr int kTriCost = 70, kShortCost = 110, kLongCost = 260, kFarCost = 4, kCloseCost = 380;
constexpr int kBusyBlocks = 1024;

__device__ __forceinline__ int64_t all_points(const CycMesh &m) {
    return m.bins ? m.P : (int64_t)m.n0 * m.ps.n1 * m.ps.n2;  // (of a slice its grid's, so that slices decide alike)
}

// Whether caps of this cost per voxel, over B edges and so many columns, make the all-pairs sum the cheaper one.
__device__ __forceinline__ bool caps_cost_more(const CycMesh &m, int64_t B, double cost, double columns = 0.0) {
    const double P = (double)all_points(m);
    return P * cost + kJoinCost * (double)B + kColumnCost * columns > P * (double)m.nF * (m.strips ? kStripCost : kFaceCost);
}

__device__ __forceinline__ double plain_cost(int tri, int other, int lng) {
    return (double)tri * kTriCost + (double)other * kShortCost + (double)lng * kLongCost;
}

// What a triangle of a long loop adds in blocks: close to it are the voxels within twice its edges (and a quarter of a
// block) of its first vertex.
struct CloseCost {
    float lo[3], hi[3], a, scale;  // the grid's box; a quarter of a block; the cost of a triangle close to all, over its volume

    __device__ __forceinline__ explicit CloseCost(const CycMesh &m) {
        const CycBlocks &g = m.grid;
        const int n[3] = {m.n0, m.ps.n1, m.ps.n2};
        const int units = g.n[0] * g.n[1] * g.n[2] * ((g.size[0] + kBlockRows - 1) / kBlockRows);
        a = 0.0f;
        scale = (float)kCloseCost * fmaxf((float)kBusyBlocks / (float)units, 1.0f);
        for (int d = 0; d < 3; ++d) {
            const float w = (float)n[d] * m.ps.h[d];
            lo[d] = m.ps.lo[d];
            hi[d] = lo[d] + w;
            scale /= w;
            a = fmaxf(a, 0.25f * (float)g.size[d] * m.ps.h[d]);
        }
    }
    __device__ __forceinline__ int operator()(const float (&p)[3][3]) const {
        float e2 = 0.0f, x = scale;
        for (int k = 1; k < 3; ++k) {
            const float dx = p[k][0] - p[0][0], dy = p[k][1] - p[0][1], dz = p[k][2] - p[0][2];
            e2 = fmaxf(e2, dx * dx + dy * dy + dz * dz);
        }
        const float r = 2.0f * fast_sqrt(e2) + a;
        for (int d = 0; d < 3; ++d) x *= fmaxf(fminf(p[0][d] + r, hi[d]) - fmaxf(p[0][d] - r, lo[d]), 0.0f);
        return (int)x;
    }
};

constexpr int kWalk = 32;  // edges of a loop that each of its edges walks; longer loops are doubled

// Loops by kind: triangles, other short loops, long loops; three counts of 21 bits.
__device__ __forceinline__ int loop_kind(int k) { return k == 3 ? 0 : k <= kCycShortLoop ? 1 : 2; }
__device__ __forceinline__ int count_of(unsigned long long x, int kind) { return (int)(x >> (21 * kind)) & 0x1fffff; }

// One workgroup per mesh.  Boundary edges are numbered in half-edge order.  Three edges that
// form a triangle are taken as a loop first (two missing faces that touch at a vertex would
// otherwise become one loop of six); then an edge entering a vertex continues with the
// leaving edge of the same rank there.  A loop starts at its lowest edge, so the cap stream
// depends on F alone.  A loop of k edges becomes a strip of k records and k - 2 triangles.
// Bound by the latency of its dependent loads and barriers: 36 us for 1364 edges, 300 for 11082
// (58 and 437 with the chains' heads read from memory and the triangles formed here).
__global__ __launch_bounds__(kCapThreads) void k_cyc_caps(const char *table) {
    __shared__ unsigned long long red[kCapThreads / 64];
    __shared__ int2 s_edge[kCapLds];
    __shared__ int32_t s_work[7][kCapLds];
    __shared__ int32_t s_bad;
    const CycHead *h = reinterpret_cast<const CycHead *>(table);
    const CycMesh *meshes = meshes_of(table);
    const int tid = threadIdx.x;
    for (int mi = blockIdx.x; mi < h->n; mi += gridDim.x) {
        const CycMesh &m = meshes[mi];
        __syncthreads();
        if (tid == 0) s_bad = 0;
        const int64_t units = (3 * m.nF + kCycUnit - 1) / kCycUnit;
        unsigned long long B64 = 0;
        for (int64_t u0 = 0; u0 < units; u0 += kCapThreads) {
            const int64_t u = u0 + tid;
            const int n = u < units ? m.blk[2 * u] : 0;
            unsigned long long all;
            const unsigned long long at = block_scan((unsigned long long)n, red, all);
            if (u < units) m.blk[2 * u + 1] = (int32_t)(B64 + at);
            B64 += all;
        }
        const bool range = m.st->max_bits > __float_as_uint(kCoordMax);  // NaN bits are larger still
        const int least = m.grid.order ? kFarCost : kTriCost;
        if (m.st->go || range || (int64_t)B64 > m.nF || (int64_t)B64 > kCycMaxEdges ||
            (m.W && caps_cost_more(m, (int64_t)B64, (double)B64 * least))) {
            if (tid == 0) atomicMax(&m.st->go, 2);
            continue;
        }
        const int B = (int)B64;
        if (B == 0) continue;
        if (!m.W) {  // the edges are all that is wanted
            __syncthreads();
            for (int64_t u = tid / kUnitLanes; u < units; u += kCapThreads / kUnitLanes) {
                const int n = m.blk[2 * u], at = m.blk[2 * u + 1];
                for (int x = tid % kUnitLanes; x < n; x += kUnitLanes) {
                    int32_t a, b;
                    half_edge(m, m.list[u * kCycUnit + x], a, b);
                    m.edge[at + x] = make_int2(a, b);
                }
            }
            if (tid == 0) m.st->n_rec = B;
            continue;
        }
        int n_tri = 0, n_short = 0;
        // (a lambda's two instances, so that LDS is addressed as LDS)
        auto join = [&](int2 *edge, int32_t *nout, int32_t *nin, int32_t *rank, int32_t *next, int32_t *succ,
                        int32_t *same, int32_t *into) -> int {
            __syncthreads();
            for (int64_t u = tid / kUnitLanes; u < units; u += kCapThreads / kUnitLanes) {
                const int n = m.blk[2 * u], at = m.blk[2 * u + 1];
                for (int x = tid % kUnitLanes; x < n; x += kUnitLanes) {
                    int32_t a, b;
                    half_edge(m, m.list[u * kCycUnit + x], a, b);
                    edge[at + x] = make_int2(a, b);
                }
            }
            __syncthreads();
            for (int i = tid; i < B; i += kCapThreads) {
                const int2 e = edge[i];
                nout[i] = atomicExch(&m.hout[e.x], i);
                nin[i] = atomicExch(&m.hin[e.y], i);
            }
            __syncthreads();
            // the chains' heads by edge: those leaving its end and its start, and those entering its end
            for (int i = tid; i < B; i += kCapThreads) {
                const int2 e = edge[i];
                succ[i] = m.hout[e.y];
                same[i] = m.hout[e.x];
                into[i] = m.hin[e.y];
            }
            __syncthreads();
            const int limit = degree_limit(B);
            // the lowest triangle (by its edges in increasing order) that edge i is part of
            auto triangle = [&](int i, int &to) -> unsigned long long {
                const int2 e = edge[i];
                unsigned long long best = ~0ull;
                int steps = 0;
                for (int j = succ[i]; j >= 0; j = nout[j])
                    for (int k = succ[j]; k >= 0; k = nout[k]) {
                        if (++steps > limit) {
                            s_bad = 1;
                            return best;
                        }
                        if (edge[k].y != e.x) continue;
                        const int lo = min(i, min(j, k)), hi = max(i, max(j, k)), mid = i + j + k - lo - hi;
                        const unsigned long long id = (unsigned long long)lo << 40 | (unsigned long long)mid << 20 | hi;
                        if (id < best) {
                            best = id;
                            to = j;
                        }
                    }
                return best;
            };
            for (int i = tid; i < B; i += kCapThreads) {
                if (*(volatile int32_t *)&s_bad) break;
                int j = -1, k = -1, x = -1;
                const unsigned long long id = triangle(i, j);
                // a loop if its other two edges choose it as well
                const bool loop = id != ~0ull && triangle(j, k) == id && triangle(k, x) == id;
                next[i] = loop ? j : -1;
            }
            __syncthreads();
            for (int i = tid; i < B; i += kCapThreads) {
                int ro = 0, ri = 0, steps = 0;
                for (int k = same[i]; k >= 0 && steps < limit; k = nout[k], ++steps)
                    ro += k < i && next[k] < 0;
                for (int k = into[i]; k >= 0 && steps < limit; k = nin[k], ++steps)
                    ri += k < i && next[k] < 0;
                if (steps >= limit) s_bad = 1;
                rank[i] = ro | (ri << 16);
            }
            __syncthreads();
            int32_t *len = nin;
            for (int i = tid; i < B; i += kCapThreads) {
                int to = next[i];
                if (to < 0) {
                    const int want = rank[i] >> 16;
                    int steps = 0;
                    for (int k = succ[i]; k >= 0 && steps < limit; k = nout[k], ++steps)
                        if (next[k] < 0 && (rank[k] & 0xffff) == want) to = k;
                    if (to < 0) s_bad = 1;
                }
                len[i] = to;  // the others still read next[]
            }
            __syncthreads();
            for (int i = tid; i < B; i += kCapThreads) next[i] = len[i];
            __syncthreads();
            if (s_bad) return -1;
            // each edge's loop (its lowest edge) and place in it, counted from there; the loop's length at its
            // lowest edge
            int32_t *lead = into, *place = nin, *size = nout;
            bool any_long = false;
            unsigned long long kinds = 0;  // edges of each kind of loop
            for (int i = tid; i < B; i += kCapThreads) {
                int n = 1, lo = i, at = 0, j = next[i];
                for (; j != i && n < kWalk; j = next[j], ++n)
                    if (j < lo) {
                        lo = j;
                        at = n;
                    }
                const bool closed = j == i;
                any_long = any_long || !closed;
                kinds += 1ull << (21 * loop_kind(n));
                lead[i] = lo;
                place[i] = closed ? (at == 0 ? 0 : n - at) : -1;
                size[i] = n;
            }
            if (!m.grid.order) {
                block_scan(kinds, red, kinds);
                if (caps_cost_more(m, B, plain_cost(count_of(kinds, 0), count_of(kinds, 1), count_of(kinds, 2)))) return -1;
            }
            // Long loops by doubling: log2 of the length rounds over their edges (each edge walking to a
            // lower one was quadratic, 1.2e6 dependent loads for a ribbon of 1e5 faces).
            if (__syncthreads_or(any_long)) {
                // x[0] the edge 2^k further on and x[1] the lowest edge before that.  Where a round
                // changes no minimum, each is its loop's: it is the same after 2^k steps, and so after
                // gcd(2^k, length), and the 2^k edges that it covers come to every such rest.
                int32_t *x[2] = {succ, same}, *y[2] = {rank, size};
                auto rounds = [&](auto step) {
                    for (int k = 0; k < 21; ++k) {
                        bool more = false;
                        for (int i = tid; i < B; i += kCapThreads)
                            if (place[i] < 0) more = step(i) || more;
                        more = __syncthreads_or(more);
                        for (int d = 0; d < 2; ++d) {
                            int32_t *const z = x[d];
                            x[d] = y[d];
                            y[d] = z;
                        }
                        if (!more) break;
                    }
                };
                for (int i = tid; i < B; i += kCapThreads)
                    if (place[i] < 0) {
                        x[0][i] = next[i];
                        x[1][i] = i;
                    }
                __syncthreads();
                rounds([&](int i) {
                    const int j = x[0][i], a = x[1][i], b = x[1][j];
                    y[0][i] = x[0][j];
                    y[1][i] = min(a, b);
                    return b < a;
                });
                for (int i = tid; i < B; i += kCapThreads)
                    if (place[i] < 0) lead[i] = x[1][i];
                __syncthreads();
                // x[0] an edge further on, the last of the loop in the end, and x[1] the steps to it
                for (int i = tid; i < B; i += kCapThreads)
                    if (place[i] < 0) {
                        const bool end = next[i] == lead[i];
                        x[0][i] = end ? i : next[i];
                        x[1][i] = !end;
                    }
                __syncthreads();
                rounds([&](int i) {
                    const int j = x[0][i], to = x[0][j];
                    y[0][i] = to;
                    y[1][i] = x[1][i] + x[1][j];
                    return to != j;
                });
                for (int i = tid; i < B; i += kCapThreads)
                    if (place[i] < 0) next[i] = x[1][lead[i]] - x[1][i];
                __syncthreads();
                for (int i = tid; i < B; i += kCapThreads)
                    if (place[i] < 0) {
                        if (lead[i] == i) size[i] = x[1][i] + 1;
                        place[i] = next[i];
                    }
                __syncthreads();
            }
            int32_t *off = rank;
            unsigned long long done = 0;  // records of each kind
            for (int i0 = 0; i0 < B; i0 += kCapThreads) {
                const int i = i0 + tid;
                const int n = i < B && lead[i] == i ? size[i] : 0, kind = loop_kind(n);
                unsigned long long all;
                const unsigned long long at = done + block_scan((unsigned long long)n << (21 * kind), red, all);
                if (n) off[i] = count_of(at, kind);
                done += all;
            }
            const int first[3] = {0, count_of(done, 0), count_of(done, 0) + count_of(done, 1)};
            if (first[2] + count_of(done, 2) != B) return -1;  // not a permutation (cannot be)
            __syncthreads();
            for (int i = tid; i < B; i += kCapThreads) {
                const int k = size[lead[i]], pos = zigzag(place[i], k), at = off[lead[i]] + first[loop_kind(k)] + pos;
                m.cvid[at] = edge[i].x;
                m.cpos[at] = pos;
            }
            n_tri = first[1] / 3;
            n_short = first[2];
            return 0;
        };
        const int bad = B <= kCapLds ? join(s_edge, s_work[0], s_work[1], s_work[2], s_work[3], s_work[4], s_work[5], s_work[6])
                                     : join(m.edge, m.nout, m.nin, m.rank, m.next, m.cvid, m.cpos,
                                            reinterpret_cast<int32_t *>(m.caps));  // (written later)
        if (bad) {
            if (tid == 0) atomicMax(&m.st->go, 2);
            continue;
        }
        __syncthreads();
        // triangles over many columns go on the raster list; k_cyc_slabs takes the others one by one
        unsigned long long cost = 0, columns = 0;
        const float *V = m.V;
        int32_t *cvid = m.cvid, *cpos = m.cpos;
        const int share = kListShare / B;
        const bool blocks = m.grid.order != 0 && n_short < B;
        const CloseCost close(m);
        const double limit = m.bins ? (double)m.bins * m.bins : (double)m.n0 * m.ps.n1;
        for (int x = tid; x < B; x += kCapThreads) {
            if (cpos[x] < 2) continue;
            float p[3][3];
            for (int k = 0; k < 3; ++k) {
                const int64_t v = 3 * (int64_t)cvid[x - 2 + k];
                for (int d = 0; d < 3; ++d) p[k][d] = V[v + d];
            }
            if (blocks && x >= n_short) cost += close(p);
            double area = 1.0;
            for (int d = 0; d < 2; ++d) {
                const float l = fminf(fminf(p[0][d], p[1][d]), p[2][d]), u = fmaxf(fmaxf(p[0][d], p[1][d]), p[2][d]);
                area *= ((double)u - l) * (m.bins ? Bins(m).inv[d] : m.inv_h[d]) + 1.0;
            }
            columns += (unsigned long long)fmin(area, limit);
            if (area > (double)kWaveColumns) {
                RasterFace f;
                if (share > 0 && set_cap(m, x, f) && f.columns() > 0) {
                    add_slabs(m, (int32_t)(m.nF + x), f.columns(), share);
                    cpos[x] |= kCapListed;
                }
            }
        }
        if (blocks) block_scan(cost, red, cost);
        block_scan(columns, red, columns);
        if (caps_cost_more(m, B, m.grid.order ? (double)cost + (double)B * kFarCost : plain_cost(3 * n_tri, n_short - 3 * n_tri, B - n_short), (double)columns)) {
            if (tid == 0) atomicMax(&m.st->go, 2);
        } else if (tid == 0) {
            m.st->n_rec = B;
            m.st->n_tri = n_tri;
            m.st->n_short = n_short;
        }
    }
}

// One wave per entry of the raster list, one column per lane, and one per record of the caps:
// it writes the record and its triangle, and takes the triangle's columns unless they are on the
// list.  (One workgroup formed all of them, in FP64: 55 us for 1364 boundary edges.)
__global__ __launch_bounds__(kCycUnit) void k_cyc_slabs(const char *table) {
    const CycHead *h = reinterpret_cast<const CycHead *>(table);
    const CycMesh *meshes = meshes_of(table);
    const int lane = threadIdx.x & 63;
    const int64_t waves = (int64_t)gridDim.x * (kCycUnit / 64);
    const int64_t wave = __builtin_amdgcn_readfirstlane((int)blockIdx.x * (kCycUnit / 64) + (int)(threadIdx.x >> 6));
    int64_t before = 0;
    for (int mi = 0; mi < h->n; ++mi) {
        const CycMesh &m = meshes[mi];
        const int64_t n = (unsigned)m.st->n_slab;
        if (m.st->go) continue;
        const int n_tri = m.st->n_tri, n_rec = m.st->n_rec;
        for (int64_t x = (wave + waves - before % waves) % waves; x < n + n_rec; x += waves) {
            RasterFace r;
            int sign = 1;
            int64_t first = 0, end = 0;  // of the columns
            if (x >= n) {
                const int at = (int)(x - n), cpos = m.cpos[at], pos = cpos & ~kCapListed;
                const float *p = m.V + 3 * (int64_t)m.cvid[at];
                VRec rec;
                rec.p = make_float4(p[0], p[1], p[2], 0.0f);
                rec.n = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
                TriRec t{};
                t.far = -1.0f;  // no triangle
                if (pos >= 2 && set_cap(m, at, r)) {
                    rec.n = make_float4((float)r.nx, (float)r.ny, (float)r.nz, 0.0f);
                    rec.p.w = 1.0f;
                    t = tri_record(r);
                    if (cpos == pos) end = r.columns();
                }
                if (lane == 0) {
                    m.caps[at] = rec;
                    if (at >= 3 * n_tri || pos == 2) {
                        const int slot = at >= 3 * n_tri ? at - 2 * n_tri : at / 3;
                        m.tri[slot] = t;
                        m.tri0[slot] = make_float4(t.v[0], t.v[1], t.v[2], t.far);
                    }
                }
                sign = -1;
            } else {
                const int2 e = m.slab[x];
                int share;
                if (e.x >= m.nF) {
                    set_cap(m, (int)(e.x - m.nF), r);
                    share = kListShare / n_rec;
                    sign = -1;
                } else {
                    const int64_t f = e.x;
                    share = face_share(m);
                    r.set(m, m.V + 3 * (int64_t)face_vertex(m, 3 * f), m.V + 3 * (int64_t)face_vertex(m, 3 * f + 1),
                          m.V + 3 * (int64_t)face_vertex(m, 3 * f + 2));
                }
                const int64_t per = list_columns(r.columns(), share);
                first = e.y * per;
                end = min(first + per, r.columns());
            }
            const int64_t nj = r.j1 - r.j0 + 1;
            for (int64_t c = first + lane; c < end; c += 64)
                r.column(m, sign, r.i0 + (int)(c / nj), r.j0 + (int)(c % nj));
        }
        before += n + n_rec;
    }
}

// Puts a voxel on the list, with one atomic on its length for the lanes that come here together.  `go`: of the
// state, as the kernel found it; a list that is full by then is not counted on.  (4e5 voxels beyond its end took
// 6 ms one by one.)
__device__ __forceinline__ void list_near(const CycMesh &m, int64_t idx, int go) {
    const int32_t x = (int32_t)(idx - m.p0);
    const uint32_t bit = 1u << (x & 31);
    if ((atomicOr(&m.mark[x >> 5], bit) & bit) || go) return;
    const unsigned long long all = __builtin_amdgcn_ballot_w64(true);
    const int leader = __builtin_ctzll(all), lane = threadIdx.x & 63, n = __popcll(all);
    int32_t at = 0;
    if (lane == leader) {
        at = atomicAdd(&m.st->n_near, n);
        if (at + n > m.near_cap) atomicMax(&m.st->go, 1);
    }
    at = __builtin_amdgcn_readlane(at, leader) + __popcll(all & ((1ull << lane) - 1ull));
    if (at < m.near_cap) m.near[at] = x;
}

// Where the occupancy map amplifies the rounding of W: within rounding of a threshold, and
// on the slope of a steep sigmoid (k |dW| there, in the loss gradients that follow as
// well, against W's own 1e-6).  Such voxels take the direct sum, so that the map's outcome does not depend
// on the path.  They lie around the holes: 0.2 % of the voxels of a mesh with 5 % of its faces missing.
__device__ __forceinline__ bool near_threshold(const OccParams &o, float w) {
    const float d = __builtin_fabsf(w - o.tau);
    if (o.mode == WN_OCC_THRESHOLD) return d < 1.0e-5f;
    return o.mode == WN_OCC_SIGMOID && o.k > 10.0f && d < fminf(10.0f / o.k, 0.25f);
}

// The blocks' weights of a mesh: [3][kBlockSide][kFine] of the fine nodes at the voxels, then
// [3][kFine][kCoarse] of the coarse nodes at the fine ones.
constexpr int kFineWeights = 3 * kBlockSide * kFine, kWeights = kFineWeights + 3 * kFine * kCoarse;

__device__ __forceinline__ void write_weights(const CycMesh &m) {
    const CycBlocks &g = m.grid;
    for (int e = threadIdx.x; e < kWeights; e += blockDim.x) {
        float w = 0.0f;
        if (e < kFineWeights) {
            const int d = e / (kBlockSide * kFine), i = e / kFine % kBlockSide, j = e % kFine;
            if (i < g.size[d] && j < g.fine[d]) w = node_weight(kFine, g.size[d], (float)i, j);
        } else {
            const int x = e - kFineWeights, d = x / (kFine * kCoarse), i = x / kCoarse % kFine, j = x % kCoarse;
            if (i < g.fine[d] && j < g.coarse[d]) w = node_weight(kCoarse, g.size[d], node_at(kFine, g.size[d], i), j);
        }
        m.weight[e] = w;
    }
}

// One wave per column, or for as many short ones as it has lanes for, from the top: W is the sum of the crossings
// at and above a voxel.  (A wave for each column of one voxel took 1.56 ms for 2000 x 2000 x 1.)
__global__ __launch_bounds__(kCycColumns * 64) void k_cyc_columns(const char *table) {
    const CycHead *h = reinterpret_cast<const CycHead *>(table);
    const int lane = threadIdx.x & 63;
    for (int64_t u = blockIdx.x; u < h->u_col; u += gridDim.x) {
        const CycMesh &m = *find_mesh<&CycMesh::u_col>(table, u);
        if (u == m.u_col && m.grid.order) write_weights(m);
        const int go = m.st->go, n_rec = m.st->n_rec;
        if (go >= 2) continue;  // (the all-pairs kernels write every voxel)
        const bool last = n_rec == 0;  // no caps to add
        if (m.bins) {
            const int64_t idx = (u - m.u_col) * (kCycColumns * 64) + threadIdx.x;
            if (idx >= m.P) continue;
            const uint32_t x = reinterpret_cast<const uint32_t *>(m.W)[idx];
            const float w = (float)((int)(x & ~kCloseBit) - (int)kCountBias);
            m.W[idx] = w;
            if (last) write_occ(m.occ, idx, w);
            if ((x & kCloseBit) || (last && near_threshold(m.occ, w))) list_near(m, idx, go);
            continue;
        }
        const int n2 = m.ps.n2, per = m.per, n = per * n2;
        const int64_t base = (m.p0 / n2 + ((u - m.u_col) * kCycColumns + (threadIdx.x >> 6)) * per) * n2;
        const int64_t lo = base > m.p0 ? base : m.p0;
        const int64_t hi = base + n < m.p0 + m.P ? base + n : m.p0 + m.P;
        int below = lane;  // voxels of its column that this pass has above the lane's
        if (per > 1) below = lane % n2;
        int carry = 0;
        for (int64_t top = per > 1 ? base + n : hi; top > lo; top -= 64) {
            const int64_t idx = top - 1 - lane;  // lane 0 is the highest voxel
            const bool live = idx >= lo && idx < hi;
            const uint32_t x = live ? reinterpret_cast<const uint32_t *>(m.W)[idx] : kCountBias;
            int s = (int)(x & ~kCloseBit) - (int)kCountBias;
            for (int o = 1; o < 64; o <<= 1) {
                const int y = __shfl_up(s, o);
                if (below >= o) s += y;
            }
            s += carry;
            carry = __shfl(s, 63);
            if (!live) continue;
            const float w = (float)s;
            m.W[idx] = w;
            bool near = (x & kCloseBit) != 0u;
            if (last) {
                write_occ(m.occ, idx, w);
                near = near || near_threshold(m.occ, w);
            }
            if (near) list_near(m, idx, go);
        }
    }
}

// ------------------------------------------------------------------ caps' solid angles

constexpr int kTriBlock = 16;   // triangles per compensated sum
constexpr int kLongBlock = 8;  // records of long loops per compensated sum

struct Slot64 {
    double x, y, z, r, dprev, rprev;
};

__device__ __forceinline__ void enter64(const float4 v, const Slot64 &B, Slot64 &C, double qx, double qy, double qz) {
    C.x = (double)v.x - qx;
    C.y = (double)v.y - qy;
    C.z = (double)v.z - qz;
    const double d = C.x * C.x + C.y * C.y + C.z * C.z;
    const double y = __builtin_amdgcn_rsq(d), g = d * y;  // one Newton step on the hardware's estimate
    C.r = d > 0.0 ? __builtin_fma(g, __builtin_fma(-0.5 * y, g, 0.5), g) : 0.0;
    C.dprev = B.x * C.x + B.y * C.y + B.z * C.z;
    C.rprev = B.r * C.r;
}

__device__ __forceinline__ float half_angle64(const float4 n, const Slot64 &A, const Slot64 &B, const Slot64 &C) {
    const double dca = C.x * A.x + C.y * A.y + C.z * A.z;
    const double pr = B.rprev * C.r;
    const double be = pr + B.dprev * C.r + C.dprev * A.r + dca * B.r;
    const double al = A.x * n.x + A.y * n.y + A.z * n.z;
    // any positive factor common to both will do: the approximate reciprocal keeps them in FP32's range
    const double scale = pr > 0.0 ? __builtin_amdgcn_rcp(pr) : 0.0;
    return atan2_eq8((float)(al * scale), (float)(be * scale));
}

// Long loops: the strips of a long loop hold thin triangles as long as the loop is wide, whose
// terms near their two long edges lose half their digits in FP32 (beta cancels
// to the product of two small angles); they are formed in FP64.  Every record completes a triangle, so this
// costs about twice an FP32 strip record; boundaries are a small part of a mesh.
__device__ __forceinline__ float add_long(const VRec *__restrict__ recs, int n, Slot64 &A, Slot64 &B, Slot64 &C,
                                          float qx, float qy, float qz) {
    const double x = qx, y = qy, z = qz;
    float ts = 0.0f;
    for (int i = 0; i < n; ++i) {
        const float4 p = recs[i].p, nn = recs[i].n;
        A = B;
        B = C;
        enter64(p, B, C, x, y, z);
        if (p.w != 0.0f) ts += half_angle64(nn, A, B, C);
    }
    return ts;
}

__device__ __forceinline__ void sum_long(const VRec *__restrict__ recs, int n, float qx, float qy, float qz, float &s,
                                         float &c) {
    Slot64 A{}, B{}, C{};
    for (int i = 0; i < n; i += kLongBlock)
        neumaier_add(s, c, add_long(recs + i, min(n - i, kLongBlock), A, B, C, qx, qy, qz));
}

// Three cap records that complete a triangle, as scalars.
struct CapRecords {
    float4 p0, p1, p2, n;

    __device__ __forceinline__ explicit CapRecords(const VRec *r) {
        typedef float Rec __attribute__((ext_vector_type(8)));
        typedef const __attribute__((address_space(4))) Rec *ConstRec;
        static_assert(sizeof(Rec) == sizeof(VRec), "one scalar load");
        ConstRec c = (ConstRec)(uintptr_t)r;
        const Rec a = c[0], b = c[1], d = c[2];
        p0 = make_float4(a[0], a[1], a[2], a[3]);
        p1 = make_float4(b[0], b[1], b[2], b[3]);
        p2 = make_float4(d[0], d[1], d[2], d[3]);
        n = make_float4(d[4], d[5], d[6], d[7]);
    }
    // Its half solid angle at (x, y, z), as the all-pairs kernel forms a lone face.
    __device__ __forceinline__ float angle(float x, float y, float z) const {
        const float qx[1] = {x}, qy[1] = {y}, qz[1] = {z};
        Slot<1> A, B, C;
        C.x[0] = C.y[0] = C.z[0] = C.r[0] = 0.0f;
        float ts[1] = {0.0f};
        push_record<1>(p0, false, n, B, C, A, qx, qy, qz, ts);
        push_record<1>(p1, false, n, C, A, B, qx, qy, qz, ts);
        push_record<1>(p2, true, n, A, B, C, qx, qy, qz, ts);
        return ts[0];
    }
    // In FP64, for the triangles of long loops.
    __device__ __forceinline__ float angle64(float x, float y, float z) const {
        Slot64 A{}, B{}, C{};
        enter64(p0, C, A, (double)x, (double)y, (double)z);
        enter64(p1, A, B, (double)x, (double)y, (double)z);
        enter64(p2, B, C, (double)x, (double)y, (double)z);
        return half_angle64(n, A, B, C);
    }
};

// Sum over the n triangles.  A triangle's 64 bytes come through the scalar cache
// and are used as scalar operands: 35 VALU and 4 transcendentals per far pair, against 52
// and 3.5 for a face of three records (the edge vectors replace two of the three
// subtractions and norms, and a small angle needs three terms of its series).  A point that is
// near uses the exact forms, whatever the points of its wave do, so that its
// value does not depend on them.
// Half solid angle of a far triangle: q = |R|^2, s1 = R . 2 d_1, s2 = R . 2 d_2, al = R . n.
__device__ __forceinline__ float far_angle(float q, float s1, float s2, float al, float d11, float d22, float d12) {
    const float r0 = fast_sqrt(q), r1 = fast_sqrt((q + d11) + s1), r2 = fast_sqrt((q + d22) + s2);
    const float p01 = __builtin_fmaf(0.5f, s1, q), p02 = __builtin_fmaf(0.5f, s2, q);
    const float p12 = p01 + __builtin_fmaf(0.5f, s2, d12);
    const float be = __builtin_fmaf(p12, r0, __builtin_fmaf(p02, r1, __builtin_fmaf(p01, r2, (r0 * r1) * r2)));
    const float t = al * __builtin_amdgcn_rcpf(be);
    const float t2 = t * t;
    return t * __builtin_fmaf(t2, __builtin_fmaf(t2, 0.2f, -0.333333333f), 1.0f);
}

// Adds the triangles [0, n) from rec on, their records at caps.  rec moves on; next is one ahead.
typedef float TriVec __attribute__((ext_vector_type(16)));
typedef const __attribute__((address_space(4))) TriVec *ConstTri;
static_assert(sizeof(TriVec) == sizeof(TriRec), "one scalar load");

template <int PPL>
__device__ __forceinline__ void add_triangles(ConstTri &rec, TriVec &next, const VRec *caps, int n,
                                              const float (&qx)[PPL], const float (&qy)[PPL], const float (&qz)[PPL],
                                              float (&ts)[PPL]) {
#pragma unroll 1
    for (int i = 0; i < n; ++i) {
        const TriVec r = next;
        next = *++rec;
        __builtin_amdgcn_sched_barrier(0);  // the load goes out before this triangle's arithmetic
        float v[PPL];
        bool near[PPL], any = false;
#pragma unroll
        for (int p = 0; p < PPL; ++p) {
            const float x = r[0] - qx[p], y = r[1] - qy[p], z = r[2] - qz[p];
            const float q = __builtin_fmaf(z, z, __builtin_fmaf(y, y, x * x));
            const float s1 = __builtin_fmaf(z, r[6], __builtin_fmaf(y, r[5], x * r[4]));
            const float s2 = __builtin_fmaf(z, r[10], __builtin_fmaf(y, r[9], x * r[8]));
            const float al = __builtin_fmaf(z, r[14], __builtin_fmaf(y, r[13], x * r[12]));
            v[p] = far_angle(q, s1, s2, al, r[7], r[11], r[15]);
            near[p] = q < r[3];
            any = any || near[p];
        }
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(any) != 0ull, 0)) {
            const CapRecords r3(caps + 3 * i);
#pragma unroll
            for (int p = 0; p < PPL; ++p)
                if (near[p]) v[p] = r3.angle(qx[p], qy[p], qz[p]);
        }
#pragma unroll
        for (int p = 0; p < PPL; ++p) ts[p] += v[p];
    }
}

template <int PPL>
__device__ __forceinline__ void sum_triangles(const TriRec *tri, const VRec *caps, int n, const float (&qx)[PPL],
                                              const float (&qy)[PPL], const float (&qz)[PPL], float (&s)[PPL],
                                              float (&c)[PPL]) {
    ConstTri rec = (ConstTri)(uintptr_t)tri;
    TriVec next = *rec;  // one ahead; the array holds one more than it has triangles
    for (int i0 = 0; i0 < n; i0 += kTriBlock) {
        float ts[PPL];
#pragma unroll
        for (int p = 0; p < PPL; ++p) ts[p] = 0.0f;
        add_triangles<PPL>(rec, next, caps + 3 * i0, min(n - i0, kTriBlock), qx, qy, qz, ts);
#pragma unroll
        for (int p = 0; p < PPL; ++p) neumaier_add(s[p], c[p], ts[p]);
    }
}

// A value that is the same in every lane, as a scalar.
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }
template <typename T>
__device__ __forceinline__ T *uniform(T *p) {
    const uint64_t a = reinterpret_cast<uint64_t>(p);
    const uint32_t lo = (uint32_t)uniform((int)(uint32_t)a), hi = (uint32_t)uniform((int)(uint32_t)(a >> 32));
    return reinterpret_cast<T *>((uint64_t)hi << 32 | lo);
}

__device__ __forceinline__ void add_caps(const CycMesh &m, int64_t at, float sum, int go) {
    const float w = m.W[at] + sum * kInv2Pi;
    m.W[at] = w;
    write_occ(m.occ, at, w);
    if (near_threshold(m.occ, w)) list_near(m, at, go);
}

template <int PPL>
__global__ __launch_bounds__(kBlock) void k_cyc_sum(const char *table) {
    __shared__ float4 tile[kRecTile * 4];
    __shared__ unsigned long long s_unit;
    __shared__ int32_t s_go;
    CycHead *h = reinterpret_cast<CycHead *>(const_cast<char *>(table));
    const int tid = threadIdx.x;
    const int64_t units = h->u_sum;
    for (int64_t u = blockIdx.x; u < units;) {
        const CycMesh &m = *uniform(find_mesh<&CycMesh::u_sum>(table, u));
        const int n_rec = uniform(m.st->n_rec), n_tri = uniform(m.st->n_tri), n_short = uniform(m.st->n_short);
        const VRec *caps = uniform(m.caps);
        if (tid == 0) s_go = m.st->go;  // other workgroups may set it meanwhile
        __syncthreads();
        if (s_go < 2 && n_rec > 0) {
            const int64_t base = (u - m.u_sum) * (kBlock * PPL) + tid;
            float qx[PPL], qy[PPL], qz[PPL], s[PPL], c[PPL];
#pragma unroll
            for (int p = 0; p < PPL; ++p) {
                int64_t idx = base + (int64_t)p * kBlock;
                idx = idx < m.P ? idx : m.P - 1;
                m.ps.get(m.p0 + idx, qx[p], qy[p], qz[p]);
                s[p] = c[p] = 0.0f;
            }
            sum_triangles<PPL>(uniform(m.tri), caps, n_tri, qx, qy, qz, s, c);
            sum_records<PPL, 2>(reinterpret_cast<const float4 *>(caps + 3 * n_tri), 0, n_short - 3 * n_tri, tile,
                                qx, qy, qz, s, c);
            if (n_rec > n_short) {
#pragma unroll
                for (int p = 0; p < PPL; ++p)
                    sum_long(caps + n_short, n_rec - n_short, qx[p], qy[p], qz[p], s[p], c[p]);
            }
#pragma unroll
            for (int p = 0; p < PPL; ++p) {
                const int64_t idx = base + (int64_t)p * kBlock;
                if (idx >= m.P) continue;
                add_caps(m, m.p0 + idx, s[p] + c[p], s_go);
            }
        }
        if (units <= gridDim.x) break;
        __syncthreads();
        if (tid == 0) s_unit = atomicAdd(&h->cursor, 1ull) + gridDim.x;
        __syncthreads();
        u = (int64_t)s_unit;
    }
}

// The same for few points: one workgroup per 64 points, its waves a block of the caps each
// (16 triangles, a tile of records, or 8 records of long loops).  The blocks' sums meet in
// LDS and are added in the caps' order, so the bits are k_cyc_sum's.  There, 12818 points
// are 200 waves with all caps in turn: 171 us for 8300 faces of which 6 % are missing, 27 here.
constexpr int kSplitRounds = 8;  // blocks per wave between two barriers

template <int kWaves>
__global__ __launch_bounds__(kWaves * 64) void k_cyc_sum_split(const char *table) {
    __shared__ float4 tiles[kWaves][2 * kRecTile];
    __shared__ float s_block[kWaves * kSplitRounds][64];
    __shared__ int32_t s_go;
    const int64_t units = reinterpret_cast<const CycHead *>(table)->u_sum;
    const int wave = uniform((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    for (int64_t u = blockIdx.x; u < units; u += gridDim.x) {
        const CycMesh &m = *uniform(find_mesh<&CycMesh::u_sum>(table, u));
        const int n_rec = uniform(m.st->n_rec), n_tri = uniform(m.st->n_tri), n_short = uniform(m.st->n_short);
        const VRec *caps = uniform(m.caps);
        __syncthreads();
        if (threadIdx.x == 0) s_go = m.st->go;  // other workgroups may set it meanwhile
        __syncthreads();
        if (s_go >= 2 || n_rec == 0) continue;
        const int64_t idx = (u - m.u_sum) * 64 + lane;
        float qx[1], qy[1], qz[1], s = 0.0f, c = 0.0f;
        m.ps.get(m.p0 + (idx < m.P ? idx : m.P - 1), qx[0], qy[0], qz[0]);
        const float4 *strips = reinterpret_cast<const float4 *>(caps + 3 * n_tri);
        const int n_strip = n_short - 3 * n_tri, n_long = n_rec - n_short;
        const int b_tri = (n_tri + kTriBlock - 1) / kTriBlock, b_strip = b_tri + (n_strip + kRecTile - 1) / kRecTile;
        const int blocks = b_strip + (n_long + kLongBlock - 1) / kLongBlock;
        for (int b0 = 0; b0 < blocks; b0 += kWaves * kSplitRounds) {
            const int b1 = min(blocks - b0, kWaves * kSplitRounds);
            for (int k = wave; k < b1; k += kWaves) {
                const int b = b0 + k;
                float ts[1] = {0.0f};
                if (b < b_tri) {
                    const int i = b * kTriBlock;
                    ConstTri rec = (ConstTri)(uintptr_t)uniform(m.tri + i);
                    TriVec next = *rec;
                    add_triangles<1>(rec, next, caps + 3 * i, min(n_tri - i, kTriBlock), qx, qy, qz, ts);
                } else if (b < b_strip) {
                    const int r = (b - b_tri) * kRecTile, nt = min(n_strip - r, kRecTile);
                    float4 *tile = tiles[wave];
                    __builtin_amdgcn_wave_barrier();
                    for (int x = lane; x < 2 * nt; x += 64) tile[x] = strips[2 * r + x];
                    __builtin_amdgcn_wave_barrier();
                    Slot<1> S0, S1, S2;
                    prime_window<1>(strips, r, S0, S1, S2, qx, qy, qz);
                    sum_tile<1>(tile, nt, tile_face_mask(tile, nt), S0, S1, S2, qx, qy, qz, ts);
                } else {
                    const int r = (b - b_strip) * kLongBlock;
                    const VRec *recs = caps + n_short;
                    Slot64 A{}, B{}, C{};
                    if (r > 0) {
                        enter64(recs[r - 2].p, A, B, (double)qx[0], (double)qy[0], (double)qz[0]);
                        enter64(recs[r - 1].p, B, C, (double)qx[0], (double)qy[0], (double)qz[0]);
                    }
                    ts[0] = add_long(recs + r, min(n_long - r, kLongBlock), A, B, C, qx[0], qy[0], qz[0]);
                }
                s_block[k][lane] = ts[0];
            }
            __syncthreads();
            if (wave == 0)
                for (int k = 0; k < b1; ++k) neumaier_add(s, c, s_block[k][lane]);
            __syncthreads();
        }
        if (wave == 0 && idx < m.P) add_caps(m, m.p0 + idx, s + c, s_go);
    }
}

// ------------------------------------------------------------------ caps, blocks of voxels

// A triangle's solid angle is smooth away from it, so a block of voxels takes those of the far
// triangles at a few Chebyshev nodes (k_cyc_nodes) and interpolates their sum (k_cyc_blocks, which
// adds the near ones at every voxel).  With a the block's half side, t = D / a its
// distance from a triangle of edge e, and rho = t + sqrt(t^2 + 1) (the interpolation of a
// function that is analytic to the distance D from an interval converges as rho^-order), the
// error is about 0.04 e^2 / D^2 (a triangle's share of W there) rho^-order: against FP64, random
// triangles were off by at most 10 times and on average 0.2 times that.  A triangle is far
// where this is below kFarError and where its far form holds at all nodes; where it is
// below kCoarseError with kCoarse nodes per axis, it takes those (most triangles do, so their errors
// add up: 4e-9 gave 6e-7 of W over 46000 faces with 8 % missing, the all-pairs sum's own error;
// 1e-9 gives 2.4e-7).
//
// One wave per split of the triangles and 64 nodes of a block: the coarse ones, or 64 of the
// fine ones.
__global__ __launch_bounds__(64) void k_cyc_nodes(const char *table) {
    const int64_t units = reinterpret_cast<const CycHead *>(table)->u_node;
    const int lane = threadIdx.x;
    for (int64_t u = blockIdx.x; u < units; u += gridDim.x) {
        const CycMesh &m = *uniform(find_mesh<&CycMesh::u_node>(table, u));
        if (uniform(m.st->go) >= 2) continue;
        const int n = uniform(m.st->n_rec - 2 * m.st->n_tri);
        if (n == 0) continue;
        const CycBlocks &g = m.grid;
        const int nc = g.coarse[0] * g.coarse[1] * g.coarse[2], nf = g.fine[0] * g.fine[1] * g.fine[2];
        const int waves = 1 + (nf + 63) / 64;
        const int64_t y = (u - m.u_node) / g.splits, b = y / waves;
        const int split = uniform((int)(u - m.u_node - y * g.splits)), part = uniform((int)(y - b * waves));
        int i0[3];
        block_origin(m, b, i0);
        const Block box(m, i0);
        const int *nodes = part == 0 ? g.coarse : g.fine;
        const int order = part == 0 ? kCoarse : kFine, want = part == 0 ? 2 : 1;
        const int j = part == 0 ? lane : (part - 1) * 64 + lane, nn = part == 0 ? nc : nf;
        const int jn = min(j, nn - 1), j0 = jn / (nodes[1] * nodes[2]), jr = jn - j0 * nodes[1] * nodes[2];
        const int j1 = jr / nodes[2], j2 = jr - j1 * nodes[2];
        const float qx = __builtin_fmaf(node_at(order, g.size[0], j0), m.ps.h[0], box.lo[0]);
        const float qy = __builtin_fmaf(node_at(order, g.size[1], j1), m.ps.h[1], box.lo[1]);
        const float qz = __builtin_fmaf(node_at(order, g.size[2], j2), m.ps.h[2], box.lo[2]);
        const TriRec *tri = uniform(m.tri);
        const float4 *tri0 = uniform(m.tri0);
        const int words = (n + 63) / 64, w1 = uniform((int)((int64_t)words * (split + 1) / g.splits));
        int w = uniform((int)((int64_t)words * split / g.splits));
        float s = 0.0f, c = 0.0f;
        float4 v = tri0[min(64 * w + lane, n - 1)];
        for (; w < w1; ++w) {
            const int kind = 64 * w + lane < n ? box.kind(v) : 0;
            v = tri0[min(64 * w + 64 + lane, n - 1)];  // the next word's
            unsigned long long far = __builtin_amdgcn_ballot_w64(kind == want);
            if (!far) continue;
            ConstTri rec = (ConstTri)(uintptr_t)(tri + 64 * w);
            float ts = 0.0f;
            TriVec next = rec[__builtin_ctzll(far)];
            while (far) {
                const TriVec r = next;
                far &= far - 1ull;
                next = rec[far ? __builtin_ctzll(far) : 0];
                __builtin_amdgcn_sched_barrier(0);  // the load goes out before this triangle's arithmetic
                const float x = r[0] - qx, y = r[1] - qy, z = r[2] - qz;
                const float q = __builtin_fmaf(z, z, __builtin_fmaf(y, y, x * x));
                const float s1 = __builtin_fmaf(z, r[6], __builtin_fmaf(y, r[5], x * r[4]));
                const float s2 = __builtin_fmaf(z, r[10], __builtin_fmaf(y, r[9], x * r[8]));
                const float al = __builtin_fmaf(z, r[14], __builtin_fmaf(y, r[13], x * r[12]));
                ts += far_angle(q, s1, s2, al, r[7], r[11], r[15]);
            }
            neumaier_add(s, c, ts);
        }
        if (j < nn) m.node[((int64_t)split * block_count(m) + b) * (nc + nf) + (part == 0 ? 0 : nc) + j] = s + c;
    }
}

// 38 VALU with 4 transcendentals per node, 30 per near point.  Counted, the nodes issue 0.90 VALU per CU and
// clock and the blocks 0.48, where the all-pairs kernel reaches 1.6: the rest is waits, for the triangles'
// scalar loads and, at the end, for few waves.  19000 faces with 5 % missing on 128^3: one by one 1956 us, here
// 204 + 221; 46000 faces with 8 % missing on 141 x 117 x 131: 7600 us, here 876 + 541.
//
// One workgroup per block and kBlockRows of its planes along x; a thread takes one (y, z) and
// the planes' points there.
__global__ __launch_bounds__(kBlock) void k_cyc_blocks(const char *table) {
    static_assert(kBlock == kBlockSide * kBlockSide, "a thread per (y, z)");
    constexpr int kWords = 64;                             // words of 64 slots looked at together
    __shared__ float T[3][kBlockSide][kFine];          // weights of the fine nodes at the voxels
    __shared__ float C[3][kFine][kCoarse];             // and of the coarse nodes at the fine ones
    __shared__ float S[kFine][kFine][kFine];
    __shared__ float A[kFine][kFine][kBlockSide];  // the intermediate sums
    __shared__ float Z[kCoarse][kCoarse][kCoarse];
    __shared__ unsigned long long s_near[kWords];
    const int64_t units = reinterpret_cast<const CycHead *>(table)->u_blk;
    const int tid = threadIdx.x, ty = tid / kBlockSide, tz = tid % kBlockSide;
    for (int64_t u = blockIdx.x; u < units; u += gridDim.x) {
        const CycMesh &m = *uniform(find_mesh<&CycMesh::u_blk>(table, u));
        const int n_tri = uniform(m.st->n_tri), n_short = uniform(m.st->n_short), n = uniform(m.st->n_rec) - 2 * n_tri;
        const int go = uniform(m.st->go);
        if (n == 0) continue;  // (go is 2 with no caps, and 1 leaves them to be added)
        const CycBlocks &g = m.grid;
        const int parts = (g.size[0] + kBlockRows - 1) / kBlockRows;
        const int64_t b = (u - m.u_blk) / parts;
        const int x0 = (int)(u - m.u_blk - b * parts) * kBlockRows;
        int i0[3];
        block_origin(m, b, i0);
        const Block box(m, i0);
        const int nc = g.coarse[0] * g.coarse[1] * g.coarse[2], nf = g.fine[0] * g.fine[1] * g.fine[2];
        const float *node = m.node + b * (nc + nf);
        const int64_t stride = block_count(m) * (nc + nf);
        auto node_sum = [&](int j) {
            float v = 0.0f;
#pragma unroll
            for (int x = 0; x < kMaxSplits; ++x) v += x < g.splits ? node[x * stride + j] : 0.0f;
            return v;
        };
        __syncthreads();
        for (int e = tid; e < kWeights; e += kBlock) (e < kFineWeights ? (&T[0][0][0])[e] : (&C[0][0][0])[e - kFineWeights]) = m.weight[e];
        if (tid < kCoarse * kCoarse * kCoarse) {
            const int j0 = tid / (kCoarse * kCoarse), j1 = tid / kCoarse % kCoarse, j2 = tid % kCoarse;
            const bool in = j0 < g.coarse[0] && j1 < g.coarse[1] && j2 < g.coarse[2];
            Z[j0][j1][j2] = in ? node_sum((j0 * g.coarse[1] + j1) * g.coarse[2] + j2) : 0.0f;
        }
        for (int e = tid; e < kFine * kFine * kFine; e += kBlock) {
            const int j0 = e / (kFine * kFine), j1 = e / kFine % kFine, j2 = e % kFine;
            const bool in = j0 < g.fine[0] && j1 < g.fine[1] && j2 < g.fine[2];
            S[j0][j1][j2] = in ? node_sum(nc + (j0 * g.fine[1] + j1) * g.fine[2] + j2) : 0.0f;
        }
        __syncthreads();
        for (int e = tid; e < kFine * kFine * kFine; e += kBlock) {  // coarse nodes onto the fine
            const int j0 = e / (kFine * kFine), j1 = e / kFine % kFine, j2 = e % kFine;
            float v = 0.0f;
#pragma unroll
            for (int k0 = 0; k0 < kCoarse; ++k0) {
                float v0 = 0.0f;
#pragma unroll
                for (int k1 = 0; k1 < kCoarse; ++k1) {
                    float v1 = 0.0f;
#pragma unroll
                    for (int k2 = 0; k2 < kCoarse; ++k2) v1 = __builtin_fmaf(Z[k0][k1][k2], C[2][j2][k2], v1);
                    v0 = __builtin_fmaf(v1, C[1][j1][k1], v0);
                }
                v = __builtin_fmaf(v0, C[0][j0][k0], v);
            }
            S[j0][j1][j2] += v;
        }
        __syncthreads();
        for (int e = tid; e < kFine * kFine * kBlockSide; e += kBlock) {
            const int j0 = e / (kFine * kBlockSide), j1 = e / kBlockSide % kFine, z = e % kBlockSide;
            float v = 0.0f;
#pragma unroll
            for (int k = 0; k < kFine; ++k) v = __builtin_fmaf(S[j0][j1][k], T[2][z][k], v);
            A[j0][j1][z] = v;
        }
        __syncthreads();
        float s[kBlockRows], c[kBlockRows], qx[kBlockRows];
#pragma unroll
        for (int p = 0; p < kBlockRows; ++p) {
            s[p] = c[p] = 0.0f;
            qx[p] = centre(m.ps, 0, i0[0] + x0 + p);
        }
#pragma unroll 1
        for (int j0 = 0; j0 < g.fine[0]; ++j0) {
            float v = 0.0f;
#pragma unroll
            for (int k = 0; k < kFine; ++k) v = __builtin_fmaf(A[j0][k][tz], T[1][ty][k], v);
#pragma unroll
            for (int p = 0; p < kBlockRows; ++p) s[p] = __builtin_fmaf(v, T[0][x0 + p][j0], s[p]);
        }
        const float qy = centre(m.ps, 1, i0[1] + ty), qz = centre(m.ps, 2, i0[2] + tz);
        const TriRec *tri = uniform(m.tri);
        const VRec *caps = uniform(m.caps);
        const float4 *tri0 = uniform(m.tri0);
        for (int w = 0; w < n; w += 64) {
            if (w % (64 * kWords) == 0) {
                __syncthreads();
#pragma unroll 4
                for (int k = tid / 64; k < kWords; k += kBlock / 64) {
                    const int at = w + 64 * k + (tid & 63);
                    const int kind = at < n ? box.kind(tri0[at]) : 0;
                    const unsigned long long mask = __builtin_amdgcn_ballot_w64(kind < 0);
                    if ((tid & 63) == 0) s_near[k] = mask;
                }
                __syncthreads();
            }
            const unsigned long long word = s_near[w / 64 % kWords];
            unsigned long long near = (unsigned long long)(unsigned)uniform((int)(word >> 32)) << 32 |
                                      (unsigned)uniform((int)(unsigned)word);
            if (!near) continue;
            ConstTri rec = (ConstTri)(uintptr_t)(tri + w);
            TriVec next = rec[__builtin_ctzll(near)];
            float ts[kBlockRows];
#pragma unroll
            for (int p = 0; p < kBlockRows; ++p) ts[p] = 0.0f;
            while (near) {
                const TriVec r = next;
                const int i = w + __builtin_ctzll(near);
                near &= near - 1ull;
                next = rec[near ? __builtin_ctzll(near) : 0];
                __builtin_amdgcn_sched_barrier(0);
                const float y = r[1] - qy, z = r[2] - qz;
                const float yz = __builtin_fmaf(z, z, y * y), yz1 = __builtin_fmaf(z, r[6], y * r[5]);
                const float yz2 = __builtin_fmaf(z, r[10], y * r[9]), yzn = __builtin_fmaf(z, r[14], y * r[13]);
                float v[kBlockRows];
                unsigned close = 0;
#pragma unroll
                for (int p = 0; p < kBlockRows; ++p) {
                    const float x = r[0] - qx[p], q = __builtin_fmaf(x, x, yz);
                    v[p] = far_angle(q, __builtin_fmaf(x, r[4], yz1), __builtin_fmaf(x, r[8], yz2),
                                     __builtin_fmaf(x, r[12], yzn), r[7], r[11], r[15]);
                    close |= q < r[3] ? 1u << p : 0u;
                }
                if (__builtin_expect(__builtin_amdgcn_ballot_w64(close != 0u) != 0ull, 0)) {
                    const int at = i < n_tri ? 3 * i : i + 2 * n_tri - 2;  // of a triangle's loop, or of its strip
                    const bool fp64 = i >= n_tri && at + 2 >= n_short;
                    const CapRecords r3(caps + at);
#pragma unroll 1
                    for (int k = 0; k < kBlockRows; ++k) {
                        if (!(close >> k & 1u)) continue;
                        float x = qx[0];
#pragma unroll
                        for (int p = 1; p < kBlockRows; ++p) x = p == k ? qx[p] : x;
                        const float a = fp64 ? r3.angle64(x, qy, qz) : r3.angle(x, qy, qz);
#pragma unroll
                        for (int p = 0; p < kBlockRows; ++p) v[p] = p == k ? a : v[p];
                    }
                }
#pragma unroll
                for (int p = 0; p < kBlockRows; ++p) ts[p] += v[p];
            }
#pragma unroll
            for (int p = 0; p < kBlockRows; ++p) neumaier_add(s[p], c[p], ts[p]);
        }
        const int iy = i0[1] + ty, iz = i0[2] + tz;
        if (ty < g.size[1] && tz < g.size[2] && iy < m.ps.n1 && iz < m.ps.n2) {
#pragma unroll
            for (int p = 0; p < kBlockRows; ++p) {
                if (x0 + p >= g.size[0] || i0[0] + x0 + p >= m.n0) break;
                const int64_t at = ((int64_t)(i0[0] + x0 + p) * m.ps.n1 + iy) * m.ps.n2 + iz;
                if (at >= m.p0 && at < m.p0 + m.P) add_caps(m, at, s[p] + c[p], go);
            }
        }
    }
}

// ------------------------------------------------------------------ direct sums

// One workgroup per listed voxel, 32 lanes per tile of the record stream, a lane per two
// records: what sum_tile does one record after another (a tile took 25 us that way), with
// the same pairing of faces and the same order of the sums.  A tile of whole six-record
// steps pairs the faces of records 2 l and 2 l + 1, and lone faces two at a time; the
// records after its last whole step (in the stream's last tile) count one by one.
constexpr int kNearThreads = 1024, kNearTiles = kNearThreads / 32, kNearSums = 1024;

__global__ __launch_bounds__(kNearThreads) void k_cyc_near(const char *table) {
    __shared__ float2 s_face[kNearTiles][32];    // (alpha, beta) of a lane's lone face
    __shared__ float s_part[kNearTiles][36];     // a tile's terms in order: 30 lanes, the last lone face, 5 tail records
    __shared__ float s_tile[kNearSums];          // tiles' sums
    __shared__ float s_chunk[kNearSums];         // chunks' sums
    const CycHead *h = reinterpret_cast<const CycHead *>(table);
    const CycMesh *meshes = meshes_of(table);
    const int tid = threadIdx.x, tl = tid >> 5, l = tid & 31;
    const int64_t g = gridDim.x;
    int64_t before = 0;
    for (int mi = 0; mi < h->n; ++mi) {
        const CycMesh &m = meshes[mi];
        if (m.st->go) {
            if (m.partials)  // of the all-pairs kernel, which went before
                for (int64_t idx = blockIdx.x * (int64_t)kNearThreads + tid; idx < m.P; idx += g * kNearThreads) {
                    if (!go_writes(m.st, m.mark, idx)) continue;
                    const float w = split_sum(m.partials, m.split, m.P, idx) * kInv2Pi;
                    m.W[idx] = w;
                    write_occ(m.occ, idx, w);
                }
            continue;
        }
        const int64_t n = m.st->n_near;
        const float4 *src = reinterpret_cast<const float4 *>(m.recs);
        const int64_t tiles = (m.nR + kRecTile - 1) / kRecTile, per = m.chunk / kRecTile;
        for (int64_t x = (blockIdx.x + g - before % g) % g; x < n; x += g) {
            const int64_t at = m.p0 + m.near[x];
            float qx[1], qy[1], qz[1];
            m.ps.get(at, qx[0], qy[0], qz[0]);
            float s = 0.0f, c = 0.0f, cs = 0.0f, cc = 0.0f;  // chunks so far, this chunk's tiles
            // whole chunks at a time where they fit, else parts of one
            const int64_t pass = per <= kNearSums ? kNearSums / per * per : kNearSums;
            for (int64_t t0 = 0; t0 < tiles; t0 += pass) {
              const int here = (int)min(pass, tiles - t0);
              for (int k = tl; k < here; k += kNearTiles) {
                const int64_t t = t0 + k;
                const int nt = (int)min((int64_t)kRecTile, m.nR - t * kRecTile);
                const int full = nt / 6 * 6;
                const bool in_step = 2 * l < full;
                Slot<1> S0, S1, S2;
                float a0[1], b0[1], a1[1], b1[1];
                unsigned bits = 0;
                if (2 * l < nt) {
                    const int64_t r = t * kRecTile + 2 * l;
                    const bool second = 2 * l + 1 < nt;
                    const float4 vx = src[2 * r], nx = src[2 * r + 1];
                    const float4 vy = second ? src[2 * r + 2] : vx, ny = second ? src[2 * r + 3] : nx;
                    prime_window<1>(src, r, S0, S1, S2, qx, qy, qz);
                    bits = (vx.w != 0.0f ? 1u : 0u) | (second && vy.w != 0.0f ? 2u : 0u);
                    enter_vertex<1>(vx, S2, S0, qx, qy, qz);
                    if (bits & 1u) face_terms<1>(nx, S1, S2, S0, a0, b0);
                    enter_vertex<1>(vy, S0, S1, qx, qy, qz);
                    if (bits & 2u) {
                        if (in_step)
                            face_terms<1, true>(ny, S2, S0, S1, a1, b1);
                        else
                            face_terms<1>(ny, S2, S0, S1, a1, b1);
                    }
                }
                const bool lone = in_step && (bits == 1u || bits == 2u);
                const unsigned all = (unsigned)(__builtin_amdgcn_ballot_w64(lone) >> (tid & 32));
                const unsigned lower = all & ((1u << l) - 1u);
                if (lone) s_face[tl][l] = bits & 1u ? make_float2(a0[0], b0[0]) : make_float2(a1[0], b1[0]);
                float *part = s_part[tl];
                if (l < 6) part[30 + l] = 0.0f;  // (the same wave writes and reads these)
                __builtin_amdgcn_wave_barrier();
                float term = 0.0f;
                if (in_step && bits == 3u) {
                    term = pair_angle(a0[0], b0[0], a1[0], b1[0]);
                } else if (lone) {
                    const float2 f = s_face[tl][l];
                    if (__popc(lower) & 1) {
                        const float2 e = s_face[tl][31 - __clz((int)lower)];
                        term = pair_angle(e.x, e.y, f.x, f.y);
                    } else if ((all >> l) == 1u) {  // the tile's last, without a partner
                        part[30] = atan2_eq8(f.x, f.y);
                    }
                } else if (!in_step && 2 * l < nt) {
                    const int k = 31 + 2 * l - full;
                    if (bits & 1u) part[k] = atan2_eq8(a0[0], b0[0]);
                    if (bits & 2u) part[k + 1] = atan2_eq8(a1[0], b1[0]);
                }
                if (l < 30) part[l] = term;
                __builtin_amdgcn_wave_barrier();
                if (l == 0) {
                    float ts = 0.0f;
#pragma unroll
                    for (int i = 0; i < 36; ++i) ts += part[i];
                    s_tile[k] = ts;
                }
                __builtin_amdgcn_wave_barrier();
              }
              __syncthreads();
              if (per <= kNearSums) {
                const int chunks = (int)((here + per - 1) / per);
                for (int i = tid; i < chunks; i += kNearThreads) {
                    float a = 0.0f, b = 0.0f;
                    for (int k = i * (int)per; k < min(here, (i + 1) * (int)per); ++k) neumaier_add(a, b, s_tile[k]);
                    s_chunk[i] = a + b;
                }
                __syncthreads();
                if (tid == 0)
                    for (int i = 0; i < chunks; ++i) neumaier_add(s, c, s_chunk[i]);
              } else if (tid == 0) {
                for (int i = 0; i < here; ++i) {
                    neumaier_add(cs, cc, s_tile[i]);
                    if ((t0 + i + 1) % per == 0 || t0 + i + 1 == tiles) {
                        neumaier_add(s, c, cs + cc);
                        cs = cc = 0.0f;
                    }
                }
              }
              __syncthreads();
            }
            if (tid == 0) {
                const float w = (s + c) * kInv2Pi;
                m.W[at] = w;
                write_occ(m.occ, at, w);
            }
        }
        before += n;
    }
}

}  // namespace

// ------------------------------------------------------------------ host

// The path's nine short launches take 45 to 55 us for a closed mesh and up to 120 us for many
// holes; the all-pairs sum took (us) 77 at 3.8e7 pairs without strips, and with them 50 at 4.3e7, 60
// at 4.8e7 (here 46, closed), 69 at 7.1e7 (here 75, 7 % missing), 103 at 9.2e7 (here 68).
// A few large faces are better summed: their close voxels are many.
// A list of points has two launches more, and its faces go through chains of points: 9120
// faces with 5 % missing at 100003 points 702 -> 269 us, 24109 at 28249 925 -> 102 us; at 2e8 pairs 235 against
// 269 without strips, below 1.5e8 it loses.  With strips the line is the same: 117 us at 1.45e8 pairs, here 170.
bool cyc_wanted(int64_t nV, int64_t nF, int64_t P, double min_pairs) {
    return nF >= 128 && nV > 0 && nV < ((int64_t)1 << 30) && nF < ((int64_t)1 << 28) && P > 0 &&
           (double)nF * (double)P >= min_pairs;
}

// Floats of node values that a grid of so many voxels may have.
static int64_t node_space(int64_t points) {
    return std::max(points * 35 / 100, std::min<int64_t>(points * 3 / 4, kSplitWaves * 64));
}

// Blocks of up to 16 voxels per axis, all of one size.  They pay from 2^18 voxels and 1.5e9
// (face, voxel) pairs on (the caps' number is not known here).  Measured (us, caps one by one | blocks), 3 to 8 %
// of the faces missing: 64^3 voxels, 1000 faces 26 | 59, 5120 faces 92 | 87, 20000 faces 525 | 411; 80^3,
// 1000 faces 43 | 63, 20000 faces 344 | 167; 128^3, 2000 faces 147 | 101, 20000 faces 1956 | 387.
CycBlocks cyc_blocks(const int32_t *n, int64_t nF) {
    CycBlocks b{};
    int64_t voxels = 1, coarse = 1, fine = 1, blocks = 1, points = 1;
    for (int d = 0; d < 3; ++d) {
        b.n[d] = (n[d] + kBlockSide - 1) / kBlockSide;
        b.size[d] = (n[d] + b.n[d] - 1) / b.n[d];
        b.n[d] = (n[d] + b.size[d] - 1) / b.size[d];
        b.coarse[d] = std::min(kCoarse, b.size[d]);
        b.fine[d] = std::min(kFine, b.size[d]);
        voxels *= b.size[d];
        coarse *= b.coarse[d];
        fine *= b.fine[d];
        blocks *= b.n[d];
        points *= n[d];
    }
    if (points < kBlockPoints || (double)nF * (double)points < 1.5e9 || 4 * fine > voxels) return CycBlocks{};
    // The coarse nodes' wave has most of the triangles, so splits help beyond filling the chip:
    // 512 blocks took 213 us with one, 165 with five.
    const int64_t waves = blocks * (1 + (fine + 63) / 64), nodes = blocks * (coarse + fine);
    if (nodes > node_space(points)) return CycBlocks{};
    b.order = kFine;
    b.splits = (int32_t)std::max<int64_t>(1, std::min<int64_t>({kSplitWaves / waves, node_space(points) / nodes, kMaxSplits}));
    return b;
}

int64_t cyc_node_floats(const CycBlocks &b, int64_t x_blocks) {
    if (b.order == 0) return 0;
    const int64_t nodes = (int64_t)b.coarse[0] * b.coarse[1] * b.coarse[2] + (int64_t)b.fine[0] * b.fine[1] * b.fine[2];
    return (int64_t)b.splits * x_blocks * b.n[1] * b.n[2] * nodes;
}

// Below 2^18 points a lane with all caps in turn leaves the chip idle: the caps are split over
// the least number of waves that gives 3000 in all.  Measured (us, k_cyc_sum | 4, 8, 16 waves):
// 12818 points 171 | 54 34 27, 59276 points 33 | 17 18 28, 97336 points 52 | 29 30 47,
// 262144 points 62 | 62 72 115 and, with twice the caps, 101 | 102 113 217.
int cyc_ppl(int64_t points, int ppl) {
    if (points >= ((int64_t)1 << 18)) return ppl;
    return points >= 48000 ? -4 : points >= 24000 ? -8 : -16;
}

bool cyc_grid_ok(const wn_grid &g) {
    for (int d = 0; d < 3; ++d) {
        const float h = (g.hi[d] - g.lo[d]) / (float)g.n[d];
        if (!(__builtin_fabsf(g.lo[d]) <= kCoordMax && __builtin_fabsf(g.hi[d]) <= kCoordMax && h > 1.0e-30f)) return false;
    }
    return true;
}

namespace {

int64_t edge_buckets(int64_t nF) {
    int64_t b = 64;
    while (b < 2 * nF) b *= 2;
    return b;
}

int64_t slab_capacity(int64_t nF) { return nF + 2 * kListShare; }

// Bins per side for so many points (0: too many): about three to a bin.
int64_t bin_side(int64_t points) {
    if (points > kCycPoints) return 0;
    return std::max<int64_t>(8, (int64_t)std::sqrt((double)points / 3.0));
}

int64_t near_capacity(int64_t P) { return P < kCycNear ? P : kCycNear; }

// Calls take(field, bytes) for every scratch array of a mesh, in layout order.
template <typename Fn>
void cyc_arrays(CycMesh &m, int64_t nodes, Fn &&take) {
    const size_t nV = (size_t)m.nV, nF = (size_t)m.nF, units = (3 * nF + kCycUnit - 1) / kCycUnit;
    take(m.st, sizeof(CycState));
    take(m.ent, 16 * 3 * nF);
    take(m.head, 4 * (size_t)edge_buckets(m.nF));
    take(m.count, 4 * nF);
    take(m.list, 4 * units * kCycUnit);
    take(m.blk, 8 * units);
    take(m.edge, 8 * nF);
    if (m.P == 0) {
        take(m.used, 4 * nV);
        take(m.most, 4 * nV);
        take(m.grad, 24 * nV);
        return;
    }
    take(m.hout, 4 * nV);
    take(m.hin, 4 * nV);
    take(m.nout, 4 * nF);
    take(m.nin, 4 * nF);
    take(m.rank, 4 * nF);
    take(m.next, 4 * nF);
    take(m.cvid, 4 * nF);
    take(m.cpos, 4 * nF);
    take(m.caps, sizeof(VRec) * nF);
    take(m.tri, sizeof(TriRec) * (nF + 2));
    take(m.tri0, 16 * (nF + 2));
    take(m.slab, 8 * (size_t)slab_capacity(m.nF));
    take(m.near, 4 * (size_t)near_capacity(m.P));
    take(m.mark, 4 * (((size_t)m.P + 31) / 32));
    take(m.weight, 4 * kWeights);
    // a grid's node values or a list's bins
    size_t shared = 4 * (size_t)(nodes < 0 ? node_space(m.P) : nodes);
    const int64_t bins = m.bins ? m.bins : nodes < 0 ? bin_side(m.P) : 0;
    const size_t bin_bytes = align_up(4 * (size_t)(bins * bins));
    if (bins) shared = std::max(shared, 2 * bin_bytes + 4 * (size_t)m.P);
    take(m.node, shared);
    m.bin = reinterpret_cast<int32_t *>(m.node);
    m.bin_n = m.bin + bin_bytes / 4;
    m.after = m.bin_n + bin_bytes / 4;
}

}  // namespace

size_t cyc_bytes(int64_t nV, int64_t nF, int64_t P, int64_t nodes) {
    CycMesh m{};
    m.nV = nV;
    m.nF = nF;
    m.P = P;
    size_t o = 0;
    cyc_arrays(m, nodes, [&](auto *&, size_t bytes) { o += align_up(bytes); });
    return o;
}

void cyc_place(CycMesh &m, char *base) {
    size_t o = 0;
    if (m.ps.Q) {
        m.bins = (int32_t)bin_side(m.P);
    } else if (m.P > 0) {
        const int64_t yz = (int64_t)m.ps.n1 * m.ps.n2;
        m.i_first = (int32_t)(m.p0 / yz);
        m.i_last = (int32_t)((m.p0 + m.P - 1) / yz);
        const int32_t n[3] = {m.n0, m.ps.n1, m.ps.n2};
        m.grid = cyc_blocks(n, m.nF);
        m.xb0 = m.grid.order ? m.i_first / m.grid.size[0] : 0;
        m.xb1 = m.grid.order ? m.i_last / m.grid.size[0] : 0;
    }
    cyc_arrays(m, cyc_node_floats(m.grid, m.xb1 - m.xb0 + 1), [&](auto *&p, size_t bytes) {
        p = reinterpret_cast<std::remove_reference_t<decltype(p)>>(base + o);
        o += align_up(bytes);
    });
    m.buckets = edge_buckets(m.nF);
    m.near_cap = (int32_t)near_capacity(m.P);
    m.slab_cap = (int32_t)slab_capacity(m.nF);
}

void cyc_units(CycMesh &m, CycHead &h) {
    auto units = [](int64_t n, int64_t per) { return (n + per - 1) / per; };
    m.per = !m.bins && m.ps.n2 <= 32 ? 64 / m.ps.n2 : 1;
    // (a list's units hold as many points as a grid's hold columns' lanes)
    const int64_t columns = m.bins ? (m.P + 63) / 64
                                   : units((m.p0 + m.P - 1) / m.ps.n2 - m.p0 / m.ps.n2 + 1, m.per);
    m.u_clear = h.u_clear;
    m.u_face = h.u_face;
    m.u_half = h.u_half;
    m.u_col = h.u_col;
    m.u_sum = h.u_sum;
    m.u_node = h.u_node;
    m.u_blk = h.u_blk;
    const int32_t n[3] = {m.n0, m.ps.n1, m.ps.n2};
    for (int d = 0; d < 3; ++d) {
        const double l = m.ps.lo[d], c = m.ps.h[d];
        m.inv_h[d] = 1.0 / c;
        m.slack[d] = 1.0e-3 + 2.4e-7 * std::max(std::fabs(l), std::fabs(l + n[d] * c)) / c;
    }
    h.u_clear += units(std::max({m.buckets, 3 * m.nV, m.nF, m.P, (int64_t)m.bins * m.bins}), kCycClear);
    h.u_face += units(m.nF, kCycUnit / kCycFaceLanes);
    h.u_half += units(3 * m.nF, kCycUnit);
    h.u_col += units(columns, kCycColumns);
    const CycBlocks &b = m.grid;
    if (b.order == 0) {
        h.u_sum += units(m.P, h.ppl > 0 ? (int64_t)kBlock * h.ppl : 64);
    } else {
        const int64_t blocks = (int64_t)(m.xb1 - m.xb0 + 1) * b.n[1] * b.n[2];
        h.u_node += blocks * (1 + units((int64_t)b.fine[0] * b.fine[1] * b.fine[2], 64)) * b.splits;
        h.u_blk += blocks * units(b.size[0], kBlockRows);
    }
    h.n += 1;
}

hipError_t launch_cyc_begin(const CycMesh &m, const CycHead &h, char *table, hipStream_t s) {
    k_cyc_begin_one<<<dim3((unsigned)h.u_clear), kCycUnit, 0, s>>>(m, h, table);
    return hipGetLastError();
}

hipError_t launch_cyc_clear(char *table, hipStream_t s) {
    k_cyc_clear<<<2048, kCycUnit, 0, s>>>(table);
    return hipGetLastError();
}

hipError_t launch_cyc(const CycHead &h, char *table, bool fixed, int64_t pack, hipStream_t s) {
    auto grid = [&](int64_t units) { return dim3((unsigned)(fixed ? 2048 : units)); };
    if (pack > 0)
        k_cyc_faces<true><<<dim3((unsigned)(h.u_face + (pack + kCycUnit - 1) / kCycUnit)), kCycUnit, 0, s>>>(table);
    else
        k_cyc_faces<false><<<grid(h.u_face), kCycUnit, 0, s>>>(table);
    k_cyc_mark<<<grid(h.u_half), kCycUnit, 0, s>>>(table);
    k_cyc_caps<<<fixed ? 256 : h.n, kCapThreads, 0, s>>>(table);
    k_cyc_slabs<<<1024, kCycUnit, 0, s>>>(table);
    k_cyc_columns<<<grid(h.u_col), kCycColumns * 64, 0, s>>>(table);
    if (h.u_node > 0) {
        k_cyc_nodes<<<dim3((unsigned)(fixed ? 16384 : h.u_node)), 64, 0, s>>>(table);
        k_cyc_blocks<<<dim3((unsigned)(fixed ? 8192 : h.u_blk)), kBlock, 0, s>>>(table);
    }
    if (h.u_sum == 0) return hipGetLastError();
    if (h.ppl == -16)
        k_cyc_sum_split<16><<<grid(h.u_sum), 16 * 64, 0, s>>>(table);
    else if (h.ppl == -8)
        k_cyc_sum_split<8><<<grid(h.u_sum), 8 * 64, 0, s>>>(table);
    else if (h.ppl == -4)
        k_cyc_sum_split<4><<<grid(h.u_sum), 4 * 64, 0, s>>>(table);
    else if (h.ppl == 1)
        k_cyc_sum<1><<<grid(h.u_sum), kBlock, 0, s>>>(table);
    else if (h.ppl == 2)
        k_cyc_sum<2><<<grid(h.u_sum), kBlock, 0, s>>>(table);
    else
        k_cyc_sum<4><<<grid(h.u_sum), kBlock, 0, s>>>(table);
    return hipGetLastError();
}

hipError_t launch_cyc_bins(const CycMesh &m, char *table, hipStream_t s) {
    k_cyc_box<<<dim3((unsigned)((std::max(m.nR, m.nV) + kCycUnit - 1) / kCycUnit)), kCycUnit, 0, s>>>(table);
    k_cyc_bin<<<dim3((unsigned)((m.P + kCycUnit - 1) / kCycUnit)), kCycUnit, 0, s>>>(table);
    return hipGetLastError();
}

hipError_t launch_cyc_edges(const CycHead &h, char *table, hipStream_t s) {
    k_cyc_faces<false><<<dim3((unsigned)h.u_face), kCycUnit, 0, s>>>(table);
    k_cyc_mark<<<dim3((unsigned)h.u_half), kCycUnit, 0, s>>>(table);
    k_cyc_caps<<<1, kCapThreads, 0, s>>>(table);
    return hipGetLastError();
}

hipError_t launch_cyc_near(char *table, hipStream_t s) {
    k_cyc_near<<<512, kNearThreads, 0, s>>>(table);
    return hipGetLastError();
}

}  // namespace wn
