// Forward by the boundary of the mesh (wn_cycle.hip): shared declarations.
//
// The solid angles of a closed oriented surface add up to an integer multiple of 4 pi
// (Eq. 3: the winding number of a closed surface is its occupancy), so with a surface C
// that has the same boundary as the mesh M ("caps" over the loops of M's unmatched
// edges), M - C is closed and
//     W(q) = n(q) + sum over the cap triangles of their half solid angle / (2 pi),
// where n(q) is the winding number of the closed surface M - C: a signed count of its
// crossings with the ray from q along +z.  On a grid a face's crossing with a column
// counts for every voxel of the column below it, so n costs a few operations per face and
// a pass over the voxels, and the all-pairs sum is left for the caps alone: nothing for a
// closed mesh, one triangle per deleted face for a mesh with holes.
// Points very close to the surface (where the side of a face is a matter of rounding) and
// points whose W is within rounding of the occupancy threshold take the direct sum over
// all faces, with the records, tiles and order of the all-pairs kernel.
#pragma once

#include "wn_internal.hpp"

namespace wn {

constexpr int kCycUnit = 256;        // half-edges per workgroup unit
constexpr int kCycFaceLanes = 8;     // lanes per face
constexpr int kCycColumns = 4;       // waves of columns of voxels per workgroup unit
constexpr int kCycClear = 2048;      // words cleared per workgroup unit
constexpr int kCycNear = 65536;      // points that may take the direct sum one by one
constexpr int kCycShortLoop = 6;     // longest loop whose caps are evaluated in FP32
constexpr int64_t kCycMaxEdges = 1 << 20;  // longest boundary

// A triangle for points far from it: with d_j = v_j - v_0 and R = v_0 - q,
// |v_j - q|^2 = |R|^2 + R . 2 d_j + |d_j|^2 and (v_0 - q) . (v_j - q) = |R|^2 + R . 2 d_j / 2.
struct alignas(64) TriRec {
    float v[3], far;      // v_0; square of the distance from which these forms are used
    float d[2][4];        // 2 d_1, |d_1|^2; 2 d_2, |d_2|^2
    float n[3], g;        // (v_1 - v_0) x (v_2 - v_0); d_1 . d_2
};

// The grid cut into blocks of voxels, for the caps' far field (wn_cycle.hip).
struct CycBlocks {
    int32_t order;      // 0: no blocks
    int32_t size[3];    // voxels per block
    int32_t n[3];       // blocks
    int32_t coarse[3];  // coarse nodes per block: min(kCoarse, size)
    int32_t fine[3];    // fine nodes: min(kFine, size)
    int32_t splits;     // of the caps over waves
};

// What the kernels find out about a mesh.
struct CycState {
    int32_t go;         // all-pairs sum: 0 none, 1 at the marked voxels, 2 at all voxels
    int32_t n_rec;      // cap records: triangles, other short loops, long loops
    int32_t n_tri;      // triangles (three records each)
    int32_t n_short;    // records of the triangles and the other short loops
    int32_t n_near;     // points on the list of direct sums
    int32_t odd;        // adjoint: dL/dW holds a value that is not finite
    uint32_t max_bits;  // bits of the largest |coordinate| of a face corner
    unsigned long long n_slab;  // entries of the raster list; in the upper half those of 64 columns asked for
    uint32_t box[6];    // point lists: largest x, y, z and -x, -y, -z of the vertices, as ordered integers
};

// One mesh (or slice of its grid) of a launch.
struct CycMesh {
    const float *V;
    const int32_t *F;
    VRec *recs;           // the all-pairs record stream
    const int32_t *R;     // its order (plain calls), or null: three records per face
    WsHeader *hdr;        // reset by the begin kernel (plain calls)
    const float *partials;  // sums of the all-pairs kernel's splits, if it has more than one (plain calls)
    int32_t split;
    int64_t nV, nF, nR;
    int64_t chunk;        // records per partial sum of the all-pairs kernel
    PointSrc ps;
    int32_t n0;           // cells along x
    int32_t strips;       // the stream has to name every face once
    int32_t per;          // columns of voxels that a wave takes at once
    int64_t p0, P;        // the voxels [p0, p0 + P)
    int32_t i_first, i_last;  // their range along x
    float *W;             // null: the boundary edges alone (the adjoint)
    OccParams occ;
    CycState *st;
    double inv_h[3], slack[3];  // cells per length, and the rounding of a voxel centre in cells
    int4 *ent;            // [3 nF] half-edges chained by bucket: next, lower vertex, upper, 1 if it runs down
    int32_t *head;        // [buckets] first half-edge of a bucket
    int64_t buckets;      // a power of two
    int32_t *hout, *hin;  // [nV] first boundary edge leaving / entering a vertex
    int32_t *used;        // [nV] adjoint: 1 for a vertex of a face
    uint32_t *most;       // [nV] adjoint: bits of the vertex's largest |term|
    int64_t *grad;        // [nV][3] adjoint: sums of its terms
    int32_t *count;       // [nF] times the stream names a face
    int32_t *list, *blk;  // boundary half-edges of each unit, and their number and offset
    int2 *edge;           // [nF] boundary edges (start, end)
    int32_t *nout, *nin, *rank, *next;  // [nF] each
    int32_t *cvid, *cpos; // [nF] cap records: vertex, place in its loop's strip
    VRec *caps;           // [nF] cap records
    TriRec *tri;          // [nF + 2] the triangles of the loops of three, then one slot per other record
    float4 *tri0;         // [nF + 2] their v and far
    CycBlocks grid;
    int32_t xb0, xb1;     // the slice's blocks along x
    float *weight;        // weights of the blocks' nodes
    float *node;          // [splits][blocks of the slice][coarse, fine nodes] far field at the nodes
    // A list of points (ps.Q) in place of a grid: bins x bins squares over the mesh's box in x and y
    // take the place of the columns.
    int32_t bins;
    int32_t *bin, *bin_n; // [bins^2] first point of a bin, and their number
    int32_t *after;       // [P] the next point of its bin
    int2 *slab;           // raster list: (face, or nF + cap record; which part of its columns)
    int32_t *near;        // voxels for the direct sum, counted from p0
    uint32_t *mark;       // a bit for each such voxel, also those that the list had no room for
    int32_t near_cap, slab_cap;
    int64_t u_clear, u_face, u_half, u_col, u_sum, u_node, u_blk;  // first units of this mesh
};

struct CycHead {
    int64_t meshes;  // offset of the meshes from the table
    int32_t n;
    int32_t ppl;  // points per lane of the caps' sum; -n: the caps split over n waves
    int64_t u_clear, u_face, u_half, u_col, u_sum, u_node, u_blk;  // units of all meshes
    unsigned long long cursor;
};

// Whether sizes make the boundary path worth its fixed cost (see wn_cycle.hip); P is the
// whole grid, so that a slice takes the path of the grid.
constexpr double kCycPairs = 3.0e7, kCycStripPairs = 7.0e7;  // without and with a strip order
constexpr double kCycPointPairs = 1.5e8;                     // a list of points
constexpr int64_t kCycPoints = (int64_t)1 << 22;             // the longest list (room for its bins)
bool cyc_wanted(int64_t nV, int64_t nF, int64_t P, double min_pairs = kCycPairs);
// Whether the grid's extent is finite and in the range of the path.
bool cyc_grid_ok(const wn_grid &g);
int cyc_ppl(int64_t points, int ppl);
CycBlocks cyc_blocks(const int32_t *n, int64_t nF);
int64_t cyc_node_floats(const CycBlocks &b, int64_t x_blocks);
// Scratch bytes of one mesh with P voxels in its slice (0: for the boundary edges alone) and
// `nodes` floats for the blocks (-1: as many as any grid of P voxels needs), and its
// pointers laid out from `base`.
size_t cyc_bytes(int64_t nV, int64_t nF, int64_t P, int64_t nodes = -1);
void cyc_place(CycMesh &m, char *base);
// Unit numbers of mesh m, after what `h` holds already.
void cyc_units(CycMesh &m, CycHead &h);
// The path in launch order: `begin` (one mesh: it also writes the table) or `clear` (a
// table that is in place), the packing of the record streams, `launch_cyc`, the all-pairs
// kernels for the meshes whose state asks for them, and `near` for the listed voxels.
// fixed: launches of fixed size, for a captured graph.  pack: records that are packed with
// the first kernel (one mesh).  `near` also adds up the all-pairs kernel's splits.
constexpr size_t kCycTable = 1024;
static_assert(sizeof(CycHead) + sizeof(CycMesh) <= kCycTable, "table size");
hipError_t launch_cyc_begin(const CycMesh &m, const CycHead &h, char *table, hipStream_t s);
hipError_t launch_cyc_clear(char *table, hipStream_t s);
hipError_t launch_cyc(const CycHead &h, char *table, bool fixed, int64_t pack, hipStream_t s);
// For a list of points, before launch_cyc: packs the records and bins the points.
hipError_t launch_cyc_bins(const CycMesh &m, char *table, hipStream_t s);
hipError_t launch_cyc_near(char *table, hipStream_t s);

// The boundary edges alone, after `begin`.
hipError_t launch_cyc_edges(const CycHead &h, char *table, hipStream_t s);

// Adjoint over the boundary edges (wn_edge_bwd.hip) for one mesh's table: the points of the
// tiles [t0, t1), the gradients of each edge's ends (G, float [B][6]), and dL/dV from
// them, or from the corners' gradients T where the state asks for the all-pairs sum.
// state: as much as the all-pairs adjoint's.
hipError_t launch_edge_bwd(const char *table, int64_t nQ, int64_t t0, int64_t t1, const float *dLdW, float2 *state,
                           hipStream_t s);
// With `splits` > 0 the state comes from the blocks of a large grid: each call of a sequence takes those that
// its points complete, from the dL/dW kept of all ranges so far (unless one call has it all).
struct EdgeBlocks {
    int splits;
    float2 *state;
    float *node, *kept;
};
EdgeBlocks edge_blocks(const CycBlocks &g, int64_t nF, int64_t nQ, char *space, size_t bytes);
hipError_t launch_edge_keep(const char *table, const float *dLdW, int64_t p0, int64_t n, const EdgeBlocks &e,
                            hipStream_t s);
hipError_t launch_edge_blocks(const char *table, const CycBlocks &g, int64_t plane, int64_t p0, int64_t p1, int64_t nQ,
                              const float *dLdW, const EdgeBlocks &e, hipStream_t s);
hipError_t launch_edge_reduce(const char *table, int64_t nQ, int splits, const float2 *state, float *G, hipStream_t s);
hipError_t launch_edge_gather(const char *table, int64_t nV, const float *G, const float *T, float *dLdV,
                              hipStream_t s);

// Whether the all-pairs kernels write voxel idx (counted from the slice's first): go is
// the state's, or null where the mesh has no boundary path.
__device__ __forceinline__ bool go_writes(const CycState *st, const uint32_t *mark, int64_t idx) {
    return st == nullptr || st->go == 2 || ((mark[idx >> 5] >> (idx & 31)) & 1u);
}

}  // namespace wn
