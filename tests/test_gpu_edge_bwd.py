"""dL/dV from the mesh's boundary edges (wn_edge_bwd.hip) against the FP64 oracle.

Above the rule's line (128 faces, 2e7 pairs) a grid's wn_backward without dL/dT takes this
path, with or without face pairs.  Tolerance: FP32 terms with a relative rounding of a few
1e-7, whose vertex sums are exact integers: 1e-5 of the largest component (the per-face
kernels are held to 1e-3 of a vertex's corner terms), and exactly 0 where no boundary edge
ends."""
import numpy as np
import pytest

import wn_inputs as wi
from .test_gpu_cycle import GRID, _centres, _dev, _mesh

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2407_11272_amd as wn
    wn.wn_version()
    return torch.device("cuda", 0)


def _weights(P, seed=2):
    import torch
    return torch.randn(P, device="cuda", generator=torch.Generator("cuda").manual_seed(seed))


def _pairs(V, F):
    import torch
    import paper_2407_11272_amd as wn
    return torch.as_tensor(wn.wn_build_face_pairs(np.ascontiguousarray(F), len(V))).cuda()


def _oracle(orc, V, F, grid, g):
    Q = _centres(grid).astype(np.float64)
    return orc.grad(np.asarray(V, np.float32).astype(np.float64), F, Q, g.cpu().numpy().astype(np.float64))


@pytest.mark.parametrize("kind", ["closed", "holes", "loop of 4", "loop of 7", "open end", "sheet",
                                  "two shells, one reversed", "repeated", "reversed faces"])
def test_boundary_edges_vs_oracle(dev, orc, kind):
    import paper_2407_11272_amd as wn
    V, F = _mesh(kind)
    Vt, Ft = _dev(V, F)
    g = _weights(GRID.size)
    Tr, Dr = _oracle(orc, V, F, GRID, g)
    corner = np.abs(Tr).sum(axis=(0, 1)).max() / len(V)
    for pairs in (None, _pairs(V, F)):
        D = wn.wn_backward(Vt, Ft, g, grid=GRID, pairs=pairs).cpu().numpy().astype(np.float64)
        assert wn.wn_get_device_error() == 0
        print(f"[{kind}] |d dL/dV| {np.abs(D - Dr).max():.2e} of {np.abs(Dr).max():.2e}", flush=True)
        if kind in ("closed", "two shells, one reversed"):
            assert not D.any()
        elif kind in ("repeated", "reversed faces"):   # edges that do not suit the path: the per-face kernels
            assert np.abs(D - Dr).max() <= 1e-3 * max(np.abs(Dr).max(), corner)
        else:
            assert np.abs(D - Dr).max() <= 1e-5 * np.abs(Dr).max()
            assert not D[np.abs(Dr).max(1) < 1e-12 * np.abs(Dr).max()].any()


@pytest.mark.parametrize("res", [(25, 23, 27), (40, 33, 64)])
def test_point_ranges_give_the_bits_of_one_call(dev, res):
    """Ranges shorter and longer than a round over the splits, with and without pairs."""
    import torch
    import paper_2407_11272_amd as wn
    V, F = _mesh("holes")
    Vt, Ft = _dev(V, F)
    grid = wn.Grid((-0.5,) * 3, (0.5,) * 3, res)
    P = grid.size
    g = _weights(P)
    for pairs in (None, _pairs(V, F)):
        D = wn.wn_backward(Vt, Ft, g, grid=grid, pairs=pairs)
        tiles = -(-P // 256)
        for cuts in ([1, 2, tiles // 2], [tiles - 1], list(range(1, tiles, 3))):
            sb = wn.SlicedBackward(Vt, Ft, grid=grid, pairs=pairs, vertex_sums=True)
            sb.begin()
            at = [0] + [256 * c for c in cuts] + [P]
            for a, b in zip(at[:-1], at[1:]):
                sb.points(a, b - a, g)
            assert torch.equal(sb.end(), D)


def test_fan_of_faces_at_one_vertex(dev, orc):
    """1000 triangles that share one vertex only, beside a closed mesh: a vertex where 2000
    boundary edges end.  Voxels as near as 1e-4 of edges 0.5 long leave FP32 few digits, so
    the bar here is the per-face kernels' own error."""
    import paper_2407_11272_amd as wn
    V, F = _mesh("closed")
    rng = np.random.default_rng(9)
    n, base = 1000, len(V)
    P = rng.uniform(-0.45, 0.45, (n, 3))
    V = np.concatenate([V, [[0.0117, 0.0039, -0.0071]], P, P + 0.02 * rng.standard_normal((n, 3))])
    a = base + 1 + np.arange(n)
    F = np.concatenate([F, np.stack([np.full(n, base), a, a + n], -1)])
    Vt, Ft = _dev(V, F)
    g = _weights(GRID.size)
    _, Dr = _oracle(orc, V, F, GRID, g)
    D = wn.wn_backward(Vt, Ft, g, grid=GRID).cpu().numpy().astype(np.float64)
    A = wn.wn_backward(Vt, Ft, g, grid=GRID, want_dLdT=True)[0].cpu().numpy().astype(np.float64)
    assert np.abs(D - Dr).max() <= np.abs(A - Dr).max()
    assert not D[:base].any()


def test_vertex_on_a_query_point_takes_the_per_face_sum(dev, orc):
    """A face with a vertex at q contributes nothing there, so its edges do not cancel its
    neighbours': the mesh takes the per-face kernels."""
    import paper_2407_11272_amd as wn
    V, F = _mesh("holes")
    V = np.asarray(V, np.float32).copy()
    V[100] = _centres(GRID)[7001]
    Vt, Ft = _dev(V, F)
    g = _weights(GRID.size)
    Tr, Dr = _oracle(orc, V, F, GRID, g)
    scale = np.zeros_like(Dr)
    np.add.at(scale, F.reshape(-1), np.abs(Tr.reshape(-1, 3)))
    D = wn.wn_backward(Vt, Ft, g, grid=GRID).cpu().numpy().astype(np.float64)
    far = np.setdiff1d(np.arange(len(V)), F[(F == 100).any(1)])
    assert np.all(np.abs(D - Dr)[far] <= 1e-3 * scale[far] + 1e-12)


@pytest.mark.parametrize("kind", ["closed", "holes"])
def test_values_that_are_not_finite_reach_every_vertex(dev, kind):
    import torch
    import paper_2407_11272_amd as wn
    V, F = _mesh(kind)
    V = np.concatenate([V, [[0.3, 0.3, 0.3]]])      # a vertex that no face uses
    Vt, Ft = _dev(V, F)
    for bad in (float("nan"), float("inf")):
        g = _weights(GRID.size)
        g[1234] = bad
        D = wn.wn_backward(Vt, Ft, g, grid=GRID)
        assert torch.isnan(D[:-1]).all() and not D[-1].any()
    Vt[3, 1] = float("nan")
    D = wn.wn_backward(Vt, Ft, _weights(GRID.size), grid=GRID)
    used = (Ft == 3).any(1)
    assert torch.isnan(D[3]).any() and used.any()


def test_fitting_step_follows_the_all_pairs_field(dev):
    """soft_occupancy: on the sigmoid's slope W is the all-pairs kernel's bit for bit, so the
    gradient that a steep sigmoid sends back does not depend on the path."""
    import torch
    import paper_2407_11272_amd as wn
    V, F = _mesh("holes")
    Vt, Ft = _dev(V, F)
    Q = torch.as_tensor(_centres(GRID)).cuda()
    W = wn.WindingNumber.apply(Vt, Ft, wn.Grid.of(GRID), None, None, None, (0.5, 50.0)).reshape(-1)
    P = wn.wn_voxelize(Vt, Ft, Q=Q)
    slope = (P - 0.5).abs() < 0.19
    assert slope.any()
    assert torch.equal(W[slope], P[slope])
    x = Vt.clone().requires_grad_(True)
    occ = wn.soft_occupancy(x, Ft, grid=wn.Grid.of(GRID), tau=0.5, k=50.0)
    (occ ** 2).mean().backward()
    y = Vt.clone().requires_grad_(True)
    occ2 = wn.soft_occupancy(y, Ft, Q=Q, tau=0.5, k=50.0)
    (occ2 ** 2).mean().backward()
    assert float((x.grad - y.grad).norm()) <= 1e-4 * float(y.grad.norm())


@pytest.mark.parametrize("n", [(84, 80, 82), (97, 61, 131), (230, 6, 400)])
@pytest.mark.parametrize("kind", ["holes", "open end", "sheet"])
def test_blocks_of_voxels(dev, kind, n):
    """Grids of at least 2^19 voxels, where far edges take nodes: ragged last blocks and an axis with
    fewer voxels than nodes, against the sum over the boundary edges in FP64, and point ranges
    against one call, bit for bit.  The nodes are allowed 4e-9 of an edge's share per block (x 10),
    and white noise for dL/dW adds up to 1e-2 of its terms: 1e-5."""
    import torch
    import wn_inputs as wi
    import paper_2407_11272_amd as wn
    V, F = _mesh(kind)
    grid = wi.Grid((-0.5, -0.45, -0.5), (0.5, 0.5, 0.47), n)
    assert grid.size >= 1 << 19 and len(F) * grid.size >= 1.5e9
    Vt, Ft = _dev(V, F)
    g = torch.as_tensor(np.random.default_rng(4).standard_normal(grid.size).astype(np.float32)).cuda() / grid.size
    D = wn.wn_backward(Vt, Ft, g, grid=grid)
    # dW/du = -(A x E) / (4 pi |A| (|A| |B| + A . B)) summed over the boundary edges in FP64
    e = np.concatenate([F[:, [0, 1]], F[:, [1, 2]], F[:, [2, 0]]]).astype(np.int64)
    code, back = e[:, 0] * len(V) + e[:, 1], e[:, 1] * len(V) + e[:, 0]
    e = torch.as_tensor(e[~np.isin(code, back)]).cuda()
    U, E = Vt.double()[e[:, 0]], Vt.double()[e[:, 1]] - Vt.double()[e[:, 0]]
    A = torch.zeros(len(V), 3, dtype=torch.float64, device="cuda")
    Q = torch.as_tensor(_centres(grid)).cuda()
    su, sv = torch.zeros_like(U), torch.zeros_like(U)
    for i in range(0, len(Q), 16384):
        R = U[:, None] - Q[None, i:i + 16384].double()
        S = R + E[:, None]
        a, b = R.norm(dim=2), S.norm(dim=2)
        w = g[i:i + 16384].double() / (a * b + (R * S).sum(2))
        su += ((w / a)[..., None] * R).sum(1)
        sv += ((w / b)[..., None] * R).sum(1)
    A.index_add_(0, e[:, 0], torch.cross(su, E, dim=1) / (-4 * np.pi))
    A.index_add_(0, e[:, 1], torch.cross(sv, E, dim=1) / (-4 * np.pi))
    err = float((D - A).norm() / A.norm())
    print(f"[{kind} {n}] relative difference {err:.2e}", flush=True)
    assert err <= 1e-5
    sb = wn.SlicedBackward(Vt, Ft, grid=grid, vertex_sums=True)
    sb.begin()
    at = [0, 256, 256 * 700, 256 * 701, grid.size]
    for a, b in zip(at[:-1], at[1:]):
        sb.points(a, b - a, g)
    assert torch.equal(sb.end(), D)
    bad = g.clone()
    bad[grid.size // 2] = float("nan")
    assert bool(torch.isnan(wn.wn_backward(Vt, Ft, bad, grid=grid)[Ft.long()]).all())


@pytest.mark.parametrize("kind", ["closed", "reversed faces"])
def test_small_terms_beside_large_ones(dev, orc, kind):
    """A triangle 4e5 away, whose gradient is some 1e-15 of that of a triangle with a vertex 1e-7 from a
    voxel centre.  From the boundary edges: 1e-5 of its largest component, as alone (FP32 terms).  With
    edges that do not suit the path: its corner terms, which are its vertices', up to a rounding."""
    import paper_2407_11272_amd as wn
    V, F = _mesh(kind)
    V = np.asarray(V, np.float32)
    base, q = len(V), _centres(GRID)[5000]
    A = np.float32([q + [1e-7, 0, 0], q + [0.1, 0.2, 0.1], q + [-0.1, 0.1, 0.2]])
    B = np.float32([[4e5, 3e5, 1e5], [4e5 + 20, 3e5, 1e5 - 10], [4e5, 3e5 + 10, 1e5 + 20]])
    Vt, Ft = _dev(np.concatenate([V, A, B]), np.concatenate([F, [[base, base + 1, base + 2], [base + 3, base + 4, base + 5]]]))
    g = _weights(GRID.size)
    D = wn.wn_backward(Vt, Ft, g, grid=GRID).cpu().numpy().astype(np.float64)
    T = wn.wn_backward(Vt, Ft, g, grid=GRID, want_dLdT=True)[1][-1].cpu().numpy().astype(np.float64)
    _, Dr = orc.grad(B.astype(np.float64), np.arange(3)[None], _centres(GRID).astype(np.float64),
                     g.cpu().numpy().astype(np.float64))
    far, ref, tol = D[-3:], (Dr if kind == "closed" else T), (1e-5 if kind == "closed" else 2.0 ** -23)
    print(f"[{kind}] largest {np.abs(D).max():.1e}, far {np.abs(ref).max():.1e}, off by {np.abs(far - ref).max():.1e}", flush=True)
    assert 0 < np.abs(ref).max() < 1e-13 * np.abs(D).max()
    assert np.abs(far - ref).max() <= tol * np.abs(ref).max()


def _edge_sums64(V, F, Q, g):
    """The sum over the boundary edges in FP64, without the terms of points on an edge (P up to 1e-6 of the
    distance to the nearer end) or so close to an end that FP32 squares of the distance are 0; and the sum of its edges' absolute values."""
    import torch
    V, Q, g = (torch.as_tensor(np.asarray(x, np.float64)).cuda() for x in (V, Q, g))
    e = np.concatenate([F[:, [0, 1]], F[:, [1, 2]], F[:, [2, 0]]]).astype(np.int64)
    n = int(F.max()) + 1
    e = torch.as_tensor(e[~np.isin(e[:, 0] * n + e[:, 1], e[:, 1] * n + e[:, 0])]).cuda()
    out, scale = torch.zeros_like(V), torch.zeros_like(V)
    for i in range(0, len(e), 8):
        u, v = V[e[i:i + 8, 0]][:, None], V[e[i:i + 8, 1]][:, None]
        E, A, B = v - u, u - Q, v - Q
        L = E.norm(dim=2)
        a, b, AB = A.norm(dim=2), B.norm(dim=2), (A * B).sum(2)
        near = torch.where((b < a)[..., None], B, A)
        P = near - (near * E).sum(2, keepdim=True) / (L ** 2)[..., None] * E
        on = ((AB < 0) & (P.norm(dim=2) <= 1e-6 * torch.minimum(a, b))) | (torch.minimum(a, b) < 1e-20 * L)
        den = torch.where(AB < 0, (P * P).sum(2) * L ** 2 / (a * b - AB), a * b + AB)
        k = torch.where(on, 0.0, g / den)
        k = torch.nan_to_num(k, nan=0.0)
        su, sv = ((torch.nan_to_num(k / x, nan=0.0)[..., None] * P).sum(1) for x in (a, b))
        for end, x in ((0, su), (1, sv)):
            x = torch.linalg.cross(x, E[:, 0]) / (-4 * np.pi)
            out.index_add_(0, e[i:i + 8, end], x)
            scale.index_add_(0, e[i:i + 8, end], x.abs())
    return out.cpu().numpy(), scale.cpu().numpy()


LATTICE = wi.Grid((-0.5 - 1 / 64,) * 3, (0.5 - 1 / 64,) * 3, (32, 32, 32))   # voxel centres at multiples of 1/32


@pytest.mark.parametrize("scale", [0, -10, -33, 20])
def test_rim_through_voxel_centres(dev, scale):
    """A sheet in a layer of voxel centres, its rim through the middle of each of its edges there: the
    terms on the rim are left out, at every scale of the mesh (2^scale) alike."""
    import torch
    import paper_2407_11272_amd as wn
    n, h = 25, 1 / 32
    x = (np.arange(n) - n // 2 + 0.5) * h
    X, Y = np.meshgrid(x, (np.arange(n) - n // 2) * h, indexing="ij")
    V = np.stack([X, Y, np.full_like(X, 3 * h)], -1).reshape(-1, 3)
    a = (np.arange(n - 1)[:, None] * n + np.arange(n - 1)[None]).reshape(-1)
    F = np.concatenate([np.stack([a, a + n, a + n + 1], -1), np.stack([a, a + n + 1, a + 1], -1)])
    assert len(F) * LATTICE.size >= 2.0e7
    f = 2.0 ** scale
    grid = wi.Grid(tuple(f * np.array(LATTICE.lo)), tuple(f * np.array(LATTICE.hi)), LATTICE.n)
    g = _weights(grid.size)
    Vt, Ft = _dev(V * f, F)
    D = wn.wn_backward(Vt, Ft, g, grid=grid).cpu().numpy().astype(np.float64) * f
    Dr, _ = _edge_sums64(V, F, _centres(LATTICE), g.cpu().numpy())
    print(f"[rim 2^{scale}] |d dL/dV| {np.abs(D - Dr).max():.2e} of {np.abs(Dr).max():.2e}", flush=True)
    assert np.abs(D - Dr).max() <= 1e-5 * np.abs(Dr).max()


@pytest.mark.parametrize("n", [(25, 23, 27), (84, 80, 82)])
@pytest.mark.parametrize("kind", ["holes", "open end"])
def test_scale_of_the_mesh(dev, kind, n):
    """Powers of two scale every product exactly, so the gradient's bits do not depend on them."""
    import torch
    import paper_2407_11272_amd as wn
    V, F = _mesh(kind)
    grid = wi.Grid(GRID.lo, GRID.hi, n)
    g = _weights(grid.size)
    Vt, Ft = _dev(V, F)
    D = wn.wn_backward(Vt, Ft, g, grid=grid)
    assert D.any()
    for e in (-33, -10, 20):
        f = 2.0 ** e
        gs = wi.Grid(tuple(float(np.float32(x)) * f for x in grid.lo), tuple(float(np.float32(x)) * f for x in grid.hi), n)
        assert torch.equal(wn.wn_backward(Vt * f, Ft, g, grid=gs) * f, D)


def test_edges_within_rounding_of_a_voxel_centre(dev):
    """Vertices that differ from a voxel centre by less than the rounding of u - q (whose terms grow as
    1 / distance), and edges through one: FP32 terms, so 1e-4 of a vertex's largest edge (two edges of the
    thin triangle here cancel to 4e-4 of either at the vertex between them)."""
    import torch
    import paper_2407_11272_amd as wn
    V, F = _mesh("closed")
    q = np.array([0.125, -0.25, 0.0625])
    d = np.array([0.36, 0.48, 0.8])
    extra = np.array([
        [0.37, 0, 0], [6.1e-17, 0, 0], [0.2, 0.1, 0.3],             # an end
        [0.25, 0, 0.01], [0.25, 6e-24, 0.3125], [0.1, -0.4, 0.2],   # beside an end
        q - 5e-5 * d, q + 7e-5 * d, [0.3, 0.3, -0.2],               # through the centre
        [-0.25, 0.125, 0.124], [-0.25, 0.125, 0.126], [-0.2, 0, 0.1]])   # the centre is the middle of an edge
    base = len(V)
    V = np.concatenate([V, extra]).astype(np.float32)
    F = np.concatenate([F, base + np.arange(12).reshape(4, 3)])
    g = _weights(LATTICE.size)
    Vt, Ft = _dev(V, F)
    D = wn.wn_backward(Vt, Ft, g, grid=LATTICE).cpu().numpy().astype(np.float64)
    Dr, terms = _edge_sums64(V, F, _centres(LATTICE), g.cpu().numpy())
    assert np.isfinite(D).all() and not D[:base].any()
    rel = np.abs(D - Dr)[base:].max(1) / terms[base:].max(1)
    print("[near a centre] relative differences", " ".join(f"{x:.1e}" for x in rel), flush=True)
    assert rel.max() <= 1e-4


@pytest.mark.parametrize("distance", [1e-2, 1e-4, 1e-6])
def test_a_voxel_close_to_a_vertex(dev, distance):
    """The gradient that one voxel sends to a triangle whose vertex is `distance` of its edges away: R and
    P are formed from that vertex, so they keep their digits (2^-24 each, some ten of them)."""
    import torch
    import paper_2407_11272_amd as wn
    V, F = _mesh("closed")
    base = len(V)
    off = distance * 0.25 * np.array([0.48, -0.6, 0.64])
    V = np.concatenate([V, [np.array([0, 0.03125, 0]) + off, [0.21, 0.13, 0.05], [-0.11, 0.19, 0.12]]]).astype(np.float32)
    Vt, Ft = _dev(V, np.concatenate([F, [[base, base + 1, base + 2]]]))
    g = torch.zeros(LATTICE.n, device="cuda")
    g[16, 17, 16] = 1.0     # the centre (0, 1/32, 0)
    D = wn.wn_backward(Vt, Ft, g.reshape(-1), grid=LATTICE).cpu().numpy().astype(np.float64)
    Dr, _ = _edge_sums64(V, base + np.arange(3)[None], _centres(LATTICE), g.cpu().numpy().reshape(-1))
    rel = np.abs(D - Dr)[base:].max(1) / np.abs(Dr)[base:].max(1)
    print(f"[{distance:g} of an edge away] relative differences", " ".join(f"{x:.1e}" for x in rel), flush=True)
    assert rel.max() <= 1e-5


def test_ranges_share_the_work_of_large_grids(dev):
    """On grids that take blocks each range does the blocks that it completes, so none takes much more than
    its share of one call: the last of eight a quarter and the launches at most (it took all of it)."""
    import time
    import torch
    import paper_2407_11272_amd as wn
    V, F, _ = wi.ellipsoid_union(np.random.default_rng(1), 4, 4000)
    F = wi.delete_faces(F, 1600, np.random.default_rng(2))
    Vt, Ft = _dev(V, F)
    grid = wn.Grid((-0.5,) * 3, (0.5,) * 3, (128, 128, 128))
    g = _weights(grid.size)

    def timed(f):
        torch.cuda.synchronize()
        t = time.perf_counter()
        out = f()
        torch.cuda.synchronize()
        return out, time.perf_counter() - t
    wn.wn_backward(Vt, Ft, g, grid=grid)
    D, whole = timed(lambda: wn.wn_backward(Vt, Ft, g, grid=grid))
    sb = wn.SlicedBackward(Vt, Ft, grid=grid, vertex_sums=True)
    for _ in range(2):
        took = [timed(sb.begin)[1]]
        for i in range(8):
            took.append(timed(lambda: sb.points(i * grid.size // 8, grid.size // 8, g))[1])
        E, last = timed(sb.end)
        took.append(last)
    assert torch.equal(E, D)
    print(f"whole {1e3 * whole:.2f} ms, begin, ranges and end " + " ".join(f"{1e3 * t:.2f}" for t in took), flush=True)
    assert max(took[:-2]) <= 0.25 * whole + 2e-4 and took[-2] + took[-1] <= 0.25 * whole + 4e-4


def test_a_coordinate_that_is_not_finite_on_a_long_axis(dev):
    """The cells that hold a vertex are looked up within the rounding of their centres; a NaN has none (it went
    through all 4e6 cells of the axis, one by one)."""
    import time
    import torch
    import paper_2407_11272_amd as wn
    V, F = _mesh("holes")
    V = np.asarray(V, np.float32).copy()
    V[5, 0] = np.nan
    Vt, Ft = _dev(V, F)
    grid = wn.Grid((-0.5,) * 3, (0.5,) * 3, (1 << 22, 1, 1))
    g = torch.zeros(grid.size, device="cuda")
    few = wn.Grid((-0.5,) * 3, (0.5,) * 3, (1 << 14, 16, 16))   # as many points, short axes

    def timed(gr):
        wn.wn_backward(Vt, Ft, g, grid=gr)
        torch.cuda.synchronize()
        t = time.perf_counter()
        D = wn.wn_backward(Vt, Ft, g, grid=gr)
        torch.cuda.synchronize()
        return D, time.perf_counter() - t
    D, t = timed(grid)
    _, t0 = timed(few)
    assert torch.isnan(D[5]).any()
    assert t <= 1.5 * t0 + 1e-3
