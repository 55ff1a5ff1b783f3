"""The forward by the mesh's boundary (wn_cycle.hip) against the FP64 oracle and against the
all-pairs kernels.

Sizes are above the rule's line (128 faces, 5e7 pairs), where a grid call takes the path;
the same points as a point list take the all-pairs kernels.  Tolerances: |dW| <= 1e-4 off
the guard band, as for every forward; a voxel of a closed mesh that is not close to the
surface has an integer W exactly (a count of crossings, converted to FP32), and a
threshold's occupancy is the all-pairs kernel's bit for bit where W is within 1e-5 of it
(those voxels take the same sum in the same order)."""
import numpy as np
import pytest

import wn_inputs as wi

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2407_11272_amd as wn
    wn.wn_version()
    return torch.device("cuda", 0)


def _sphere(seed=0, sub=4):
    rng = np.random.default_rng(seed)
    V, F = wi.icosphere(sub)
    return wi.jitter(V * 0.4, 0.005, rng), F, rng


def _sheet(n=52):
    g = np.linspace(-0.43, 0.41, n)
    X, Y = np.meshgrid(g, g, indexing="ij")
    V = np.stack([X, Y, 0.1 * np.sin(7 * X) * np.cos(5 * Y)], -1).reshape(-1, 3)
    a = (np.arange(n - 1)[:, None] * n + np.arange(n - 1)[None]).reshape(-1)
    return V, np.concatenate([np.stack([a, a + n, a + n + 1], -1), np.stack([a, a + n + 1, a + 1], -1)])


def _mesh(kind):
    V, F, rng = _sphere()
    if kind == "closed":
        return V, F
    if kind == "holes":            # triangles, and neighbouring faces missing together
        return V, wi.delete_faces(F, 256, rng)
    if kind == "loop of 4":        # the longest short loop but two, and the shortest long one
        return V, np.delete(F, np.nonzero((F == F[0, 0]).any(1))[0][:2], axis=0)
    if kind in ("loops of 5 and 6", "loop of 7"):
        ring = {"loops of 5 and 6": [0, 700], "loop of 7": [0]}[kind]
        drop = np.isin(F, ring).any(1)
        if kind == "loop of 7":    # one more face, across an edge of the ring
            rim = set(F[drop].reshape(-1)) - {0}
            more = np.nonzero(~drop & (np.isin(F, list(rim)).sum(1) == 2))[0][0]
            drop[more] = True
        return V, F[~drop]
    if kind == "open end":         # one long loop
        return V, F[V[F].mean(1)[:, 2] < 0.15]
    if kind == "sheet":
        return _sheet()
    if kind == "two shells, one reversed":
        return np.concatenate([V, 0.5 * V]), np.concatenate([F, F[:, ::-1] + len(V)])
    if kind == "repeated":         # some faces three times: edges used twice the same way
        return V, np.concatenate([F, F[:40], F[:40]])
    if kind == "reversed faces":   # inconsistent winding: edges that do not cancel
        F = F.copy()
        F[::50] = F[::50][:, ::-1]
        return V, F
    raise ValueError(kind)


KINDS = ["closed", "holes", "loop of 4", "loops of 5 and 6", "loop of 7", "open end", "sheet",
         "two shells, one reversed", "repeated", "reversed faces"]
GRID = wi.Grid((-0.5, -0.45, -0.5), (0.5, 0.5, 0.47), (25, 23, 27))


def _dev(V, F):
    import torch
    import paper_2407_11272_amd as wn
    return wn.as_mesh(torch.as_tensor(np.asarray(V, np.float32)), torch.as_tensor(np.ascontiguousarray(F)))


def _strips(V, F):
    import torch
    import paper_2407_11272_amd as wn
    return torch.as_tensor(wn.wn_build_strips(np.ascontiguousarray(F), len(V))).cuda()


def _centres(grid):
    """The FP32 voxel centres that the kernels form."""
    ax = []
    for d in range(3):
        lo, h = np.float32(grid.lo[d]), np.float32((np.float64(np.float32(grid.hi[d])) - np.float64(np.float32(grid.lo[d]))) / grid.n[d])
        ax.append(((np.arange(grid.n[d]) + 0.5) * np.float64(h) + np.float64(lo)).astype(np.float32))
    return np.stack(np.meshgrid(*ax, indexing="ij"), -1).reshape(-1, 3)


@pytest.mark.parametrize("kind", KINDS)
def test_boundary_path_vs_oracle_and_all_pairs(dev, orc, kind):
    import torch
    import paper_2407_11272_amd as wn
    V, F = _mesh(kind)
    assert len(F) * GRID.size >= 5.0e7
    Vt, Ft = _dev(V, F)
    R = _strips(V, F)
    Q = _centres(GRID)
    Qt = torch.as_tensor(Q).cuda()
    V64 = np.asarray(V, np.float32).astype(np.float64)
    Wr = orc.winding(V64, F, Q.astype(np.float64))
    guard = orc.guard_mask(V64, F, Q.astype(np.float64))
    for strips in (None, R):
        def call(**kw):
            return wn.wn_voxelize(Vt, Ft, **kw) if strips is None else wn.wn_voxelize_strips(Vt, Ft, strips, **kw)
        W, occ = call(grid=GRID, occupancy="threshold")
        Ws, soft = call(grid=GRID, occupancy="sigmoid", k=20.0)
        P = call(Q=Qt)
        assert wn.wn_get_device_error() == 0
        Wg = W.cpu().numpy().reshape(-1)
        err = np.abs(Wg - Wr)
        print(f"[{kind}] max |dW| {err[~guard].max():.2e}, all pairs {np.abs(P.cpu().numpy() - Wr)[~guard].max():.2e}",
              flush=True)
        assert err[~guard].max() <= 1e-4
        m = ~guard & (np.abs(Wr - 0.5) > 1e-3)
        np.testing.assert_array_equal(occ.cpu().numpy().reshape(-1)[m], orc.occupancy_threshold(Wr)[m])
        # on the sigmoid's slope this call's field is the all-pairs sum
        torch.testing.assert_close(soft, wn.wn_occupancy(Ws, "sigmoid", 0.5, 20.0), rtol=0, atol=0)
        assert np.abs(Ws.cpu().numpy().reshape(-1) - Wr)[~guard].max() <= 1e-4
        if kind in ("closed", "two shells, one reversed"):
            exact = Wg == np.round(Wg)
            assert exact.mean() > 0.99 and np.abs(Wg - np.round(Wr))[exact].max() == 0.0
        again = call(grid=GRID)
        torch.testing.assert_close(again, W, rtol=0, atol=0)


@pytest.mark.parametrize("kind,tau,res", [("closed", 0.0, (24, 25, 26)), ("closed", 1.0, (24, 25, 26)),
                                          ("closed", 0.0, (52, 51, 50)), ("holes", 0.5, (24, 25, 26))])
def test_voxels_at_the_threshold_take_the_all_pairs_sum(dev, kind, tau, res):
    """tau = 0 or 1 puts most voxels of a closed mesh within rounding of the threshold; the
    finer grid has more of them than the list holds (65 536), so the all-pairs kernels run
    for the marked voxels.  Either way they get the all-pairs bits, in plain and batched
    launches (which split the sum in their own ways)."""
    import torch
    import paper_2407_11272_amd as wn
    V, F = _mesh(kind)
    Vt, Ft = _dev(V, F)
    grid = wi.Grid((-0.5,) * 3, (0.5,) * 3, res)
    Q = torch.as_tensor(_centres(grid)).cuda()
    for strips in (None, _strips(V, F)):
        def call(**kw):
            return wn.wn_voxelize(Vt, Ft, **kw) if strips is None else wn.wn_voxelize_strips(Vt, Ft, strips, **kw)
        W, occ = call(grid=grid, occupancy="threshold", tau=tau)
        P, pocc = call(Q=Q, occupancy="threshold", tau=tau)
        at = (P - tau).abs() < 5e-6
        if kind == "closed":
            assert int(at.sum()) > (65536 if res[0] > 50 else 500)
        torch.testing.assert_close(W.reshape(-1)[at], P[at], rtol=0, atol=0)
        torch.testing.assert_close(occ.reshape(-1), pocc, rtol=0, atol=0)
        job = wn.MeshJob(Vt, Ft, wn.Grid.of(grid), "threshold", tau=tau, strips=strips)
        wn.wn_voxelize_batched([job])
        assert float((job.W - W).abs().max()) <= 2e-6
        assert int((job.occ != occ).sum()) <= int(at.sum())


def test_slices_are_the_whole_grid_bit_for_bit(dev):
    """Slices that begin and end inside a column, in one batch with the whole grid."""
    import torch
    import paper_2407_11272_amd as wn
    V, F = _mesh("holes")
    Vt, Ft = _dev(V, F)
    R = _strips(V, F)
    g = wn.Grid.of(GRID)
    whole = wn.MeshJob(Vt, Ft, g, "threshold", strips=R)
    W = torch.full(GRID.n, float("nan"), device="cuda")
    occ = torch.full(GRID.n, 9, dtype=torch.uint8, device="cuda")
    cuts = [0, 1, 40, 41 * 27, 4000, 4013, GRID.size - 1, GRID.size]
    parts = [wn.MeshJob(Vt, Ft, g, "threshold", W=W, occ=occ, point_begin=a, point_count=b - a, strips=R)
             for a, b in zip(cuts[:-1], cuts[1:])]
    wn.wn_voxelize_batched(parts + [whole])
    torch.cuda.synchronize()
    assert torch.equal(W, whole.W) and torch.equal(occ, whole.occ)


def test_streams_and_meshes_that_go_all_pairs(dev):
    """A stream that leaves out faces, coordinates that are not finite or out of range, and a
    face soup give what the all-pairs kernels give, bit for bit."""
    import torch
    import paper_2407_11272_amd as wn
    V, F = _mesh("closed")
    Q = torch.as_tensor(_centres(GRID)).cuda()
    R = wn.wn_build_strips(F, len(V))
    part = torch.as_tensor(R[:len(R) // 2].copy()).cuda()
    Vt, Ft = _dev(V, F)
    # (the strips' own split depends on the points alone, so both calls sum alike)
    torch.testing.assert_close(wn.wn_voxelize_strips(Vt, Ft, part, grid=GRID).reshape(-1),
                               wn.wn_voxelize_strips(Vt, Ft, part, Q=Q), rtol=0, atol=0)
    rng = np.random.default_rng(3)
    soup = (rng.uniform(-0.5, 0.5, (6000, 3)), rng.integers(0, 6000, (6000, 3)))
    for name, (v, f) in {"nan": (V.copy(), F), "inf": (V.copy(), F), "far": (V.copy(), F), "soup": soup}.items():
        if name != "soup":
            v[17] = {"nan": np.nan, "inf": np.inf, "far": 3e9}[name]
        vt, ft = _dev(v, f)
        torch.testing.assert_close(wn.wn_voxelize(vt, ft, grid=GRID).reshape(-1), wn.wn_voxelize(vt, ft, Q=Q),
                                   rtol=0, atol=0, equal_nan=True)


def test_voxels_on_the_surface(dev, orc):
    """A box of 6 x 32 x 32 quads whose sides lie on layers of voxel centres, so that voxels
    fall on faces, edges and vertices: what the all-pairs kernels give, and W exact off the
    sides."""
    import torch
    import paper_2407_11272_amd as wn
    n = 33
    g = np.linspace(-0.25, 0.25, n)
    A, B = np.meshgrid(g, g, indexing="ij")
    V, F = [], []
    a = (np.arange(n - 1)[:, None] * n + np.arange(n - 1)[None]).reshape(-1)
    quads = np.concatenate([np.stack([a, a + n, a + n + 1], -1), np.stack([a, a + n + 1, a + 1], -1)])
    for d in range(3):
        for s in (-0.25, 0.25):
            P = np.zeros((n * n, 3))
            P[:, d], P[:, (d + 1) % 3], P[:, (d + 2) % 3] = s, A.reshape(-1), B.reshape(-1)
            F.append((quads if s > 0 else quads[:, ::-1]) + len(V) * n * n)
            V.append(P)
    V, F = np.concatenate(V), np.concatenate(F)
    V, inv = np.unique(V, axis=0, return_inverse=True)   # welded
    F = inv.reshape(-1)[F]
    lo = -0.25 - 8.5 / 32   # cell 8's centre is -0.25 and cell 24's 0.25, exactly
    grid = wi.Grid((lo,) * 3, (lo + 1,) * 3, (32, 32, 32))
    Q = _centres(grid)
    Vt, Ft = _dev(V, F)
    W = wn.wn_voxelize(Vt, Ft, grid=grid).cpu().numpy().reshape(-1)
    P = wn.wn_voxelize(Vt, Ft, Q=torch.as_tensor(Q).cuda()).cpu().numpy()
    on = np.abs(Q).max(1) == 0.25
    assert on.sum() > 500
    np.testing.assert_array_equal(W[on], P[on])
    np.testing.assert_array_equal(W[~on], (np.abs(Q).max(1) < 0.25)[~on].astype(np.float32))


@pytest.mark.parametrize("n", [(78, 74, 83), (213, 6, 370), (450, 3, 350)])
@pytest.mark.parametrize("kind", ["holes", "open end", "sheet", "two shells, one reversed"])
def test_blocks_of_voxels(dev, orc, kind, n):
    """Grids above the blocks' line (2^18 voxels, 1.5e9 pairs): the caps' far field comes from
    nodes.  Ragged last blocks, and axes with fewer voxels than fine and than coarse nodes.

    Tolerance: the rule takes at most 10 x 4e-8 per far triangle, of either sign; the 300
    triangles here add up to 10 x 4e-8 x sqrt(300) = 7e-6 at most.  Off the surface the FP32
    forms add less than 3e-6 (as at the other sizes of this file)."""
    import torch
    import paper_2407_11272_amd as wn
    V, F = _mesh(kind)
    grid = wi.Grid((-0.5, -0.45, -0.5), (0.5, 0.5, 0.47), n)
    assert grid.size >= 1 << 18 and len(F) * grid.size >= 1.5e9
    Vt, Ft = _dev(V, F)
    W, occ = wn.wn_voxelize(Vt, Ft, grid=grid, occupancy="threshold")
    Q = _centres(grid)
    pick = np.random.default_rng(5).choice(grid.size, 4000, replace=False)
    V64 = np.asarray(V, np.float32).astype(np.float64)
    Wr = orc.winding(V64, F, Q[pick].astype(np.float64))
    guard = orc.guard_mask(V64, F, Q[pick].astype(np.float64))
    Wg = W.cpu().numpy().reshape(-1)[pick]
    err = np.abs(Wg - Wr)[~guard]
    print(f"[{kind} {n}] max |dW| {err.max():.2e}, rms {np.sqrt((err ** 2).mean()):.2e}", flush=True)
    assert err.max() <= 1e-5
    m = ~guard & (np.abs(Wr - 0.5) > 1e-4)
    np.testing.assert_array_equal(occ.cpu().numpy().reshape(-1)[pick][m], orc.occupancy_threshold(Wr)[m])
    # a call without occupancy, a batch and slices of it: the same bits, but at voxels near the
    # threshold, which only a call with one lists, and listed voxels of the batch (its own chunks)
    again = wn.wn_voxelize(Vt, Ft, grid=grid)
    assert bool(((again == W) | ((W - 0.5).abs() < 2e-5)).all())
    g = wn.Grid.of(grid)
    whole = wn.MeshJob(Vt, Ft, g, "threshold")
    S = torch.full(n, float("nan"), device="cuda")
    cuts = [0, 5, n[1] * n[2] * 17 + 31, grid.size]
    parts = [wn.MeshJob(Vt, Ft, g, "none", W=S, point_begin=a, point_count=b - a) for a, b in zip(cuts[:-1], cuts[1:])]
    wn.wn_voxelize_batched(parts + [whole])
    torch.cuda.synchronize()
    assert float((W - whole.W).abs().max()) <= 2e-6 and float((W != whole.W).float().mean()) < 0.01
    assert bool(((S == whole.W) | ((whole.W - 0.5).abs() < 2e-5)).all())


@pytest.mark.parametrize("kind", KINDS)
def test_lists_of_points(dev, orc, kind):
    """Lists above the points' line (1.5e8 pairs): points over the whole box, on and very near the
    surface, on its vertices, far away, on a line through it along z, and with coordinates that
    are not finite.

    Off the guard band |dW| <= 1e-4 as for every forward; points on the surface or not finite take
    the all-pairs sum, so shorter lists (below the line) give their W up to the splits' order."""
    import torch
    import paper_2407_11272_amd as wn
    V, F = _mesh(kind)
    rng = np.random.default_rng(11)
    T = V[F]
    f = rng.integers(0, len(F), 4000)
    b = rng.dirichlet([1, 1, 1], 4000)
    on = np.einsum("ij,ijk->ik", b, T[f])
    line = np.stack([np.full(40, 0.013), np.full(40, -0.021), np.linspace(-0.6, 0.6, 40)], -1)
    odd = np.array([[np.nan, 0, 0], [0, np.inf, 0], [0.1, 0.1, -np.inf], [1e12, 0, 0], [0.0, 0.0, -3e9]])
    n = int(1.6e8 / len(F)) + 1
    Q = np.concatenate([rng.uniform(-0.6, 0.6, (n, 3)), on, on + 1e-5 * rng.standard_normal(on.shape), V[:500], line,
                        rng.uniform(-40, 40, (500, 3)), odd]).astype(np.float32)
    order = rng.permutation(len(Q))
    Q, surface = Q[order], (order >= n) & (order < n + len(on))
    assert len(F) * len(Q) >= 1.5e8
    Vt, Ft = _dev(V, F)
    Qt = torch.as_tensor(Q).cuda()
    W, occ = wn.wn_voxelize(Vt, Ft, Q=Qt, occupancy="threshold")
    Ws = wn.wn_voxelize_strips(Vt, Ft, _strips(V, F), Q=Qt)
    assert wn.wn_get_device_error() == 0
    step = 8192
    assert len(F) * step < 1.5e8
    A = torch.cat([wn.wn_voxelize(Vt, Ft, Q=Qt[i:i + step].contiguous()) for i in range(0, len(Q), step)])
    ok = np.isfinite(Q).all(1) & (np.abs(Q) < 1e9).all(1)
    torch.testing.assert_close(W.cpu()[~ok], A.cpu()[~ok], rtol=0, atol=2e-6, equal_nan=True)
    pick = np.nonzero(ok)[0][rng.permutation(int(ok.sum()))[:6000]]
    V64 = np.asarray(V, np.float32).astype(np.float64)
    Wr = orc.winding(V64, F, Q[pick].astype(np.float64))
    guard = orc.guard_mask(V64, F, Q[pick].astype(np.float64))
    for X in (W, Ws):
        x = X.cpu().numpy()[pick]
        print(f"[points {kind}] {len(Q)} off-guard {np.abs(x - Wr)[~guard].max():.2e} on-guard {guard.sum()}", flush=True)
        assert np.abs(x - Wr)[~guard].max() <= 1e-4
    assert float((W - A).abs()[torch.as_tensor(surface).cuda()].max()) <= 2e-6
    m = ~guard & (np.abs(Wr - 0.5) > 1e-3)
    np.testing.assert_array_equal(occ.cpu().numpy()[pick][m], orc.occupancy_threshold(Wr)[m])


def test_points_that_crowd_take_all_pairs(dev):
    """More points in one square than a bin holds: the all-pairs sum, bit for bit what a
    list in another order gives."""
    import torch
    import paper_2407_11272_amd as wn
    V, F = _mesh("holes")
    Vt, Ft = _dev(V, F)
    Q = np.random.default_rng(2).uniform(-0.01, 0.01, (40000, 3)).astype(np.float32)
    Q[:, 2] *= 50
    p = np.random.default_rng(3).permutation(len(Q))
    W = wn.wn_voxelize(Vt, Ft, Q=torch.as_tensor(Q).cuda())
    torch.testing.assert_close(wn.wn_voxelize(Vt, Ft, Q=torch.as_tensor(Q[p]).cuda()), W[torch.as_tensor(p).cuda()],
                               rtol=0, atol=0)
    A = torch.cat([wn.wn_voxelize(Vt, Ft, Q=torch.as_tensor(Q[i:i + 8000]).cuda()) for i in range(0, len(Q), 8000)])
    assert float((W - A).abs().max()) <= 2e-6
