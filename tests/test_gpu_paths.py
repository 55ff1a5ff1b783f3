"""The boundary path against the all-pairs kernels themselves: the C entry point takes those alone where the
workspace has no room for the path.  (A list of the same points takes the path too from
1.5e8 pairs on.)"""
import numpy as np
import pytest

import wn_inputs as wi
from .test_gpu_cycle import _centres, _dev, _mesh, _strips
from .test_gpu_long_loops import all_pairs
from .test_gpu_thin_grids import _box

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2407_11272_amd as wn
    wn.wn_version()
    return torch.device("cuda", 0)


@pytest.mark.parametrize("strips", [False, True])
@pytest.mark.parametrize("kind,tau,res", [("closed", 0.0, (24, 25, 26)), ("closed", 1.0, (24, 25, 26)),
                                          ("closed", 0.0, (52, 51, 50)), ("holes", 0.5, (24, 25, 26)),
                                          ("closed", 0.0, (70, 66, 68))])
def test_voxels_at_the_threshold(dev, kind, tau, res, strips):
    """Those within rounding of the threshold get the all-pairs bits, one by one or, where the list is full (the
    finer grids: 132600 and 314160 voxels, most of them at tau), from the kernels run for the marked voxels."""
    import torch
    import paper_2407_11272_amd as wn
    V, F = _mesh(kind)
    Vt, Ft = _dev(V, F)
    R = _strips(V, F) if strips else None
    grid = wi.Grid((-0.5,) * 3, (0.5,) * 3, res)
    assert len(F) * grid.size >= 7.0e7
    kw = dict(grid=grid, occupancy="threshold", tau=tau)
    W, occ = wn.wn_voxelize(Vt, Ft, **kw) if R is None else wn.wn_voxelize_strips(Vt, Ft, R, **kw)
    A, aocc = all_pairs(Vt, Ft, grid, R, occupancy=1, tau=tau)
    at = (A - tau).abs() < 5e-6
    if kind == "closed":
        assert int(at.sum()) > (65536 if res[0] > 50 else 500)
    assert torch.equal(W[at], A[at]) and torch.equal(occ, aocc)
    assert not torch.equal(W, A) or bool(at.all())


@pytest.mark.parametrize("strips", [False, True])
def test_a_sigmoid_s_slope(dev, strips):
    """With k > 10 the voxels within min(10 / k, 1 / 4) of tau get the all-pairs bits."""
    import torch
    import paper_2407_11272_amd as wn
    V, F = _mesh("holes")
    Vt, Ft = _dev(V, F)
    R = _strips(V, F) if strips else None
    grid = wi.Grid((-0.5,) * 3, (0.5,) * 3, (30, 29, 31))
    assert len(F) * grid.size >= 7.0e7
    for k in (11.0, 50.0, 400.0):
        kw = dict(grid=grid, occupancy="sigmoid", k=k)
        W, occ = wn.wn_voxelize(Vt, Ft, **kw) if R is None else wn.wn_voxelize_strips(Vt, Ft, R, **kw)
        A, aocc = all_pairs(Vt, Ft, grid, R, occupancy=2, k=k)
        slope = (A - 0.5).abs() < 0.99 * min(10.0 / k, 0.25)
        assert bool(slope.any())
        assert torch.equal(W[slope], A[slope]) and torch.equal(occ[slope], aocc[slope])


def test_voxels_on_faces_edges_and_vertices(dev):
    """A box of 6 x 16 x 16 quads whose sides lie on layers of voxel centres."""
    import torch
    import paper_2407_11272_amd as wn
    V, F = _box(16)
    V = V * 0.625      # sides at -0.25 and 0.25
    lo = -0.25 - 8.5 / 32
    grid = wi.Grid((lo,) * 3, (lo + 1,) * 3, (32, 32, 32))
    Vt, Ft = _dev(V, F)
    for R in (None, _strips(V, F)):
        W = wn.wn_voxelize(Vt, Ft, grid=grid) if R is None else wn.wn_voxelize_strips(Vt, Ft, R, grid=grid)
        on = torch.as_tensor((np.abs(_centres(grid)).max(1) == 0.25).reshape(grid.n)).cuda()
        assert int(on.sum()) > 500
        assert torch.equal(W[on], all_pairs(Vt, Ft, grid, R)[on])


@pytest.mark.parametrize("n", [(29, 28, 30), (78, 74, 83)])
@pytest.mark.parametrize("kind", ["holes", "open end", "sheet", "loops of 5 and 6"])
def test_long_and_short_loops_with_and_without_strips(dev, orc, kind, n):
    """Both calls above their lines (3e7, and 7e7 with strips), one by one and in blocks: |dW| <= 1e-4 off the
    guard band, as for every forward, and not the all-pairs sum."""
    import torch
    import paper_2407_11272_amd as wn
    V, F = _mesh(kind)
    grid = wi.Grid((-0.5, -0.45, -0.5), (0.5, 0.5, 0.47), n)
    assert len(F) * grid.size >= 7.0e7
    Vt, Ft = _dev(V, F)
    Q = _centres(grid).astype(np.float64)
    pick = np.random.default_rng(5).choice(grid.size, 4000, replace=False)
    V64 = np.asarray(V, np.float32).astype(np.float64)
    Wr = orc.winding(V64, F, Q[pick])
    guard = orc.guard_mask(V64, F, Q[pick])
    for R in (None, _strips(V, F)):
        W = wn.wn_voxelize(Vt, Ft, grid=grid) if R is None else wn.wn_voxelize_strips(Vt, Ft, R, grid=grid)
        assert not torch.equal(W, all_pairs(Vt, Ft, grid, R))
        err = np.abs(W.cpu().numpy().reshape(-1)[pick] - Wr)[~guard]
        print(f"[{kind} {n} {'strips' if R is not None else 'faces'}] max |dW| {err.max():.2e}", flush=True)
        assert err.max() <= 1e-4


@pytest.mark.parametrize("n", [(29, 28, 30), (78, 74, 83)])
@pytest.mark.parametrize("kind", ["closed", "holes", "open end"])
def test_scale_of_the_mesh(dev, kind, n):
    """Powers of two scale every product exactly, so W's bits do not depend on them while the products of two
    faces' terms (the sixth power of a length) stay normal numbers; at 1e-10 and 4e6 those leave FP32's range and
    two angles are added instead, which moves W by the rounding of each."""
    import torch
    import paper_2407_11272_amd as wn
    V, F = _mesh(kind)
    grid = wi.Grid((-0.5, -0.45, -0.5), (0.5, 0.5, 0.47), n)
    Vt, Ft = _dev(V, F)
    R = _strips(V, F)
    for strips in (None, R):
        def call(v, g):
            return wn.wn_voxelize(v, Ft, grid=g) if strips is None else wn.wn_voxelize_strips(v, Ft, strips, grid=g)
        W = call(Vt, grid)
        assert not torch.equal(W, all_pairs(Vt, Ft, grid, strips))
        for e in (-33, -10, 15, 22):
            f = 2.0 ** e
            gs = wi.Grid(tuple(float(np.float32(x)) * f for x in grid.lo), tuple(float(np.float32(x)) * f for x in grid.hi), n)
            Ws = call(Vt * f, gs)
            assert torch.equal(Ws, W) if e in (-10, 15) else float((Ws - W).abs().max()) <= 2e-6, e


@pytest.mark.parametrize("scale", [1e-3, 1e4, 1e7])
def test_any_scale(dev, scale):
    """Other factors round the coordinates anew, as for the all-pairs sum."""
    import torch
    import paper_2407_11272_amd as wn
    V, F = _mesh("holes")
    grid = wi.Grid((-0.5, -0.45, -0.5), (0.5, 0.5, 0.47), (40, 41, 42))
    gs = wi.Grid(tuple(np.float32(x * scale) for x in grid.lo), tuple(np.float32(x * scale) for x in grid.hi), grid.n)
    Vt, Ft = _dev(V, F)
    Vs, _ = _dev(np.asarray(V) * scale, F)
    d = (wn.wn_voxelize(Vs, Ft, grid=gs) - wn.wn_voxelize(Vt, Ft, grid=grid)).abs()
    a = (all_pairs(Vs, Ft, wn.Grid.of(gs)) - all_pairs(Vt, Ft, grid)).abs()
    print(f"[scale {scale:g}] 99.9 % {float(d.flatten().quantile(0.999)):.1e}, all pairs {float(a.flatten().quantile(0.999)):.1e}", flush=True)
    assert float(d.flatten().quantile(0.999)) <= 1e-4
