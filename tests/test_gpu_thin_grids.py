"""Grids of short columns and few large faces over many columns, through the mesh's boundary.

Against the all-pairs kernels: |dW| <= 2e-6 (both are FP32 sums with errors of some 5e-7), and slices
against the whole grid bit for bit."""
import numpy as np
import pytest

import wn_inputs as wi
from .test_gpu_cycle import _dev, _mesh, _sheet
from .test_gpu_long_loops import all_pairs, fan

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2407_11272_amd as wn
    wn.wn_version()
    return torch.device("cuda", 0)


@pytest.mark.parametrize("n2", [1, 2, 3, 5, 16, 21, 22, 31, 32, 33, 63, 64, 65, 130])
def test_short_columns(dev, n2):
    """As many columns per wave as it has lanes for up to 32 voxels each, one beyond."""
    import torch
    import paper_2407_11272_amd as wn
    V, F = _mesh("holes")
    Vt, Ft = _dev(V, F)
    n1 = 83
    n0 = int(np.ceil(3.1e7 / (len(F) * n1 * n2))) + 2
    grid = wn.Grid((-0.5, -0.45, -0.31), (0.5, 0.5, 0.37), (n0, n1, n2))
    W, occ = wn.wn_voxelize(Vt, Ft, grid=grid, occupancy="threshold")
    A, aocc = all_pairs(Vt, Ft, grid, occupancy=1)
    assert float((W - A).abs().max()) <= 2e-6
    assert int((occ != aocc).sum()) == 0
    g = wn.Grid.of(grid)
    whole = wn.MeshJob(Vt, Ft, g, "threshold")
    S = torch.full(grid.n, float("nan"), device="cuda")
    so = torch.full(grid.n, 9, dtype=torch.uint8, device="cuda")
    P = grid.size
    cuts = sorted({0, 1, n2 + 1, P // 3, P // 2 + 1, P - 1, P})
    wn.wn_voxelize_batched([wn.MeshJob(Vt, Ft, g, "threshold", W=S, occ=so, point_begin=a, point_count=b - a)
                            for a, b in zip(cuts[:-1], cuts[1:])] + [whole])
    torch.cuda.synchronize()
    assert torch.equal(S, whole.W) and torch.equal(so, whole.occ)


def _box(k):
    """A box of 12 k^2 faces."""
    g = np.linspace(-0.4, 0.4, k + 1)
    A, B = np.meshgrid(g, g, indexing="ij")
    a = (np.arange(k)[:, None] * (k + 1) + np.arange(k)[None]).reshape(-1)
    q = np.concatenate([np.stack([a, a + k + 1, a + k + 2], -1), np.stack([a, a + k + 2, a + 1], -1)])
    V, F = [], []
    for d in range(3):
        for s in (-0.4, 0.4):
            P = np.zeros(((k + 1) ** 2, 3))
            P[:, d], P[:, (d + 1) % 3], P[:, (d + 2) % 3] = s, A.reshape(-1), B.reshape(-1)
            F.append((q if s > 0 else q[:, ::-1]) + len(V) * (k + 1) ** 2)
            V.append(P)
    V, inv = np.unique(np.concatenate(V).round(9), axis=0, return_inverse=True)
    return V, inv.reshape(-1)[np.concatenate(F)]


LARGE = {"box": lambda: _box(4), "sheet": lambda: _sheet(11), "fan": lambda: fan(200),
         "soup": lambda: (np.random.default_rng(3).uniform(-0.5, 0.5, (450, 3)), np.arange(450).reshape(-1, 3))}


@pytest.mark.parametrize("n", [(2000, 2000, 1), (700, 700, 10)])
@pytest.mark.parametrize("kind", list(LARGE))
def test_few_large_faces_over_a_wide_plane(dev, kind, n):
    """A face here meets up to four million columns: they are shared out over the raster list whatever it
    holds.  Off the closest points W is the all-pairs kernels' to 1e-4 (large faces leave those some 1e-5), and a
    call takes at most three times theirs (one face's columns on eight lanes took it 15 to 200 times)."""
    import time
    import torch
    import paper_2407_11272_amd as wn
    V, F = LARGE[kind]()
    Vt, Ft = _dev(V, F)
    grid = wn.Grid((-0.5,) * 3, (0.5,) * 3, n)
    assert len(F) >= 128 and len(F) * grid.size >= 3.0e7

    def timed(f):
        f()
        torch.cuda.synchronize()
        t = time.perf_counter()
        out = f()
        torch.cuda.synchronize()
        return out, time.perf_counter() - t
    A = all_pairs(Vt, Ft, grid)
    few = wn.as_mesh(Vt, Ft[:127].contiguous())    # below the path's line: all pairs, and a little less than these faces take
    _, ta = timed(lambda: wn.wn_voxelize(*few, grid=grid))
    W, tw = timed(lambda: wn.wn_voxelize(Vt, Ft, grid=grid))
    d = (W - A).abs().reshape(-1)
    print(f"[{kind} {n}] {1e3 * tw:.2f} ms, all pairs {1e3 * ta * len(F) / 127:.2f} ms; |dW| {float(d.max()):.1e}", flush=True)
    assert float((d > 1e-4).float().mean()) <= 1e-5
    assert tw <= 3.0 * ta * len(F) / 127
