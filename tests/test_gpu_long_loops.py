"""Boundaries that are long loops (ribbons, tubes, sheets): the forward joins them by walking short
loops and by doubling long ones, in LDS up to 4096 edges and in global memory beyond.

Against the FP64 oracle, |dW| <= 1e-4 off the guard band as for every forward; a face order does not
change the loops, only where they start, so shuffled faces are held to the same."""
import numpy as np
import pytest

import wn_inputs as wi
from .test_gpu_cycle import _centres, _dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2407_11272_amd as wn
    wn.wn_version()
    return torch.device("cuda", 0)


def ribbon(n, w):
    """n quads along a winding band, w across: one loop of 2 (n + w) edges, faces in order along it."""
    t, y = np.meshgrid(np.linspace(0, 1, n + 1), np.linspace(-1, 1, w + 1), indexing="ij")
    a, r = 11 * np.pi * t, 0.12 + 0.3 * t
    V = np.stack([r * np.cos(a), r * np.sin(a), 0.07 * y + 0.05 * np.sin(3 * a)], -1).reshape(-1, 3)
    a = (np.arange(n)[:, None] * (w + 1) + np.arange(w)[None]).reshape(-1)
    b = a + w + 1
    return V, np.stack([np.stack([a, b, b + 1], -1), np.stack([a, b + 1, a + 1], -1)], 1).reshape(-1, 3)


def tubes(lengths, h=6):
    """Open tubes side by side with loops of the given lengths at both ends, and the other way round inside
    one another in pairs."""
    V, F, base = [], [], 0
    for i, n in enumerate(lengths):
        a = 2 * np.pi * np.arange(n) / n
        for k in range(h + 1):
            V.append(np.stack([0.04 * np.cos(a) + 0.11 * (i % 8) - 0.39, 0.04 * np.sin(a) + 0.21 * (i // 8) - 0.3,
                               np.full(n, -0.4 + 0.7 * k / h)], -1))
        p = (np.arange(h)[:, None] * n + np.arange(n)[None]).reshape(-1)
        q = (np.arange(h)[:, None] * n + (np.arange(n)[None] + 1) % n).reshape(-1)
        f = np.concatenate([np.stack([p, q, q + n], -1), np.stack([p, q + n, p + n], -1)]) + base
        F.append(f if i % 2 == 0 else f[:, ::-1])
        base += (h + 1) * n
    return np.concatenate(V), np.concatenate(F)


MESHES = {"ribbon of 3016 edges": lambda: ribbon(1500, 8), "ribbon of 12016 edges": lambda: ribbon(6000, 8),
          "tubes, 3 to 8": lambda: tubes([3, 4, 5, 6, 7, 8] * 4),
          "tubes about the walk's length": lambda: tubes([31, 32, 33, 34, 63, 64, 65, 66, 7, 100]),
          "tubes, more edges than LDS holds": lambda: tubes([5, 33, 900, 3, 700, 64, 1025, 6])}


@pytest.mark.parametrize("shuffled", [False, True])
@pytest.mark.parametrize("kind", list(MESHES))
def test_long_loops(dev, orc, kind, shuffled):
    import torch
    import paper_2407_11272_amd as wn
    V, F = MESHES[kind]()
    if shuffled:
        F = F[np.random.default_rng(4).permutation(len(F))]
    grid = wi.Grid((-0.5, -0.48, -0.5), (0.5, 0.52, 0.47), (40, 41, 42))
    assert len(F) * grid.size >= 3.0e7
    Vt, Ft = _dev(V, F)
    W = wn.wn_voxelize(Vt, Ft, grid=grid)
    assert not torch.equal(W, all_pairs(Vt, Ft, wn.Grid.of(grid)))  # (the path was taken)
    W = W.cpu().numpy().reshape(-1)
    Q = _centres(grid).astype(np.float64)
    pick = np.random.default_rng(5).choice(grid.size, min(grid.size, 3000), replace=False)
    V64 = np.asarray(V, np.float32).astype(np.float64)
    Wr = orc.winding(V64, F, Q[pick])
    guard = orc.guard_mask(V64, F, Q[pick])
    err = np.abs(W[pick] - Wr)[~guard]
    print(f"[{kind}] {len(F)} faces, max |dW| {err.max():.2e}", flush=True)
    assert err.max() <= 1e-4


def test_an_ordered_ribbon_takes_milliseconds(dev):
    """5e5 faces and 50 020 boundary edges in one loop, numbered along it: about 34 rounds of 49 edges per
    thread.  Walks to the next lower edge were 1.2e6 loads in a row, 0.4 s at 300 ns each; the bar is a
    quarter of that."""
    import time
    import torch
    import paper_2407_11272_amd as wn
    V, F = ribbon(25000, 10)
    Vt, Ft = _dev(V, F)
    grid = wn.Grid((-0.5,) * 3, (0.5,) * 3, (32, 32, 32))
    assert not torch.equal(wn.wn_voxelize(Vt, Ft, grid=grid), all_pairs(Vt, Ft, grid))  # (the path was taken)
    torch.cuda.synchronize()
    t = time.perf_counter()
    wn.wn_voxelize(Vt, Ft, grid=grid)
    torch.cuda.synchronize()
    t = time.perf_counter() - t
    print(f"{1e3 * t:.2f} ms", flush=True)
    assert t < 0.1


def all_pairs(V, F, grid, strips=None, occupancy=0, tau=0.5, k=50.0):
    """The C entry point with the smallest workspace that it accepts, found by bisection: without room for the
    boundary path, so the all-pairs kernels alone."""
    import ctypes
    import torch
    import paper_2407_11272_amd as wn
    from paper_2407_11272_amd import _lib as L
    lib, p, grid = L.load(), ctypes.c_void_p, wn.Grid.of(grid)
    full = wn.wn_workspace_size(L.WN_OP_VOXELIZE, V.shape[0], F.shape[0], grid.size)
    ws = torch.empty(full, dtype=torch.uint8, device="cuda")
    W = torch.empty(tuple(grid.n), device="cuda")
    occ = torch.empty(tuple(grid.n), dtype=torch.float32 if occupancy == L.WN_OCC_SIGMOID else torch.uint8, device="cuda")
    R = () if strips is None else (p(strips.data_ptr()), strips.shape[0])

    def call(n):
        return (lib.wn_voxelize if strips is None else lib.wn_voxelize_strips)(
            p(V.data_ptr()), V.shape[0], p(F.data_ptr()), F.shape[0], *R, ctypes.byref(grid.to_c()), p(0), 0,
            p(W.data_ptr()), occupancy, tau, k, p(occ.data_ptr()) if occupancy else p(0), p(ws.data_ptr()), n,
            p(torch.cuda.current_stream().cuda_stream))
    lo, hi = 0, full
    while hi - lo > 256:    # (sizes are multiples of 256 bytes)
        mid = (lo + hi) // 512 * 256
        lo, hi = (lo, mid) if call(mid) == L.WN_OK else (mid, hi)
    assert call(hi) == L.WN_OK and call(hi - 256) == L.WN_ERR_WORKSPACE
    torch.cuda.synchronize()
    return (W, occ) if occupancy else W


def fan(n):
    a = 2 * np.pi * np.arange(n) / n
    V = np.concatenate([[[0, 0, 0.1]], np.stack([0.4 * np.cos(a), 0.4 * np.sin(a), 0.05 * np.sin(5 * a)], -1)])
    return V, np.stack([np.zeros(n, int), 1 + np.arange(n), 1 + (np.arange(n) + 1) % n], -1)


@pytest.mark.parametrize("mesh,n", [("fan", 40), ("fan", 128), ("ribbon", 32), ("ribbon", 64)])
def test_caps_that_cost_more_than_the_faces(dev, mesh, n):
    """As many boundary edges as faces, or half as many in one long loop: the caps would take more than the
    faces, below the line of the blocks and above, so the mesh goes direct (the all-pairs bits)."""
    import torch
    import paper_2407_11272_amd as wn
    V, F = fan(3000) if mesh == "fan" else ribbon(2500, 2)
    Vt, Ft = _dev(V, F)
    grid = wn.Grid((-0.5,) * 3, (0.5,) * 3, (n, n, n + 1))
    assert len(F) * grid.size >= 7.0e7
    R = torch.as_tensor(wn.wn_build_strips(np.ascontiguousarray(F), len(V))).cuda()
    assert torch.equal(wn.wn_voxelize(Vt, Ft, grid=grid), all_pairs(Vt, Ft, grid))
    assert torch.equal(wn.wn_voxelize_strips(Vt, Ft, R, grid=grid), all_pairs(Vt, Ft, grid, R))
