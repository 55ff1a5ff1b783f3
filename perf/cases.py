"""The work that users of this framework have it do, as cases with sizes.

Every path goes through a public entry point: the forward on a voxel grid (device faces, or
a triangle-strip order kept with the mesh), at a list of points, and for a batch of meshes;
the adjoint for dL/dV and for dL/dT; the fitting step (soft occupancy, loss, backward); the
Eq. 4 flux sum with its backward; and the evaluation chain.  Meshes are those of this
repository's workloads: jittered icospheres and unions of ellipsoids with a share of their
faces deleted (scans and hand-made meshes are seldom watertight), seeded per case.
"""
import math

import numpy as np
import torch

import paper_2407_11272_amd as wn
import wn_inputs as wi

DEV = "cuda"
K = 50.0      # sigmoid steepness of the differentiable workloads
TAU = 0.5


def listed():
    return [
        # the smallest call: a coarse preview of one small closed mesh, launch-bound
        dict(name="preview", path="grid", mesh="sphere", sub=2, faces=320, holes=0.0, n0=16, n1=16, n2=16,
             occ="threshold", strips=False),
        # the smallest workload of the repository: 1280 faces at 32^3
        dict(name="icosphere-32", path="grid", mesh="sphere", sub=3, faces=1280, holes=0.0, n0=32, n1=32, n2=32,
             occ="threshold", strips=False),
        # the forward of a fitting loop on a closed mesh: sigmoid occupancy, strips built once
        dict(name="soft-64", path="grid", mesh="sphere", sub=4, faces=5120, holes=0.0, n0=64, n1=64, n2=64,
             occ="sigmoid", strips=True),
        # the non-watertight union at 128^3, the ordinary large call
        dict(name="union-128", path="grid", mesh="union", sub=8, faces=20000, holes=0.05, n0=128, n1=128, n2=128,
             occ="threshold", strips=True),
        # the largest: 50 000 faces on an odd, non-cubic grid, W alone, faces as they come
        dict(name="union-odd", path="grid", mesh="union", sub=5, faces=50000, holes=0.08, n0=141, n1=117, n2=131,
             occ="none", strips=False),
        # W at scattered points (inside tests for samples or particles), a ragged count
        dict(name="points", path="points", mesh="union", sub=6, faces=10000, holes=0.05, n0=100003, n1=1, n2=1,
             occ="none", strips=True),
        # many meshes of uneven size in one launch
        dict(name="batch-16", path="batch", mesh="union", sub=16, faces=50000, holes=0.10, n0=128, n1=64, n2=32,
             occ="threshold", strips=True),
        # one fitting step on an open mesh: soft occupancy, MSE, backward to the vertices
        dict(name="fit-step", path="fit", mesh="sphere", sub=4, faces=5120, holes=0.05, n0=64, n1=64, n2=64,
             occ="sigmoid", strips=True),
        # the adjoint alone at a higher resolution (dL/dV only, faces in pairs)
        dict(name="adjoint-96", path="adjoint", mesh="union", sub=3, faces=8000, holes=0.05, n0=96, n1=88, n2=97,
             occ="none", strips=True),
        # the adjoint per face corner (dL/dT as well), one face per lane
        dict(name="corners-48", path="corners", mesh="sphere", sub=4, faces=5120, holes=0.0, n0=48, n1=48, n2=48,
             occ="none", strips=False),
        # the two halves of a morphing step by the Eq. 4 flux sum: the field, and the vertex
        # gradient for a given dL/dW
        dict(name="flux-step", path="flux", mesh="sphere", sub=4, faces=5120, holes=0.0, n0=64, n1=64, n2=64,
             occ="none", strips=False),
        # the evaluation chain on a 128^3 occupancy: cube surface, smoothing, samples, metrics
        dict(name="evaluate-128", path="evaluate", mesh="union", sub=8, faces=20000, holes=0.0, n0=128, n1=128,
             n2=128, occ="threshold", strips=False),
    ]


def draw(rng):
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    path = rng.choice(["grid", "grid", "grid", "points", "batch", "fit", "adjoint", "corners", "flux", "evaluate"])
    # a closed surface has no vertex gradient, so the fitting paths are given open meshes
    holes = rng.uniform(0.02, 0.10) if path in ("fit", "adjoint") else rng.choice([0.0, rng.uniform(0.0, 0.10)])
    c = dict(path=path, mesh="union", sub=rng.randint(1, 8), faces=log(500, 50000), holes=holes,
             n0=log(16, 128), n1=log(16, 128), n2=log(16, 128), occ=rng.choice(["none", "threshold", "sigmoid"]),
             strips=rng.random() < 0.5)
    if path == "points":
        c.update(n0=log(100, 300000), n1=1, n2=1, occ="none")
    elif path == "batch":
        c.update(sub=rng.randint(2, 12), faces=log(1000, 50000))
    elif path in ("fit", "adjoint", "corners"):
        c.update(faces=log(500, 10000), n0=log(16, 80), n1=log(16, 80), n2=log(16, 80))
    elif path == "flux":
        c.update(faces=log(500, 20000), n0=log(16, 96), n1=log(16, 96), n2=log(16, 96), occ="none")
    elif path == "evaluate":
        c.update(n0=log(24, 128), n1=log(24, 128), n2=log(24, 128), occ="threshold", holes=0.0)
    return c


# ------------------------------------------------------------------ inputs

def _grid(c):
    return wn.Grid((-0.5, -0.5, -0.5), (0.5, 0.5, 0.5), (c["n0"], c["n1"], c["n2"]))


def _points(c):
    return c["n0"] * c["n1"] * c["n2"]


def _mesh(c, rng):
    """Host mesh: float32 vertices, int32 faces."""
    if c["mesh"] == "sphere":
        V, F = wi.icosphere(c["sub"])
        V = wi.jitter(V * 0.4, 0.01, rng)
    else:
        V, F, _ = wi.ellipsoid_union(rng, c["sub"], max(8, c["faces"] // c["sub"]))
    F = wi.delete_faces(F, round(c["holes"] * len(F)), rng)
    return np.asarray(V, np.float32), np.asarray(F, np.int32)


def _dev(V, F):
    return torch.as_tensor(V, device=DEV), torch.as_tensor(F, device=DEV)


def _strips(V, F):
    return torch.as_tensor(wn.wn_build_strips(F, len(V)), device=DEV)


def _pairs(V, F):
    return torch.as_tensor(wn.wn_build_face_pairs(F, len(V)), device=DEV)


def _target(c, rng):
    e = wi.random_ellipsoid(rng, 0.25, 0.4, -0.05, 0.05)
    g = wi.Grid((-0.5, -0.5, -0.5), (0.5, 0.5, 0.5), (c["n0"], c["n1"], c["n2"]))
    return torch.as_tensor(wi.ellipsoid_target_on_grid(g, e), device=DEV).reshape(c["n0"], c["n1"], c["n2"])


def _batch(c, rng):
    """(host mesh, grid side) of each mesh of a batch: sizes spread as in a served mix (they
    belong to the case), shapes and holes from ``rng``."""
    size = np.random.default_rng([c["sub"], c["faces"], c["n0"], c["n1"], c["n2"]])
    out = []
    for _ in range(c["sub"]):
        faces = int(round(math.exp(size.uniform(math.log(500), math.log(c["faces"])))))
        m = dict(mesh="union", sub=int(size.integers(1, 9)), faces=faces, holes=float(size.uniform(0.0, c["holes"])))
        n = int(size.choice([c["n0"], c["n1"], c["n2"]]))
        V, F = _mesh(m, rng)
        out.append((V, F, n))
    return out


def _inputs(case, seed):
    """Everything random of a case, from its sizes and the seed alone."""
    c, rng = dict(case), np.random.default_rng([seed, 2407])
    s = dict(c=c, rng=rng)
    if c["path"] == "batch":
        s["batch"] = _batch(c, rng)
        return s
    s["V"], s["F"] = _mesh(c, rng)
    if c["path"] == "points":
        s["Q"] = torch.as_tensor(rng.uniform(-0.5, 0.5, (c["n0"], 3)).astype(np.float32), device=DEV)
    elif c["path"] in ("fit", "adjoint", "corners"):
        s["target"] = _target(c, rng)
        if c["path"] != "fit":  # the gradient that a sigmoid-MSE loss sends back to W
            V, F = _dev(s["V"], s["F"])
            W = _winding64(V.double(), F.long(), _centres64(c))
            sg = torch.sigmoid(K * (W - TAU))
            g = 2.0 / len(W) * (sg - s["target"].reshape(-1)) * K * sg * (1 - sg)
            if c["path"] == "corners":  # a closed mesh: weights of a general functional of W
                g = torch.as_tensor(rng.standard_normal(len(W)), device=DEV) / len(W)
            s["g"] = g.to(torch.float32)
    elif c["path"] == "flux":
        # dL/dW of a sigmoid-MSE loss is largest where the field crosses the threshold: a
        # band around the ellipsoid that the surface is drawn to
        t = _target(c, rng)
        pull = torch.as_tensor(rng.standard_normal(t.shape, np.float32), device=DEV)
        s["g"] = ((0.1 + t) * pull / t.numel()).reshape(-1).contiguous()
    elif c["path"] == "evaluate":
        # the occupied shape belongs to the case (the surface's size with it), seen from one
        # of its eight mirror sides
        g = wi.Grid((-0.5, -0.5, -0.5), (0.5, 0.5, 0.5), (c["n0"], c["n1"], c["n2"]))
        occ = np.zeros((c["n0"], c["n1"], c["n2"]), np.float32)
        shape = np.random.default_rng([c["sub"], c["faces"], c["n0"], c["n1"], c["n2"]])
        for _ in range(c["sub"]):
            e = wi.random_ellipsoid(shape, 0.05, 0.3, -0.3, 0.3)
            occ = np.maximum(occ, wi.ellipsoid_target_on_grid(g, e).reshape(occ.shape))
        occ = np.flip(occ, [d for d in range(3) if rng.random() < 0.5])
        s["occ"] = torch.as_tensor(np.ascontiguousarray(occ).astype(np.uint8), device=DEV).reshape(-1)
        s["u"] = [torch.as_tensor(rng.random((20000, 3)), device=DEV) for _ in range(2)]
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    c = s["c"]
    if c["path"] == "batch":
        s["jobs"] = []
        for V, F, n in s["batch"]:
            Vt, Ft = _dev(V, F)
            s["jobs"].append(wn.MeshJob(Vt, Ft, wn.Grid.cube(n), None if c["occ"] == "none" else c["occ"],
                                        strips=_strips(V, F) if c["strips"] else None).prepare())
        return s
    V, F = s["V"], s["F"]
    s["V"], s["F"] = _dev(V, F)
    s["grid"] = None if c["path"] == "points" else _grid(c)
    s["R"] = _strips(V, F) if c["strips"] else None
    s["pairs"] = _pairs(V, F) if c["path"] in ("fit", "adjoint") and c["strips"] else None
    return s


# ------------------------------------------------------------------ one pass

def run(s):
    c = s["c"]
    path = c["path"]
    if path == "batch":
        wn.wn_voxelize_batched(s["jobs"])
        return [j.W for j in s["jobs"]] + ([] if c["occ"] == "none" else [j.occ for j in s["jobs"]])
    V, F = s["V"], s["F"]
    if path in ("grid", "points"):
        kw = dict(grid=s["grid"], Q=s.get("Q"), occupancy=None if c["occ"] == "none" else c["occ"], tau=TAU, k=K)
        return wn.wn_voxelize(V, F, **kw) if s["R"] is None else wn.wn_voxelize_strips(V, F, s["R"], **kw)
    if path == "fit":
        x = V.detach().requires_grad_(True)
        occ = wn.soft_occupancy(x, F, grid=s["grid"], tau=TAU, k=K, strips=s["R"], pairs=s["pairs"])
        loss = ((occ - s["target"]) ** 2).mean()
        loss.backward()
        return occ.detach(), loss.detach(), x.grad
    if path == "adjoint":
        return wn.wn_backward(V, F, s["g"], grid=s["grid"], pairs=s["pairs"])
    if path == "corners":
        return wn.wn_backward(V, F, s["g"], grid=s["grid"], want_dLdT=True)[1]
    if path == "flux":
        return wn.wn_voxelize_naive(V, F, grid=s["grid"]), wn.wn_backward_naive(V, F, s["g"], grid=s["grid"])
    Vc, Fc = wn.wn_cubify(s["occ"], s["grid"])
    Vs = wn.wn_laplacian_smooth(Vc, Fc)
    Pa, fa = wn.wn_sample_surface(Vs, Fc, s["u"][0])
    Pb, fb = wn.wn_sample_surface(V, F, s["u"][1])
    return Vs, Fc, Pa, fa, Pb, fb, wn.wn_chamfer_hausdorff(Pa, Pb)


# ------------------------------------------------------------------ work

# Operations of one solid angle, of its gradient, and of one Eq. 4 term with its gradient.
SOLID, SOLID_GRAD, FLUX = 86, 182, 20 + 36


def work(case):
    """W is an integer plus the solid angles of the holes (closed surfaces have W constant
    on each side), and only the hole rims carry a vertex gradient; dL/dT and the flux sum
    need every face at every point."""
    c, P = case, _points(case)
    nf = 20 * 4 ** c["sub"] if c["mesh"] == "sphere" else c["faces"]
    mesh = 12 * nf + 6 * nf + (8 * 1.15 * nf if c["strips"] else 0)
    out = P * {"none": 4, "threshold": 5, "sigmoid": 8}[c["occ"]]
    missing = c["holes"] * nf
    if c["path"] == "batch":
        P = c["sub"] * (c["n0"] ** 3 + c["n1"] ** 3 + c["n2"] ** 3) / 3
        nf = (c["faces"] - 500) / math.log(c["faces"] / 500)
        out = P * {"none": 4, "threshold": 5, "sigmoid": 8}[c["occ"]]
        return dict(bytes=27 * nf * c["sub"] + out, flops=SOLID * P * nf * c["holes"] / 2)
    if c["path"] == "points":
        return dict(bytes=mesh + 16 * P, flops=SOLID * P * missing)
    if c["path"] == "fit":
        return dict(bytes=2 * mesh + 16 * P, flops=(SOLID + SOLID_GRAD) * P * missing)
    if c["path"] == "adjoint":
        return dict(bytes=mesh + 4 * P, flops=SOLID_GRAD * P * missing)
    if c["path"] == "corners":
        return dict(bytes=mesh + 4 * P + 36 * nf, flops=SOLID_GRAD * P * (1 - c["holes"]) * nf)
    if c["path"] == "flux":
        return dict(bytes=2 * mesh + 20 * P, flops=FLUX * P * (1 - c["holes"]) * nf)
    if c["path"] == "evaluate":
        surface = 12 * P ** (2 / 3)
        return dict(bytes=P + 400 * surface, flops=2 * 8 * 20000.0 ** 2)
    return dict(bytes=mesh + out, flops=SOLID * P * missing)


# ------------------------------------------------------------------ in 64 bits

def _centres64(c):
    """Voxel centres, rounded to the float32 positions that a grid stands for."""
    ax = []
    for d in range(3):
        n = c["n%d" % d]
        h = torch.tensor(np.float32(1.0 / n), device=DEV, dtype=torch.float64)
        ax.append(((torch.arange(n, device=DEV, dtype=torch.float64) + 0.5) * h - 0.5).float().double())
    return torch.stack(torch.meshgrid(*ax, indexing="ij"), -1).reshape(-1, 3)


def _chunks(P, nF, pairs=1 << 26):
    step = max(256, min(P, pairs // max(1, min(nF, 16384))))
    return range(0, P, step), step


def _winding64(V, F, Q):
    """Eq. 5 by the half-angle formula, R_j . R_k through matrix products."""
    W = torch.zeros(len(Q), dtype=torch.float64, device=DEV)
    steps, step = _chunks(len(Q), len(F))
    for f0 in range(0, len(F), 16384):
        T = V[F[f0:f0 + 16384]]
        a, b, d = T[:, 0], T[:, 1], T[:, 2]
        n = torch.linalg.cross(b - a, d - a)
        for q0 in steps:
            q = Q[q0:q0 + step]
            qq = (q * q).sum(1, keepdim=True)

            def dot(x, y):
                return torch.addmm((x * y).sum(1).expand(len(q), -1), q, -(x + y).T).add_(qq)

            ra, rb, rd = (dot(x, x).clamp_(min=0).sqrt_() for x in (a, b, d))
            be = dot(a, b).mul_(rd)
            be.addcmul_(dot(b, d), ra).addcmul_(dot(d, a), rb).addcmul_(ra.mul_(rb), rd)
            al = torch.addmm((n * a).sum(1).expand(len(q), -1), q, -n.T)
            W[q0:q0 + step] += torch.atan2(al, be).sum(1)
    return W / (2 * math.pi)


def _corner_grad64(V, F, Q, g):
    """sum_q g[q] dW(q)/dT for every face corner: the edge form of the solid angle's
    derivative, closed for a linear motion of the edge's ends."""
    T = V[F]
    out = torch.zeros(len(F), 3, 3, dtype=torch.float64, device=DEV)
    live = g.nonzero()[:, 0]
    Q, g = Q[live], g[live]
    steps, step = _chunks(len(Q), len(F), 1 << 24)
    for f0 in range(0, len(F), 16384):
        t = T[f0:f0 + 16384]
        for q0 in steps:
            q, w = Q[q0:q0 + step], g[q0:q0 + step, None]
            R = [[t[:, j, d] - q[:, d, None] for d in range(3)] for j in range(3)]
            r = [torch.sqrt(x[0] * x[0] + x[1] * x[1] + x[2] * x[2]) for x in R]
            for j in range(3):
                k = (j + 1) % 3
                A, B, a, b = R[j], R[k], r[j], r[k]
                cr = [A[1] * B[2] - A[2] * B[1], A[2] * B[0] - A[0] * B[2], A[0] * B[1] - A[1] * B[0]]
                dt = A[0] * B[0] + A[1] * B[1] + A[2] * B[2]
                # d Omega = -int (delta x t) . R / |R|^3 along the edge; 1/(ab(ab+A.B)) is its
                # closed form, shared out between the two ends
                base = w / (a * b * (a * b + dt))
                ca, cb = base * b, base * a
                for d in range(3):
                    out[f0:f0 + 16384, j, d] -= (ca * cr[d]).sum(0)
                    out[f0:f0 + 16384, k, d] -= (cb * cr[d]).sum(0)
    return out / (4 * math.pi)


def _gather64(T, F, nV):
    return torch.zeros(nV, 3, dtype=torch.float64, device=DEV).index_add_(0, F.reshape(-1), T.reshape(-1, 3))


def _occ64(c, W):
    """Threshold occupancies are whole numbers: compared as they are, no value here."""
    return torch.sigmoid(K * (W - TAU)) if c["occ"] == "sigmoid" else None


def exact(case, seed):
    c = dict(case)
    if c["path"] == "evaluate":
        return None
    s = _inputs(case, seed)
    if c["path"] == "batch":
        Ws = []
        for V, F, n in s["batch"]:
            Vt, Ft = _dev(V, F)
            Ws.append(_winding64(Vt.double(), Ft.long(), _centres64(dict(n0=n, n1=n, n2=n))).reshape(n, n, n))
        return Ws + ([] if c["occ"] == "none" else [_occ64(c, W) for W in Ws])
    V, F = _dev(s["V"], s["F"])
    V, F = V.double(), F.long()
    shape = (c["n0"], c["n1"], c["n2"])
    if c["path"] == "points":
        return _winding64(V, F, s["Q"].double())
    Q = _centres64(c)
    if c["path"] == "grid":
        W = _winding64(V, F, Q).reshape(shape)
        return W if c["occ"] == "none" else (W, _occ64(c, W))
    if c["path"] in ("adjoint", "corners"):
        T = _corner_grad64(V, F, Q, s["g"].double())
        return T if c["path"] == "corners" else _gather64(T, F, len(V))
    if c["path"] == "flux":
        return _flux64(V, F, Q, s["g"].double(), shape)
    target = s["target"].double().reshape(-1)
    W = _winding64(V, F, Q)
    sg = torch.sigmoid(K * (W - TAU))
    g = 2.0 / len(W) * (sg - target) * K * sg * (1 - sg)
    g = torch.where(g.abs() > 1e-14 * g.abs().max(), g, torch.zeros_like(g))
    return sg.reshape(shape), ((sg - target) ** 2).mean(), _gather64(_corner_grad64(V, F, Q, g), F, len(V))


def _flux64(V, F, Q, g, shape):
    """Eq. 4's sum and sum_q g[q] dW(q)/dV."""
    x = V.clone().requires_grad_(True)
    W = []
    steps, step = _chunks(len(Q), len(F), 1 << 25)
    for q0 in steps:
        q, t = Q[q0:q0 + step], x[F]
        n, m = torch.linalg.cross(t[:, 1] - t[:, 0], t[:, 2] - t[:, 0]), t.mean(1)
        r = [m[:, d] - q[:, d, None] for d in range(3)]
        r2 = r[0] * r[0] + r[1] * r[1] + r[2] * r[2]
        w = ((r[0] * n[:, 0] + r[1] * n[:, 1] + r[2] * n[:, 2]) * r2 ** -1.5).sum(1) / (8 * math.pi)
        w.backward(g[q0:q0 + step])
        W.append(w.detach())
    return torch.cat(W).reshape(shape), x.grad
