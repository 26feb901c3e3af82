"""The work that programs have this library do, as measurable cases.

Every case goes through the package's public entry points: the forward solve
(``function.forward``), the differentiable solve (``function.solve``), the
batched solve (``batch.BatchPlan``), the mesh layer (``mesh.mesh``), the
sampled Chamfer loss of the fitting loop (``optimize.SampleFunction``,
``optimize.ChamferFunction``) and the slab solve of large scenes
(``slab.forward``).

``listed()`` names the cases, ``draw(rng)`` gives one more of the same ranges,
``prepare`` makes what a program holds before the call (inputs on the GPU, and
the buffers or plan it keeps), ``run`` is one pass, ``work`` the bytes and
operations a pass cannot do without, and ``exact`` the same outputs in 64 bits
from plain torch.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2106_03452_amd import batch as B
from paper_2106_03452_amd import function as F
from paper_2106_03452_amd import mesh as M
from paper_2106_03452_amd import optimize as O
from paper_2106_03452_amd import slab as S

DEV = torch.device("cuda", 0)


# --------------------------------------------------------------------------
# cases
# --------------------------------------------------------------------------
def listed():
    return [
        # one small object solved on its own, in an interactive or serving loop:
        # a few thousand points on the coarsest grid, where launches set the time
        {"name": "forward_32_3k", "path": "forward", "res": 32, "points": 3000, "sigma": 2.0, "cloud": "sphere"},
        # the first two levels of the fitting schedule: 20,000 points on coarse
        # grids (many points per cell), solved and differentiated a thousand times each
        {"name": "grad_32_20k", "path": "grad", "res": 32, "points": 20000, "sigma": 2.0, "cloud": "torus"},
        {"name": "grad_64_20k", "path": "grad", "res": 64, "points": 20000, "sigma": 2.0, "cloud": "torus"},
        # fitting and training at 128^3, the size of the learned pipeline
        {"name": "grad_128_20k", "path": "grad", "res": 128, "points": 20000, "sigma": 2.0, "cloud": "torus"},
        # ground-truth grids for training data: forward only, 100,000 points
        {"name": "forward_256_100k", "path": "forward", "res": 256, "points": 100000, "sigma": 2.0,
         "cloud": "superellipsoid"},
        # the same cloud with its gradient: the finest grid of fitting, and the benchmark's step
        {"name": "grad_256_100k", "path": "grad", "res": 256, "points": 100000, "sigma": 2.0,
         "cloud": "superellipsoid"},
        # a scan with outliers all over the volume: no plane or tile of the grid is empty
        {"name": "grad_256_outliers", "path": "grad", "res": 256, "points": 100000, "sigma": 2.0,
         "cloud": "outliers"},
        # the largest single grid
        {"name": "grad_512_100k", "path": "grad", "res": 512, "points": 100000, "sigma": 2.0,
         "cloud": "superellipsoid"},
        # a training or serving batch of mixed objects, forward and backward in one call
        {"name": "batch_20", "path": "batch", "jobs": 20, "lo": 64, "hi": 128, "points_lo": 1000, "points_hi": 50000,
         "sigma": 2.0, "mix": 3},
        # meshing a finished 256^3 grid and the loss gradient back to it
        {"name": "mesh_256", "path": "mesh", "res": 256, "blobs": 3, "mix": 5},
        # the loss of one fitting iteration: samples of the mesh against a scanned target, with its gradient
        {"name": "fit_20k", "path": "fit", "samples": 20000, "target": 20000, "nu": 160, "nv": 64},
        # a scene of many objects on the largest grid, forward
        {"name": "scene_1024_1m", "path": "scene", "res": 1024, "points": 1000000, "sigma": 2.0, "slabs": 8,
         "objects": 16},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above; odd point counts throughout."""
    path = rng.choice(["forward", "forward", "grad", "grad", "grad", "batch", "mesh", "fit", "scene"])
    if path in ("forward", "grad"):
        res = rng.choice([16, 32, 64, 128, 256, 512])
        return {"path": path, "res": res, "points": _log_int(rng, 1000, 200000), "sigma": rng.choice([2.0, 3.0]),
                "cloud": rng.choice(["sphere", "torus", "superellipsoid", "outliers"])}
    if path == "batch":
        lo, hi = rng.choice([(64, 128), (64, 256), (32, 128)])
        return {"path": path, "jobs": rng.randint(2, 20), "lo": lo, "hi": hi, "points_lo": 1000, "points_hi": 50000,
                "sigma": rng.choice([2.0, 3.0]), "mix": rng.randrange(1000)}
    if path == "mesh":
        return {"path": path, "res": rng.choice([32, 64, 128, 256]), "blobs": rng.randint(1, 6),
                "mix": rng.randrange(1000)}
    if path == "fit":
        return {"path": path, "samples": _log_int(rng, 3000, 60000), "target": _log_int(rng, 3000, 60000),
                "nu": rng.randint(40, 400), "nv": rng.randint(20, 160)}
    res = rng.choice([256, 512])
    return {"path": path, "res": res, "points": _log_int(rng, 100000, 1000000), "sigma": 2.0,
            "slabs": rng.choice([2, 4, 8, 16]), "objects": rng.randint(4, 16)}


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _rand(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV, dtype=torch.float64)


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV, dtype=torch.float64)


def _unit(v):
    return v / v.norm(dim=-1, keepdim=True).clamp_min(1e-300)


def _sphere(g, n, radius):
    d = _unit(_randn(g, n, 3))
    return radius * d, d


def _torus(g, n, big, small):
    """n points by area: the tube angle is drawn from its tabulated distribution."""
    v = torch.linspace(0, 2 * math.pi, 4097, device=DEV, dtype=torch.float64)
    cdf = (big * v + small * torch.sin(v)) / (2 * math.pi * big)
    x = _rand(g, n)
    i = torch.searchsorted(cdf, x).clamp(1, 4096)
    tv = v[i - 1] + (x - cdf[i - 1]) / (cdf[i] - cdf[i - 1]) * (v[i] - v[i - 1])
    u = 2 * math.pi * _rand(g, n)
    nrm = torch.stack([tv.cos() * u.cos(), tv.cos() * u.sin(), tv.sin()], 1)
    ring = torch.stack([u.cos(), u.sin(), torch.zeros_like(u)], 1)
    return big * ring + small * nrm, nrm


def _superellipsoid(g, n, axes, e1, e2):
    """n points by area (cells of an angle grid drawn in proportion to their area) and the implicit normals."""
    def power(x, e):
        return torch.sign(x) * x.abs() ** e

    def position(et, om):
        return torch.stack([axes[0] * power(et.cos(), e1) * power(om.cos(), e2),
                            axes[1] * power(et.cos(), e1) * power(om.sin(), e2),
                            axes[2] * power(et.sin(), e1)], -1)

    ne, nw = 512, 1024
    et = torch.linspace(-math.pi / 2, math.pi / 2, ne + 1, device=DEV, dtype=torch.float64)
    om = torch.linspace(-math.pi, math.pi, nw + 1, device=DEV, dtype=torch.float64)
    x = position(*torch.meshgrid(et, om, indexing="ij"))
    a, b = x[1:, :-1] - x[:-1, :-1], x[:-1, 1:] - x[:-1, :-1]
    area = torch.linalg.cross(a, b).norm(dim=-1).reshape(-1).cumsum(0)
    cell = torch.searchsorted(area, _rand(g, n) * area[-1]).clamp_max(ne * nw - 1)
    u = et[cell // nw] + _rand(g, n) * (et[1] - et[0])
    w = om[cell % nw] + _rand(g, n) * (om[1] - om[0])
    p = position(u, w)
    q = (p / torch.tensor(axes, device=DEV, dtype=torch.float64)).abs().clamp_min(1e-12)
    s = q[:, 0] ** (2 / e2) + q[:, 1] ** (2 / e2)
    pre = s ** (e2 / e1 - 1.0)
    d = torch.stack([pre * q[:, 0] ** (2 / e2 - 1.0) / axes[0], pre * q[:, 1] ** (2 / e2 - 1.0) / axes[1],
                     q[:, 2] ** (2 / e1 - 1.0) / axes[2]], 1) * torch.sign(p)
    return p, _unit(torch.nan_to_num(d, nan=0.0, posinf=0.0, neginf=0.0) + 1e-6 * p)


def _cloud(g, rnd, kind, n, res):
    """n oriented points in the unit box, float32: a scan of one object, its
    positions jittered by a tenth of a cell and its normals by a few degrees."""
    if kind == "sphere":
        p, d = _sphere(g, n, rnd.uniform(0.2, 0.35))
    elif kind == "torus":
        p, d = _torus(g, n, rnd.uniform(0.2, 0.28), rnd.uniform(0.06, 0.1))
    else:
        p, d = _superellipsoid(g, n, [rnd.uniform(0.15, 0.35) for _ in range(3)], rnd.uniform(0.3, 1.5),
                               rnd.uniform(0.3, 1.5))
    p = 0.5 + p + _randn(g, n, 3) * (0.1 / res)
    d = _unit(d + 0.05 * _randn(g, n, 3))
    if kind == "outliers":  # half of the points anywhere in the volume, with small normals
        out = _rand(g, n) < 0.5
        p = torch.where(out[:, None], _rand(g, n, 3), p)
        d = torch.where(out[:, None], _unit(_randn(g, n, 3)) * (0.05 * _rand(g, n, 1)), d)
    return p.float().contiguous(), d.float().contiguous()


def _residual(g, res):
    """The gradient of a mean squared error on the grid: a noisy and a smooth part, 2 / res^3 times the residual."""
    x = torch.arange(res, device=DEV, dtype=torch.float32) * (2 * math.pi / res)
    smooth = torch.sin(x)[:, None, None] * torch.cos(2 * x)[None, :, None] + torch.cos(x)[None, None, :]
    noise = torch.randn((res, res, res), generator=g, device=DEV)
    return ((0.05 * noise + 0.02 * smooth) * (2.0 / res ** 3)).contiguous()


def _scene(g, rnd, n, objects, res):
    """Objects of many sizes all over the box, points shared in proportion to area."""
    size = [rnd.uniform(0.04, 0.12) for _ in range(objects)]
    total = sum(s * s for s in size)
    count = [int(n * s * s / total) for s in size]
    count[0] += n - sum(count)
    ps, ds = [], []
    for s, k in zip(size, count):
        kind = rnd.choice(["sphere", "torus", "superellipsoid"])
        if kind == "sphere":
            p, d = _sphere(g, k, s)
        elif kind == "torus":
            p, d = _torus(g, k, s, s * rnd.uniform(0.25, 0.45))
        else:
            p, d = _superellipsoid(g, k, [s * rnd.uniform(0.5, 1.0) for _ in range(3)], rnd.uniform(0.3, 1.5),
                                   rnd.uniform(0.3, 1.5))
        centre = torch.tensor([rnd.uniform(0.14, 0.86) for _ in range(3)], device=DEV, dtype=torch.float64)
        ps.append(p + centre)
        ds.append(d)
    order = torch.randperm(n, generator=g, device=DEV)
    p = torch.cat(ps)[order] + _randn(g, n, 3) * (0.25 / res)
    return p.float().contiguous(), torch.cat(ds)[order].float().contiguous()


def _field(g, rnd, res, blobs, mix):
    """An indicator-like grid: -0.5 inside a union of soft balls, 0.5 outside,
    with a little roughness. The balls and the roughness belong to the case;
    the seed moves them by whole cells and scales the values by a smooth
    positive factor, so that every seed's mesh has the same size."""
    own, gm = random.Random(mix), _gen(mix)
    x = torch.arange(res, device=DEV, dtype=torch.float32) / res
    d = torch.full((res, res, res), 1.0, device=DEV)
    for _ in range(blobs):
        c = [own.uniform(0.36, 0.64) for _ in range(3)]
        r = own.uniform(0.08, 0.22)
        q = (x[:, None, None] - c[0]) ** 2 + (x[None, :, None] - c[1]) ** 2 + (x[None, None, :] - c[2]) ** 2
        d = torch.minimum(d, q.sqrt() - r)
    d = d * (res / 4.0)
    rough = 0.01 * torch.randn((res, res, res), generator=gm, device=DEV)
    chi = 0.5 * torch.tanh(d) + rough * torch.exp(-d * d)
    chi = torch.roll(chi, [rnd.randint(-(res // 12), res // 12) for _ in range(3)], (0, 1, 2))
    wave = 1.0 + 0.2 * torch.sin(2 * math.pi * (x * rnd.randint(1, 3) + rnd.random()))
    noise = 1.0 + 0.1 * torch.rand((res, res, res), generator=g, device=DEV)
    return (chi * wave[:, None, None] * noise).contiguous()


def _mesh(rnd, nu, nv):
    """A torus as nu x nv quads split in triangles: vertices float32, faces int32."""
    u = torch.arange(nu, device=DEV, dtype=torch.float64) * (2 * math.pi / nu)
    v = torch.arange(nv, device=DEV, dtype=torch.float64) * (2 * math.pi / nv)
    big, small = rnd.uniform(0.2, 0.28), rnd.uniform(0.06, 0.1)
    ring = big + small * torch.cos(v)[None, :]
    verts = 0.5 + torch.stack([ring * torch.cos(u)[:, None], ring * torch.sin(u)[:, None],
                               (small * torch.sin(v))[None, :].expand(nu, nv)], -1).reshape(-1, 3)
    i, j = torch.meshgrid(torch.arange(nu, device=DEV), torch.arange(nv, device=DEV), indexing="ij")
    a, b = i * nv + j, ((i + 1) % nu) * nv + j
    c, d = ((i + 1) % nu) * nv + (j + 1) % nv, i * nv + (j + 1) % nv
    faces = torch.stack([torch.stack([a, b, c], -1), torch.stack([a, c, d], -1)], 2).reshape(-1, 3)
    return verts.float().contiguous(), faces.to(torch.int32).contiguous()


def _jobs(case):
    """(resolution, points, cloud) of every job of a batch: part of the case, not of the seed."""
    rnd = random.Random(case["mix"])
    sizes = [r for r in (32, 64, 128, 256) if case["lo"] <= r <= case["hi"]]
    return [(rnd.choice(sizes), _log_int(rnd, case["points_lo"], case["points_hi"]),
             rnd.choice(["sphere", "torus", "superellipsoid"])) for _ in range(case["jobs"])]


def _inputs(case, seed):
    g, rnd, path = _gen(seed), random.Random(seed), case["path"]
    if path in ("forward", "grad"):
        p, n = _cloud(g, rnd, case["cloud"], case["points"], case["res"])
        return (p, n, _residual(g, case["res"]) if path == "grad" else None)
    if path == "batch":
        got = []
        for res, points, kind in _jobs(case):
            p, n = _cloud(g, rnd, kind, points, res)
            got.append((p, n, _residual(g, res), res))
        return got
    if path == "mesh":
        return _field(g, rnd, case["res"], case["blobs"], case["mix"])
    if path == "fit":
        verts, faces = _mesh(rnd, case["nu"], case["nv"])
        target = (0.5 + _torus(g, case["target"], rnd.uniform(0.2, 0.28), rnd.uniform(0.06, 0.1))[0]).float()
        u = torch.rand((case["samples"], 3), generator=g, device=DEV)
        return verts, faces, u, target.contiguous()
    return _scene(g, rnd, case["points"], case["objects"], case["res"])


def prepare(case, seed):
    got, path = _inputs(case, seed), case["path"]
    st = {"path": path, "case": dict(case)}
    if path == "forward":
        # a program that solves in a loop keeps its workspace
        p, n, _ = got
        st |= {"p": p, "n": n, "ws": torch.empty(F._lib.workspace_bytes(case["res"], case["points"]),
                                                 dtype=torch.uint8, device=DEV)}
    elif path == "grad":
        p, n, gr = got
        st |= {"p": p.requires_grad_(True), "n": n.requires_grad_(True), "g": gr}
    elif path == "batch":
        st["plan"] = B.BatchPlan([B.Job(p, n, res, case["sigma"], gr) for p, n, gr, res in got])
    elif path == "mesh":
        st["chi"] = got.requires_grad_(True)
    elif path == "fit":
        v, f, u, t = got
        st |= {"v": v.requires_grad_(True), "f": f, "u": u, "t": t}
    else:
        p, n = got
        st |= {"p": p, "n": n, "ws": torch.empty(S.workspace_bytes(case["res"], case["points"], case["slabs"]),
                                                 dtype=torch.uint8, device=DEV)}
    return st


def run(state):
    case, path = state["case"], state["path"]
    if path == "forward":
        return F.forward(state["p"], state["n"], case["res"], case["sigma"], workspace=state["ws"])[0]
    if path == "grad":
        chi = F.solve(state["p"], state["n"], case["res"], case["sigma"])
        dp, dn = torch.autograd.grad(chi, (state["p"], state["n"]), state["g"])
        return chi.detach(), dp, dn
    if path == "batch":
        state["plan"].run()
        return state["plan"].results()
    if path == "mesh":
        verts, faces, normals = M.mesh(state["chi"])
        # a loss that pulls the surface to the centre of the box
        dchi, = torch.autograd.grad(verts, state["chi"], verts.detach() - 0.5)
        return verts.detach(), faces, normals, dchi
    if path == "fit":
        x = O.SampleFunction.apply(state["v"], state["f"], state["u"])
        loss = O.ChamferFunction.apply(x, state["t"])
        dv, = torch.autograd.grad(loss, state["v"])
        return x.detach(), loss.detach(), dv
    return S.forward(state["p"], state["n"], case["res"], case["sigma"], case["slabs"], workspace=state["ws"])[0]


# --------------------------------------------------------------------------
# work
# --------------------------------------------------------------------------
def _solve_work(res, points, grad):
    """Points and normals in, the grid out (and the gradients); three transforms in and one back, each way."""
    n = float(res) ** 3
    by, fl = 24.0 * points + 4.0 * n, 4 * 2.5 * n * math.log2(n)
    if grad:
        by, fl = by + 4.0 * n + 24.0 * points, 2 * fl
    return by, fl


def work(case):
    path = case["path"]
    if path in ("forward", "grad", "scene"):
        by, fl = _solve_work(case["res"], case["points"], path == "grad")
    elif path == "batch":
        by, fl = (sum(x) for x in zip(*(_solve_work(r, p, True) for r, p, _ in _jobs(case))))
    elif path == "mesh":
        # the grid in and its gradient out; a vertex has its position and normal, two triangles and a gradient
        nv = 1.2 * case["blobs"] ** 0.5 * case["res"] ** 2 * 0.4
        by, fl = 8.0 * case["res"] ** 3 + nv * (24 + 24 + 12), 30.0 * nv
    else:
        nv, nf = case["nu"] * case["nv"], 2 * case["nu"] * case["nv"]
        q = case["samples"] + case["target"]
        # mesh, random numbers and target in, samples and gradient out; a query meets a few dozen neighbours
        by, fl = 24.0 * nv + 12.0 * nf + 24.0 * case["samples"] + 12.0 * case["target"], q * 64 * 8.0
    return {"bytes": by, "flops": fl}


# --------------------------------------------------------------------------
# the same in 64 bits
# --------------------------------------------------------------------------
def _corners(p, res):
    """For each of the 8 cell corners of every point: flat vertex index and weight (trilinear, periodic)."""
    t = (p - torch.floor(p)) * res
    b = torch.floor(t.detach()).clamp(0, res - 1)
    f, b = t - b, b.long()
    for o in range(8):
        idx, w = 0, 1.0
        for a in range(3):
            bit = (o >> a) & 1
            idx = idx * res + (b[:, a] + bit) % res
            w = w * (f[:, a] if bit else 1.0 - f[:, a])
        yield idx, w


def _exact_solve(p, n, res, sigma, dchi=None, m=0.5):
    p, n = p.detach().double(), n.detach().double()
    if dchi is not None:
        p.requires_grad_(True)
        n.requires_grad_(True)
    k = torch.fft.fftfreq(res, 1.0 / res, device=DEV, dtype=torch.float64)
    odd = k.clone()
    odd[res // 2] = 0.0
    kh, oh = k[: res // 2 + 1].abs(), odd[: res // 2 + 1].abs()
    corners = list(_corners(p, res))
    acc = None
    for a in range(3):
        v = torch.zeros(res ** 3, device=DEV, dtype=torch.float64)
        for idx, w in corners:
            v = v.index_add(0, idx, w * n[:, a]) if dchi is not None else v.index_add_(0, idx, w * n[:, a])
        spec = torch.fft.rfftn(v.view(res, res, res))
        del v
        fac = (odd[:, None, None], odd[None, :, None], oh[None, None, :])[a]
        acc = spec * fac if acc is None else acc + spec * fac
        del spec
    q = k[:, None, None] ** 2 + k[None, :, None] ** 2 + kh[None, None, :] ** 2
    filt = torch.exp(q * (-2.0 * sigma ** 2 / res ** 2)) / (-2.0 * math.pi * q)
    filt[0, 0, 0] = 0.0
    del q
    chi = torch.fft.irfftn(acc * filt * 1j, s=(res, res, res))
    del acc, filt
    flat = chi.reshape(-1)
    mu = sum((w * flat[idx]).sum() for idx, w in corners) / p.shape[0]
    chi = (chi - mu) * (m / (chi[0, 0, 0] - mu).abs())
    if dchi is None:
        return chi
    dp, dn = torch.autograd.grad(chi, (p, n), dchi.double())
    return chi.detach(), dp, dn


def _exact_mesh(chi):
    """Vertices and normals on the crossing edges in global edge order, and the gradient spread on the edge ends."""
    c = chi.detach().double()
    r = c.shape[0]
    h = 0.5 * r
    grad = torch.stack([(torch.roll(c, -1, a) - torch.roll(c, 1, a)) * h for a in range(3)], -1)
    inside = chi.detach() < 0
    cross = torch.zeros((r, r, r, 3), dtype=torch.bool, device=DEV)
    cross[:-1, :, :, 0] = inside[:-1] != inside[1:]
    cross[:, :-1, :, 1] = inside[:, :-1] != inside[:, 1:]
    cross[:, :, :-1, 2] = inside[:, :, :-1] != inside[:, :, 1:]
    i, j, k, a = cross.nonzero(as_tuple=True)
    lo = torch.stack([i, j, k], 1)
    step = torch.nn.functional.one_hot(a, 3)
    hi = lo + step
    c0, c1 = c[i, j, k], c[hi[:, 0], hi[:, 1], hi[:, 2]]
    t = (c0 / (c0 - c1))[:, None]
    verts = (lo + t * step) / r
    normals = _unit((1 - t) * grad[i, j, k] + t * grad[hi[:, 0], hi[:, 1], hi[:, 2]])
    g = -((verts - 0.5) * normals).sum(1)
    dchi = torch.zeros(r ** 3, device=DEV, dtype=torch.float64)
    flat = (lo[:, 0] * r + lo[:, 1]) * r + lo[:, 2]
    dchi.index_add_(0, flat, (1 - t[:, 0]) * g)
    dchi.index_add_(0, (hi[:, 0] * r + hi[:, 1]) * r + hi[:, 2], t[:, 0] * g)
    return verts, None, normals, dchi.view(r, r, r)


def _exact_fit(verts, faces, u, target):
    v, f, u, y = verts.detach().double().requires_grad_(True), faces.long(), u.double(), target.double()
    with torch.no_grad():
        area = 0.5 * torch.linalg.cross(v[f[:, 1]] - v[f[:, 0]], v[f[:, 2]] - v[f[:, 0]]).norm(dim=1)
        csum = area.cumsum(0)
        face = torch.searchsorted(csum, u[:, 0] * csum[-1], right=True).clamp_max(f.shape[0] - 1)
    s = u[:, 1].sqrt()
    bary = torch.stack([1 - s, s * (1 - u[:, 2]), s * u[:, 2]], 1)
    x = (bary[:, :, None] * v[f[face]]).sum(1)
    with torch.no_grad():
        nx = torch.cat([((q[:, None] - y[None]) ** 2).sum(-1).argmin(1) for q in x.split(2048)])
        ny = torch.cat([((q[:, None] - x[None]) ** 2).sum(-1).argmin(1) for q in y.split(2048)])
    loss = ((x - y[nx]) ** 2).sum(1).mean() + ((y - x[ny]) ** 2).sum(1).mean()
    dv, = torch.autograd.grad(loss, v)
    return x.detach(), loss.detach(), dv


def exact(case, seed):
    got, path = _inputs(case, seed), case["path"]
    if path == "forward":
        return _exact_solve(got[0], got[1], case["res"], case["sigma"])
    if path == "grad":
        return _exact_solve(got[0], got[1], case["res"], case["sigma"], got[2])
    if path == "batch":
        return [_exact_solve(p, n, res, case["sigma"], gr) for p, n, gr, res in got]
    if path == "mesh":
        return _exact_mesh(got)
    if path == "fit":
        return _exact_fit(*got)
    return _exact_solve(got[0], got[1], case["res"], case["sigma"])
