"""Performance cases of the framework: what a user's program calls, at the sizes it calls it.

Each case is one pass through the public entry points of ``paper_1809_00845_amd.binding``:

* ``apply``  -- one operator application r = c u + D[u] - S[q] (the matrix-vector product of every solve);
* ``grid``   -- the field over the grid box (the solution inside the body after a solve);
* ``gmres``  -- a mixed boundary-value problem solved from zero, FP32 with FP64 refinement;
* ``cg``     -- a Dirichlet problem solved by conjugate gradients in FP64;
* ``batch``  -- one application of many boundaries x right-hand sides;
* ``grad``   -- loss and gradients of one training problem of the learned-start network;
* ``guess``  -- the learned initial guess of one Dirichlet problem (FP16 inference).

Geometries are closed surfaces voxelised on a uniform grid, fixed by the case; the boundary data are
drawn from the seed.  ``exact`` evaluates the same discrete definitions in FP64 with plain torch.
"""

import functools
import math
import random

import numpy as np
import torch

from paper_1809_00845_amd import binding as B

KERNEL = {"l2d": B.LAPLACE2D, "l3d": B.LAPLACE3D, "nav": B.NAVIER3D, "hs": B.HALFSPACE}
PREC = {"fp64": B.FP64, "fp32": B.FP32, "bf16": B.BF16_MFMA}
SIZES = (32, 64, 96, 128, 192, 256, 320, 384, 512, 1024)  # padded transform lengths
NU, MU = 0.3, 1.0
DILATIONS = (1, 2, 4, 8)


def listed():
    return [
        # the smallest call: a 2D boundary of a few hundred nodes, FP64 (launches and latency)
        {"name": "apply_l2d_circle128_fp64", "op": "apply", "kernel": "l2d", "shape": "circle", "nx": 128, "ny": 128,
         "nz": 1, "precision": "fp64"},
        # the paper's own setting: the square with 500 points per side, solved by CG
        {"name": "cg_l2d_square500_fp64", "op": "cg", "kernel": "l2d", "shape": "square", "nx": 500, "ny": 500,
         "nz": 1, "precision": "fp64"},
        # contact mechanics: the displacement of a whole loaded half-space surface
        {"name": "apply_hs_surface256_fp32", "op": "apply", "kernel": "hs", "shape": "surface", "nx": 256, "ny": 256,
         "nz": 1, "precision": "fp32"},
        # the benchmark's configuration: cube surface, 100 points per edge in 128^3
        {"name": "apply_l3d_cube128_fp32", "op": "apply", "kernel": "l3d", "shape": "cube", "nx": 128, "ny": 128,
         "nz": 128, "precision": "fp32"},
        # the potential inside a body after a solve, FP64, a box with odd unequal sides
        {"name": "grid_l3d_blob119x87x101_fp64", "op": "grid", "kernel": "l3d", "shape": "blob", "nx": 119, "ny": 87,
         "nz": 101, "precision": "fp64"},
        # the 16-bit operator used for inner iterations
        {"name": "apply_l3d_blob128_bf16", "op": "apply", "kernel": "l3d", "shape": "blob", "nx": 128, "ny": 128,
         "nz": 128, "precision": "bf16"},
        # elastostatics at the benchmark's size: 192^3, FP32 (the longest single application)
        {"name": "apply_nav_blob192_fp32", "op": "apply", "kernel": "nav", "shape": "blob", "nx": 192, "ny": 192,
         "nz": 192, "precision": "fp32"},
        # elastostatics in FP64 at an ordinary, odd size
        {"name": "apply_nav_blob93_fp64", "op": "apply", "kernel": "nav", "shape": "blob", "nx": 93, "ny": 93,
         "nz": 93, "precision": "fp64"},
        # time to solve: mixed boundary data, FP32 iterations refined with FP64 residuals
        {"name": "gmres_l3d_blob96_fp32", "op": "gmres", "kernel": "l3d", "shape": "blob", "nx": 96, "ny": 96,
         "nz": 96, "precision": "fp32"},
        # many boundaries of mixed sizes with four load cases each, one batched application
        {"name": "batch_l3d_8x4_fp32", "op": "batch", "kernel": "l3d", "shapes": 8, "nmin": 64, "nmax": 160,
         "nrhs": 4, "shape_seed": 2, "precision": "fp32"},
        # training of the learned start at its full grid
        {"name": "grad_net96", "op": "grad", "shape": "blob", "nx": 96, "ny": 96, "nz": 96},
        # the learned start in use
        {"name": "guess_net96", "op": "guess", "kernel": "l3d", "shape": "blob", "nx": 96, "ny": 96, "nz": 96,
         "precision": "fp64"},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the same ranges."""
    op = rng.choice(["apply2d", "apply3d", "apply3d", "applynav", "applynav", "cg", "grid", "gmres", "batch", "grad",
                     "guess"])
    if op == "apply2d":
        kernel = rng.choice(["l2d", "hs"])
        n = _log_int(rng, 40, 512) if kernel == "l2d" else _log_int(rng, 40, 300)
        shape = rng.choice(["circle", "square"]) if kernel == "l2d" else rng.choice(["surface", "disc"])
        return {"op": "apply", "kernel": kernel, "shape": shape, "nx": n, "ny": n, "nz": 1,
                "precision": rng.choice(["fp64", "fp32"])}
    if op == "cg":
        n = _log_int(rng, 60, 500)
        return {"op": "cg", "kernel": "l2d", "shape": rng.choice(["circle", "square"]), "nx": n, "ny": n, "nz": 1,
                "precision": "fp64"}
    if op == "batch":
        lo = rng.randint(24, 64)
        return {"op": "batch", "kernel": "l3d", "shapes": rng.randint(2, 8), "nmin": lo, "nmax": lo + rng.randint(0, 64),
                "nrhs": rng.randint(1, 4), "shape_seed": rng.randint(0, 999), "precision": rng.choice(["fp32", "fp64"])}
    if op in ("grad", "guess"):
        n = rng.randint(32, 96)
        c = {"op": op, "shape": "blob", "nx": n, "ny": n, "nz": n}
        if op == "guess":
            c.update({"kernel": "l3d", "precision": "fp64"})
        return c
    if op == "applynav":
        prec = rng.choice(["fp32", "fp64", "bf16"])
        n = _log_int(rng, 24, 192 if prec != "fp64" else 128)
        shape = rng.choice(["blob", "blob", "cube"])
        kernel = "nav"
    else:
        prec = rng.choice(["fp32", "fp64", "bf16"]) if op == "apply3d" else rng.choice(["fp32", "fp64"])
        if op == "gmres":
            prec = "fp32"
        n = _log_int(rng, 24, {"apply3d": 192, "grid": 160, "gmres": 112}[op])
        shape = rng.choice(["blob", "blob", "cube"])
        kernel = "l3d"
    c = {"op": "apply" if op.startswith("apply") else op, "kernel": kernel, "shape": shape, "nx": n, "ny": n, "nz": n,
         "precision": prec}
    if shape == "blob" and rng.random() < 0.5:  # a box with unequal sides
        c["ny"] = max(20, int(n * rng.uniform(0.6, 1.0)))
        c["nz"] = max(20, int(n * rng.uniform(0.6, 1.0)))
    return c


# ------------------------------------------------------------------ geometry


class _Geom:
    def __init__(self, dim, n, nodes, normals, weights):
        self.dim, self.n = dim, n
        self.h = 1.0 / max(n)
        self.origin = (0.0, 0.0, 0.0)
        self.nodes, self.normals, self.weights = nodes, normals, weights
        self.m = int(weights.shape[0])
        self.index = np.rint(nodes / self.h).astype(np.int64)
        self.center = 0.5 * self.h * np.asarray(n[:dim], dtype=np.float64)


def _cells(n, pts, vec):
    """Surface pieces (midpoints, outward area vectors) summed per grid cell."""
    h = 1.0 / max(n)
    dim = pts.shape[1]
    g = np.floor(pts / h + 0.5).astype(np.int64)
    lin = g[:, dim - 1]
    for a in range(dim - 2, -1, -1):
        lin = lin * n[a] + g[:, a]
    cells, inv = np.unique(lin, return_inverse=True)
    size = np.linalg.norm(vec, axis=1)
    w = np.bincount(inv, weights=size, minlength=cells.size)
    nv = np.stack([np.bincount(inv, weights=vec[:, a], minlength=cells.size) / w for a in range(dim)], 1)
    idx = np.empty((cells.size, dim), dtype=np.int64)
    rest = cells
    for a in range(dim - 1):
        idx[:, a] = rest % n[a]
        rest = rest // n[a]
    idx[:, dim - 1] = rest
    return _Geom(dim, n, idx * h, nv, w)


@functools.lru_cache(maxsize=64)
def _geometry(shape, nx, ny, nz, shape_seed):
    n = (nx, ny, nz)
    h = 1.0 / max(n)
    if shape == "blob":
        # a smooth star-shaped body: an ellipsoid that follows the box, with bumps of degree 1 to 3
        rng = np.random.default_rng(1000 + shape_seed)
        amp = rng.uniform(-0.06, 0.06, 6)
        k = int(3.2 * max(n))
        th = np.linspace(0.0, math.pi, k + 1)[:, None]
        ph = np.linspace(0.0, 2.0 * math.pi, 2 * k + 1)[None, :]
        e = np.stack([np.sin(th) * np.cos(ph), np.sin(th) * np.sin(ph), np.cos(th) + 0.0 * ph], -1)
        ex, ey, ez = e[..., 0], e[..., 1], e[..., 2]
        r = 1.0 + amp[0] * ex + amp[1] * ez + amp[2] * ex * ey + amp[3] * ey * ez + amp[4] * ex * ey * ez + amp[5] * ez ** 3
        c = 0.5 * h * np.asarray(n)
        p = c + e * r[..., None] * (0.36 * h * np.asarray(n))
        a, b, cc, d = p[:-1, :-1], p[1:, :-1], p[1:, 1:], p[:-1, 1:]
        vec = 0.5 * np.cross(cc - a, d - b)
        mid = 0.25 * (a + b + cc + d)
        return _cells(n, mid.reshape(-1, 3), vec.reshape(-1, 3))
    if shape == "cube":
        # faces on grid planes, about 0.78 of the grid's points per edge
        e = int(round(0.78125 * nx))
        lo = (nx - e) // 2
        hi = lo + e - 1
        r = np.arange(lo, hi + 1)
        g = np.stack(np.meshgrid(r, r, r, indexing="ij"), -1).reshape(-1, 3)
        g = g[((g == lo) | (g == hi)).any(1)]
        nv = (g == hi).astype(float) - (g == lo).astype(float)
        cnt = np.abs(nv).sum(1)
        w = np.where(cnt == 3, 0.75, 1.0) * h * h
        return _Geom(3, n, g * h, nv / cnt[:, None], w)
    if shape == "circle":
        k = 40 * nx
        t = np.linspace(0.0, 2.0 * math.pi, k + 1)
        p = np.stack([0.5 + 0.4 * np.cos(t), 0.5 + 0.4 * np.sin(t)], 1) * (h * nx)
        d = p[1:] - p[:-1]
        return _cells(n, 0.5 * (p[1:] + p[:-1]), np.stack([d[:, 1], -d[:, 0]], 1))
    if shape == "square":
        # grid-aligned sides that use the whole grid (the paper's boundary)
        r = np.arange(nx)
        g = np.stack(np.meshgrid(r, r, indexing="ij"), -1).reshape(-1, 2)
        g = g[((g == 0) | (g == nx - 1)).any(1)]
        nv = (g == nx - 1).astype(float) - (g == 0).astype(float)
        return _Geom(2, n, g * h, nv / np.abs(nv).sum(1, keepdims=True), np.full(len(g), h))
    r = np.arange(nx)  # half-space surface: all of it, or a circular contact patch
    g = np.stack(np.meshgrid(r, r, indexing="ij"), -1).reshape(-1, 2)
    if shape == "disc":
        g = g[np.linalg.norm(g - 0.5 * (nx - 1), axis=1) <= 0.3 * nx]
    return _Geom(2, n, g * h, np.zeros((len(g), 2)), np.full(len(g), h * h))


def _geom(case):
    return _geometry(case["shape"], case["nx"], case["ny"], case["nz"], case.get("shape_seed", 0))


def _batch_geoms(case):
    r = random.Random(case["shape_seed"])
    out = []
    for i in range(case["shapes"]):
        n = r.randint(case["nmin"], case["nmax"])
        out.append(_geometry("blob", n, n, n, case["shape_seed"] + i))
    return out


# ------------------------------------------------------------------ data


def _smooth(g, rng):
    """A random smooth field at the nodes: harmonic polynomials of degree <= 3 (2D: <= 3 too)."""
    x = (g.nodes - g.center[None, :]) / 0.5
    c = rng.standard_normal(10)
    if g.dim == 2:
        z = x[:, 0] + 1j * x[:, 1]
        return sum(c[k] * (z ** k).real + c[k + 4] * (z ** k).imag for k in range(4))
    x, y, z = x.T
    return (c[0] + c[1] * x + c[2] * y + c[3] * z + c[4] * x * y + c[5] * y * z + c[6] * (x * x - y * y)
            + c[7] * x * y * z + c[8] * x * (x * x - 3 * y * y) + c[9] * z * (2 * z * z - 3 * x * x - 3 * y * y))


def _fields(g, kernel, rng):
    """(q, u) as a solve meets them: smooth data with a rough part, one value per node and component."""
    nc = 3 if kernel in ("nav", "hs") else 1
    q = np.concatenate([_smooth(g, rng) + 0.3 * rng.standard_normal(g.m) for _ in range(nc)])
    u = np.concatenate([_smooth(g, rng) + 0.05 * rng.standard_normal(g.m) for _ in range(nc)])
    return q, u


def _data(case, seed):
    """Everything the seed decides, as numpy arrays."""
    rng = np.random.default_rng(seed)
    op = case["op"]
    if op == "batch":
        qs, us = [], []
        for g in _batch_geoms(case):
            for _ in range(case["nrhs"]):
                q, u = _fields(g, case["kernel"], rng)
                qs.append(q)
                us.append(u)
        return {"q": np.concatenate(qs), "u": np.concatenate(us)}
    g = _geom(case)
    if op in ("apply", "grid"):
        q, u = _fields(g, case["kernel"], rng)
        return {"q": q, "u": u}
    if op == "cg":
        return {"u": _smooth(g, rng)}
    if op == "gmres":  # above the centre the potential is known, below it the flux
        bc = np.where(g.nodes[:, 2] > g.center[2], 0, 1).astype(np.uint8)
        return {"bc": bc, "known": np.where(bc == 0, _smooth(g, rng), 0.5 * _smooth(g, rng))}
    params = []  # He-normal weights, small biases, as a trained network has
    widths = [6] + [16] * (len(DILATIONS) - 1) + [1]
    for ci, co in zip(widths[:-1], widths[1:]):
        params.append(rng.standard_normal(co * ci * 27) * math.sqrt(2.0 / (ci * 27)))
        params.append(0.05 * rng.standard_normal(co))
    params = np.concatenate(params).astype(np.float32)
    u = _smooth(g, rng)
    if op == "guess":
        return {"params": params, "known": u}
    # one training problem: the input channels at the boundary's voxels and the flux to learn
    s = 1.0 / math.sqrt(float(np.mean(u * u)))
    a = g.weights / g.h ** 2
    b = 0.1 * _smooth(g, rng) * s
    vox = ((g.index[:, 2] * g.n[1] + g.index[:, 1]) * g.n[0] + g.index[:, 0]).astype(np.int32)
    x = np.zeros((6, g.n[0] * g.n[1] * g.n[2]), dtype=np.float32)
    for c, v in enumerate([a, a * g.normals[:, 0], a * g.normals[:, 1], a * g.normals[:, 2], a * s * u, a * b]):
        x[c, vox] = v
    t = (s * g.h * _smooth(g, rng)).astype(np.float32)
    wt = (g.weights / np.sum(g.weights * t.astype(np.float64) ** 2)).astype(np.float32)
    return {"params": params, "x": x, "vox": vox, "tgt": t, "wt": wt}


# ------------------------------------------------------------------ the measured path


def _plan(g, case, **kw):
    return B.Plan(g, KERNEL[case["kernel"]], precision=PREC[case["precision"]], nu=NU, mu=MU, **kw)


def prepare(case, seed):
    op = case["op"]
    dev = torch.device("cuda")
    t = {k: torch.from_numpy(np.ascontiguousarray(v)).to(dev) for k, v in _data(case, seed).items() if k != "params"}
    st = dict(t, op=op)
    if op == "batch":
        st["batch"] = B.Batch([_plan(g, case) for g in _batch_geoms(case)], nrhs=case["nrhs"])
        st["r"] = torch.empty_like(t["q"])
        return st
    g = _geom(case)
    if op == "apply":
        st["plan"] = _plan(g, case)
        st["r"] = torch.empty_like(t["u"])
    elif op == "grid":
        st["plan"] = _plan(g, case)
        inf = st["plan"].info()
        st["out"] = torch.empty((inf["z_count"], g.n[1], g.n[0]), dtype=torch.float64, device=dev)
    elif op == "gmres":
        st["plan"] = _plan(g, case, keep_fp64=True)
        st["x"] = torch.zeros_like(t["known"])
    elif op == "cg":
        st["plan"] = _plan(g, case)
        st["x"] = torch.zeros_like(t["u"])
    else:
        st["net"] = B.Net(g.n[0], DILATIONS, seed=1)
        st["net"].set_params(_data(case, seed)["params"])
        if op == "guess":
            st["plan"] = _plan(g, case)
            st["xbuf"] = torch.empty((6, st["net"].V), dtype=torch.float32, device=dev)
            st["x0"] = torch.empty_like(t["known"])
    return st


def run(st):
    op = st["op"]
    if op == "apply":
        return st["plan"].apply(st["q"], st["u"], st["r"])
    if op == "grid":
        return st["plan"].eval_grid(st["q"], st["u"], st["out"])
    if op == "batch":
        st["batch"].apply(st["q"], st["u"], st["r"])
        return st["r"]
    if op == "gmres":
        st["plan"].solve(st["bc"], st["known"], st["x"], tol=1e-6, use_x0=0, refine=1)
        return st["x"]
    if op == "cg":
        st["plan"].solve_cg(st["u"], st["x"], tol=1e-6, use_x0=0)
        return st["x"]
    if op == "grad":
        loss, grad = st["net"].gradients(st["x"], st["vox"], st["tgt"], st["wt"])
        return {"loss": loss, "grad": grad}
    return st["net"].guess(st["plan"], None, st["known"], st["xbuf"], st["x0"])


# ------------------------------------------------------------------ work and tolerance


def _pad(n):
    return next(s for s in SIZES if s >= 2 * n)


def _apply_work(g, kernel, precision):
    """Node data and kernel spectra in, result out; the transforms of the padded grid (half of it: the
    data are real) and the spectral products."""
    fields, spectra, outs, nc = {"l2d": (3, 3, 1, 1), "l3d": (4, 4, 1, 1), "nav": (9, 24, 3, 3), "hs": (3, 8, 3, 3)}[kernel]
    size = {"fp64": 8, "fp32": 4, "bf16": 2}[precision]
    pads = [_pad(k) for k in g.n[: g.dim]]
    full = math.prod(pads)
    octant = math.prod(p // 2 + 1 for p in pads)
    terms = {"l2d": 3, "l3d": 4, "nav": 27, "hs": 9}[kernel]
    node = g.m * (8 * (3 * nc + 1 + g.dim + 2 * nc * nc) + 16)
    flops = (fields + outs) * 2.5 * full * math.log2(full) + terms * 4.0 * full / 2
    return node + octant * spectra * size, flops


def work(case):
    op = case["op"]
    if op == "batch":
        ws = [_apply_work(g, case["kernel"], case["precision"]) for g in _batch_geoms(case)]
        return {"bytes": float(sum(b for b, _ in ws) * 1.0), "flops": float(case["nrhs"] * sum(f for _, f in ws))}
    g = _geom(case)
    if op in ("grad", "guess"):
        v = g.n[0] * g.n[1] * g.n[2]
        macs = 27 * (6 * 16 + 16 * 16 * (len(DILATIONS) - 2) + 16)
        if op == "grad":  # forward, data gradient (not of the input) and weight gradient
            back = 27 * (16 * 16 * (len(DILATIONS) - 2) + 16)
            return {"bytes": v * 24.0 + g.m * 12.0, "flops": 2.0 * v * (2 * macs + back)}
        b, f = _apply_work(g, "l3d", "fp64")
        return {"bytes": float(b + g.m * 16), "flops": f + 2.0 * v * macs}
    b, f = _apply_work(g, case["kernel"], case["precision"])
    if op == "grid":
        return {"bytes": float(b + 8 * g.n[0] * g.n[1] * (np.ptp(g.index[:, 2]) + 1)), "flops": f}
    if op == "gmres":  # about 40 iterations, each with one application
        return {"bytes": float(40 * b), "flops": 40.0 * f}
    if op == "cg":
        return {"bytes": float(35 * b), "flops": 35.0 * f}
    return {"bytes": float(b), "flops": f}


def tolerance(case):
    """About four times the largest distance from ``exact`` that was measured over listed and drawn cases.  The
    iterative solves stop at 1e-6 of their residual, so their solutions differ by that times the conditioning."""
    op = case["op"]
    if op == "grad":  # 7e-8: FP32 sums over the grid
        return {"rel": 1e-6}
    if op == "guess":  # 5e-4: FP16 activations
        return {"rel": 2e-3}
    if op == "gmres":  # 8e-6
        return {"rel": 4e-5}
    if op == "cg":  # 1.2e-4
        return {"rel": 5e-4}
    return {"rel": {"fp64": 1e-14, "fp32": 1.5e-6, "bf16": 1.5e-2}[case["precision"]]}  # 6e-16, 3e-7, 4e-3


# ------------------------------------------------------------------ FP64 reference


_PAIRS = [(0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2)]


class _Exact:
    """The discrete operator in FP64: kernels sampled on the padded grid, torch's FFT, node terms."""

    def __init__(self, g, kernel, dev):
        self.g, self.kernel, self.dev = g, kernel, dev
        self.nc = 3 if kernel in ("nav", "hs") else 1
        d = g.dim
        self.shape = tuple(_pad(k) for k in reversed(g.n[:d]))  # (z, y, x)
        idx = torch.as_tensor(g.index, device=dev)
        lin = idx[:, d - 1]
        for a in range(d - 2, -1, -1):
            lin = lin * self.shape[d - 1 - a] + idx[:, a]
        self.lin = lin
        self.w = torch.as_tensor(g.weights, device=dev)
        self.nrm = torch.as_tensor(g.normals, device=dev).T.contiguous()
        self.spec = {}
        ax = []
        for a in range(d):
            p = self.shape[d - 1 - a]
            k = torch.arange(p, device=dev, dtype=torch.float64)
            k = torch.where(k < p // 2, k, k - p) * g.h
            ax.append(k.reshape([-1 if i == d - 1 - a else 1 for i in range(d)]))
        self.ax = ax
        self.L = math.log(1.0 + math.sqrt(2.0))

    def _khat(self, name, fn, k0):
        """Transform of kernel fn(offsets, r) with value k0 at offset 0."""
        if name in self.spec:
            return self.spec[name]
        x = [a.expand(self.shape) for a in self.ax]
        r2 = sum(a * a for a in self.ax)
        zero = (0,) * len(self.shape)
        r2[zero] = 1.0
        v = fn(x, r2, torch.sqrt(r2)).clone()
        v[zero] = k0
        for dim, p in enumerate(self.shape):  # offsets of half the padded length: no pair reaches them
            v.select(dim, p // 2).zero_()
        k = torch.fft.rfftn(v)
        if self.kernel != "nav":  # Navier's 24 spectra are made when needed
            self.spec[name] = k
        return k

    def _hat(self, f):
        b = torch.zeros(math.prod(self.shape), dtype=torch.float64, device=self.dev)
        b.index_add_(0, self.lin, f)
        return torch.fft.rfftn(b.reshape(self.shape))

    def grid_sums(self, q, u):
        """[nrhs][nc] grids of D[u] - S[q] (half-space: K[q]); q, u: [nrhs][nc][m]."""
        h, w, n, d, pi = self.g.h, self.w, self.nrm, self.g.dim, math.pi
        nr, nc = q.shape[0], self.nc
        acc = [[0.0] * nc for _ in range(nr)]
        if self.kernel in ("l2d", "l3d"):
            if d == 2:
                ks = self._khat("u", lambda x, r2, r: -torch.log(r) / (2 * pi), (1.0 - math.log(0.5 * h)) / (2 * pi))
                kg = [self._khat(i, lambda x, r2, r, i=i: -x[i] / (2 * pi * r2), 0.0) for i in range(2)]
            else:
                ks = self._khat("u", lambda x, r2, r: 1.0 / (4 * pi * r), self.L / (pi * h))
                kg = [self._khat(i, lambda x, r2, r, i=i: -x[i] / (4 * pi * r2 * r), 0.0) for i in range(3)]
            for j in range(nr):
                s = ks * self._hat(q[j, 0] * w)
                for i in range(d):  # the double layer reads the kernel at source - target
                    s = s + kg[i] * self._hat(u[j, 0] * n[i] * w)
                acc[j][0] = -s
        elif self.kernel == "hs":
            g0, a0 = 1.0 / (2 * pi * MU), 4.0 * self.L / h / (2 * pi * MU)
            fns = {(0, 0): (lambda x, r2, r: g0 * ((1 - NU) / r + NU * x[0] ** 2 / (r2 * r)), a0 * (1 - 0.5 * NU)),
                   (1, 1): (lambda x, r2, r: g0 * ((1 - NU) / r + NU * x[1] ** 2 / (r2 * r)), a0 * (1 - 0.5 * NU)),
                   (2, 2): (lambda x, r2, r: g0 * (1 - NU) / r, a0 * (1 - NU)),
                   (0, 1): (lambda x, r2, r: g0 * NU * x[0] * x[1] / (r2 * r), 0.0),
                   (0, 2): (lambda x, r2, r: -0.5 * g0 * (1 - 2 * NU) * x[0] / r2, 0.0),
                   (1, 2): (lambda x, r2, r: -0.5 * g0 * (1 - 2 * NU) * x[1] / r2, 0.0)}
            for j in range(nr):
                f = [self._hat(q[j, b] * w) for b in range(3)]
                for a in range(3):
                    for b in range(3):
                        key = (min(a, b), max(a, b))
                        k = self._khat(key, *fns[key])
                        sign = -1.0 if a > b and key != (0, 1) else 1.0
                        acc[j][a] = acc[j][a] + sign * k * f[b]
        else:
            pre, k0 = 1.0 / (16 * pi * MU * (1 - NU)), 4.0 * self.L / h * ((3 - 4 * NU) + 1.0 / 3.0)
            for b in range(3):  # single layer
                f = [self._hat(q[j, b] * w) if bool(q[j, b].any()) else None for j in range(nr)]
                for a in range(3):
                    def disp(x, r2, r, a=a, b=b):
                        v = x[a] * x[b] / (r2 * r)
                        return pre * (v + (3 - 4 * NU) / r if a == b else v)
                    k = self._khat(None, disp, pre * k0 if a == b else 0.0)
                    for j in range(nr):
                        if f[j] is not None:
                            acc[j][a] = acc[j][a] - k * f[j]
            c1 = 1.0 - 2.0 * NU
            for i, l in _PAIRS:  # double layer: the stress of the fundamental displacement
                f = [self._hat((u[j, i] * n[l] + (u[j, l] * n[i] if i != l else 0.0)) * w) for j in range(nr)]
                for a in range(3):
                    def stress(x, r2, r, a=a, i=i, l=l):
                        v = 3.0 * x[i] * x[l] * x[a] / (r2 * r)
                        if a == i:
                            v = v + c1 * x[l] / r
                        if a == l:
                            v = v + c1 * x[i] / r
                        if i == l:
                            v = v - c1 * x[a] / r
                        return -v / (8 * pi * (1 - NU) * r2)
                    k = self._khat(None, stress, 0.0)
                    for j in range(nr):
                        acc[j][a] = acc[j][a] - k * f[j]
        return [[torch.fft.irfftn(acc[j][a], s=self.shape) if torch.is_tensor(acc[j][a])
                 else torch.zeros(self.shape, dtype=torch.float64, device=self.dev) for a in range(nc)] for j in range(nr)]

    def _self(self):
        """Exact single-layer self term minus the grid's value at offset 0, per node ([nc][nc][m])."""
        h, w, n, pi, L = self.g.h, self.w, self.nrm, math.pi, self.L
        if self.kernel == "l2d":
            return ((math.log(0.5 * h) - torch.log(0.5 * w)) * w / (2 * pi))[None, None]
        if self.kernel == "l3d":
            return (torch.sqrt(w) * L / pi - w * L / (pi * h))[None, None]
        out = torch.zeros(3, 3, w.numel(), dtype=torch.float64, device=self.dev)
        if self.kernel == "hs":
            for a, f in enumerate((1 - 0.5 * NU, 1 - 0.5 * NU, 1 - NU)):
                out[a, a] = -4.0 * L / (2 * pi * MU) * f * (torch.sqrt(w) - w / h)
            return out
        pre = 1.0 / (16 * pi * MU * (1 - NU))
        for a in range(3):
            for b in range(3):
                d = 1.0 if a == b else 0.0
                out[a, b] = pre * 4.0 * L * (torch.sqrt(w) * ((3 - 4 * NU) * d + 0.5 * (d - n[a] * n[b]))
                                             - w / h * ((3 - 4 * NU) + 1.0 / 3.0) * d)
        return out

    def _at_nodes(self, grids):
        return torch.stack([t.reshape(-1)[self.lin] for t in grids])

    def apply(self, q, u):
        """r [nc][m] of one (q, u), with the implicit free term."""
        nc, m = self.nc, self.g.m
        q, u = q.reshape(nc, m), u.reshape(nc, m)
        if self.kernel == "hs":
            r = self._at_nodes(self.grid_sums(q[None], u[None])[0]) - u
        else:
            if not hasattr(self, "c"):
                ones = torch.zeros(nc, nc, m, dtype=torch.float64, device=self.dev)
                for l in range(nc):
                    ones[l, l] = 1.0
                if self.kernel == "nav":  # one sweep over the kernels for all four data sets
                    gs = self.grid_sums(torch.cat([q[None], torch.zeros_like(ones)]), torch.cat([u[None], ones]))
                    first, gs = gs[0], gs[1:]
                else:
                    first, gs = None, self.grid_sums(torch.zeros_like(ones), ones)
                self.c = -torch.stack([self._at_nodes(t) for t in gs], 1)  # [row][column][m]
                r = self._at_nodes(first) if first is not None else None
            else:
                r = None
            if r is None:
                r = self._at_nodes(self.grid_sums(q[None], u[None])[0])
            r = r + (self.c * u[None]).sum(1)
        return r - (self._self() * q[None]).sum(1)


def _gmres(op, b, steps=200, tol=1e-13):
    """Full GMRES in FP64 (one cycle, modified Gram-Schmidt twice)."""
    beta = b.norm()
    V, H = [b / beta], np.zeros((steps + 1, steps))
    for k in range(steps):
        w = op(V[k])
        for _ in range(2):
            for i, v in enumerate(V):
                h = float(torch.dot(v, w))
                H[i, k] += h
                w = w - h * v
        H[k + 1, k] = float(w.norm())
        e = np.zeros(k + 2)
        e[0] = float(beta)
        y, *_ = np.linalg.lstsq(H[: k + 2, : k + 1], e, rcond=None)
        if np.linalg.norm(H[: k + 2, : k + 1] @ y - e) <= tol * float(beta):
            break
        V.append(w / H[k + 1, k])
    return sum(float(c) * v for c, v in zip(y, V))


def _net(params, x, n):
    """y [n^3] of the network in FP64; params a flat tensor, x [6][n^3]."""
    widths = [6] + [16] * (len(DILATIONS) - 1) + [1]
    act, off = x, 0
    for l, (ci, co, d) in enumerate(zip(widths[:-1], widths[1:], DILATIONS)):
        W = params[off:off + co * ci * 27].reshape(co, ci, 27)
        b = params[off + co * ci * 27:off + co * ci * 27 + co]
        off += co * ci * 27 + co
        p = torch.nn.functional.pad(act.reshape(ci, n, n, n), (d,) * 6)
        s = b[:, None].expand(co, n ** 3)
        for t in range(27):
            dz, dy, dx = t // 9, (t // 3) % 3, t % 3
            win = p[:, d * dz:d * dz + n, d * dy:d * dy + n, d * dx:d * dx + n].reshape(ci, -1)
            s = s + W[:, :, t] @ win
        act = torch.relu(s) if l + 1 < len(DILATIONS) else s
    return act.reshape(-1)


def exact(case, seed):
    op = case["op"]
    dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
    d = {k: torch.as_tensor(v, device=dev) for k, v in _data(case, seed).items()}
    if op == "batch":
        out, o = [], 0
        for g in _batch_geoms(case):
            ex = _Exact(g, case["kernel"], dev)
            for _ in range(case["nrhs"]):
                out.append(ex.apply(d["q"][o:o + g.m], d["u"][o:o + g.m]).reshape(-1))
                o += g.m
        return torch.cat(out).cpu().numpy()
    g = _geom(case)
    if op == "apply":
        return _Exact(g, case["kernel"], dev).apply(d["q"], d["u"]).reshape(-1).cpu().numpy()
    if op == "grid":
        out = _Exact(g, case["kernel"], dev).grid_sums(d["q"][None, None], d["u"][None, None])[0][0]
        lo, hi = int(g.index[:, 2].min()), int(g.index[:, 2].max())
        return (-out[lo:hi + 1, : g.n[1], : g.n[0]]).contiguous().cpu().numpy()
    if op == "cg":  # S[q] = c u + D[u]; scaled by the weights' roots the system is symmetric
        ex = _Exact(g, case["kernel"], dev)
        zero = torch.zeros_like(d["u"])
        sw = torch.sqrt(ex.w)
        b = ex.apply(zero, d["u"])[0] * sw
        y = _gmres(lambda v: -ex.apply(v / sw, zero)[0] * sw, b)
        return (y / sw).cpu().numpy()
    if op == "gmres":
        ex = _Exact(g, case["kernel"], dev)
        dirichlet = d["bc"] == 0
        zero = torch.zeros_like(d["known"])

        def split(v, unknown):
            on_q = dirichlet if unknown else ~dirichlet
            return ex.apply(torch.where(on_q, v, zero), torch.where(on_q, zero, v))[0]

        ex.apply(zero, zero)  # the free term
        # columns scaled by the diagonal: minus the self term where q is sought, c where u is
        diag = torch.where(dirichlet, -torch.sqrt(ex.w) * ex.L / math.pi, ex.c[0, 0])
        diag = torch.where(diag == 0, torch.ones_like(diag), diag)
        y = _gmres(lambda v: split(v / diag, True), -split(d["known"], False))
        return (y / diag).cpu().numpy()
    n = g.n[0]
    params = d["params"].double()
    if op == "guess":
        ex = _Exact(g, "l3d", dev)
        u = d["known"]
        s = 1.0 / torch.sqrt(torch.mean(u * u))
        b = -ex.apply(torch.zeros_like(u), u)[0]
        a = ex.w / g.h ** 2
        idx = torch.as_tensor(g.index, device=dev)
        vox = (idx[:, 2] * n + idx[:, 1]) * n + idx[:, 0]
        x = torch.zeros(6, n ** 3, dtype=torch.float64, device=dev)
        x[:, vox] = torch.stack([a, a * ex.nrm[0], a * ex.nrm[1], a * ex.nrm[2], a * s * u, a * s * b])
        with torch.no_grad():
            return (_net(params, x, n)[vox] / (s * g.h)).cpu().numpy()
    params = params.requires_grad_(True)
    y = _net(params, d["x"].double(), n)
    loss = (d["wt"].double() * (y[d["vox"].long()] - d["tgt"].double()) ** 2).sum()
    loss.backward()
    return {"loss": float(loss.detach()), "grad": params.grad.cpu().numpy()}
