"""The work that a user of this framework has it do, as timed cases.

The paper's cells are spheres of 2,000 to 5,000 vertices (10,000 to 30,000
tetrahedra); the repository's own workloads reach from one cell of 1,000
nodes over one of 20,000 to batches of 4,096 cells.  Every case goes through
the Python entry points on device tensors in the handle's internal node
order, as a simulation or a fit keeps them between calls.

Cases are dicts of
  kind    what is called (see `run`)
  cells   number of cells
  nodes   nodes of a cell, about (uneven: the largest cell)
  mesh    "own" every cell its own reference mesh (one size),
          "uneven" sizes spread from nodes / 40 to nodes,
          "shared" copies of one reference mesh
  regions material regions per cell (nucleus, cortex, rest) or 1
  tile    tetrahedra per tile, 0 = the default
  steps   plate steps (plate, bptt) or plate positions (curve)

Meshes are body-centred-cubic lattices clipped to a ball, their surface nodes
moved onto the sphere, every cell stretched to semi-axes of its own and
deformed by compression and shear with node noise.
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2003_03130_amd import CellBatch, HostLayout
from paper_2003_03130_amd.autograd import mr_forces
from paper_2003_03130_amd.quasistatic import QuasiStaticCompression
from paper_2003_03130_amd.relax import PlateCompression

K_PLATE = 100.0
MOBILITY = 1e-3 / 0.25


def _case(name, kind, cells, nodes, mesh, regions=1, tile=0, steps=0):
    return {"name": name, "kind": kind, "cells": cells, "nodes": nodes,
            "mesh": mesh, "regions": regions, "tile": tile, "steps": steps}


def listed():
    return [
        # the smallest call: forces and energy of one coarse cell, as an
        # immersed-cell simulation asks for them once a time step
        _case("forces_cell_1k", "forces", 1, 1000, "own"),
        # a fit of one cell of the paper's finest size with torch: loss on
        # forces and energy, gradients of positions and parameters
        _case("autograd_cell_5k", "autograd", 1, 5000, "own"),
        # the finest single cell, forward and backward captured once and
        # replayed (differentiation configuration)
        _case("graph_cell_20k", "graph", 1, 20000, "own"),
        # the paper's suspension: 8 equal cells per run
        _case("forces_suspension_8", "forces", 8, 3100, "shared"),
        # vector-Jacobian products of cells with nucleus and cortex
        _case("backward_regions_64", "backward", 64, 2000, "own", regions=3),
        # explicit plate compression (the paper's set-up) of a batch
        _case("plate_32", "plate", 32, 4000, "own", steps=40),
        # its parameter gradient by checkpointed back-propagation
        _case("bptt_8", "bptt", 8, 2500, "own", steps=40),
        # a batch of uneven cells, forces and gradient in one step
        _case("step_uneven_256", "step", 256, 3800, "uneven"),
        # forces of a large uneven batch
        _case("forces_uneven_1024", "forces", 1024, 3800, "uneven"),
        # the largest: 4,096 cells that share one mesh
        _case("step_shared_4096", "step", 4096, 2000, "shared"),
        # Taylor deformation and strain of every cell of a batch
        _case("shape_uneven_512", "shape", 512, 3800, "uneven"),
        # force-indentation curve: Newton-CG equilibria between plates
        _case("curve_16", "curve", 16, 1900, "own", steps=3),
    ]


# kind: (cells, nodes, largest number of nodes over all cells, meshes);
# the ranges that the listed cases stand for
_RANGES = {
    "forces": ((1, 2048), (300, 20000), 2_500_000, ("own", "uneven", "shared")),
    "autograd": ((1, 64), (300, 20000), 300_000, ("own", "uneven", "shared")),
    "graph": ((1, 64), (300, 20000), 300_000, ("own", "uneven")),
    "backward": ((1, 512), (300, 20000), 1_500_000, ("own", "uneven", "shared")),
    "step": ((1, 2048), (300, 20000), 4_000_000, ("own", "uneven", "shared")),
    "plate": ((1, 128), (500, 9000), 400_000, ("own", "shared")),
    "bptt": ((1, 32), (500, 9000), 100_000, ("own", "shared")),
    "shape": ((1, 1024), (300, 9000), 2_000_000, ("own", "uneven", "shared")),
    "curve": ((1, 16), (600, 2600), 30_000, ("own",)),
}


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(sorted(_RANGES))
    (c0, c1), (n0, n1), most, meshes = _RANGES[kind]
    nodes = _log(rng, n0, n1)
    cells = _log(rng, c0, max(c0, min(c1, most // nodes)))
    mesh = rng.choice(meshes)
    if mesh == "uneven" and nodes < 2000:
        mesh = "own"
    # handles of many distinct cells take their time to lay out on the host
    if mesh != "shared":
        cells = max(1, min(cells, 1_500_000 // nodes))
    regions = rng.choice((1, 1, 3)) if kind in ("forces", "backward", "step") else 1
    tile = rng.choice((0, 0, 0, 512, 640, 1024))
    steps = rng.randint(10, 40) if kind in ("plate", "bptt") else (
        rng.randint(1, 3) if kind == "curve" else 0)
    c = _case("", kind, cells, nodes, mesh, regions, tile, steps)
    del c["name"]
    return c


# ------------------------------------------------------------------ meshes
@functools.lru_cache(maxsize=64)
def _ball(n_target):
    """(x, tets, sigma) of a unit ball with about n_target nodes: every two
    neighbouring body centres and each edge of the face between them span a
    tetrahedron; those with a corner outside are dropped, and nodes on the
    surface are moved out to the sphere.  sigma: standard deviation of a
    node's noise, 8 % of the smallest height of its tetrahedra (so that the
    noise turns none of them inside out)."""
    a = (2.0 * (4.0 / 3.0 * math.pi) / n_target) ** (1.0 / 3.0)
    a /= 1.0 + 0.42 * a  # the clipped layer
    n = int(math.ceil(1.0 / a)) + 1
    m = 2 * n + 1
    g = (np.arange(m) - n) * a
    corner = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
    x = np.concatenate([corner, corner + 0.5 * a])
    x = x + np.array([0.11, 0.07, 0.05]) * a  # no lattice point on the axis
    idx = np.arange(m ** 3).reshape(m, m, m)
    tets = []
    for ax in range(3):
        u, v = (ax + 1) % 3, (ax + 2) % 3
        i = np.moveaxis(idx, (ax, u, v), (0, 1, 2))
        c0 = i[:-1, :-1, :-1] + m ** 3
        c1 = i[1:, :-1, :-1] + m ** 3
        f = [i[1:, :-1, :-1], i[1:, 1:, :-1], i[1:, 1:, 1:], i[1:, :-1, 1:]]
        for k in range(4):
            tets.append(np.stack([c0, c1, f[k], f[(k + 1) % 4]], -1).reshape(-1, 4))
    tets = np.concatenate(tets)
    tets = tets[(np.linalg.norm(x, axis=1) < 1.0 - 0.35 * a)[tets].all(axis=1)]
    # surface nodes: corners of faces that one tetrahedron has
    f = np.sort(tets[:, [[1, 2, 3], [0, 2, 3], [0, 1, 3], [0, 1, 2]]].reshape(-1, 3), axis=1)
    key = (f[:, 0].astype(np.int64) * len(x) + f[:, 1]) * len(x) + f[:, 2]
    _, first, count = np.unique(key, return_index=True, return_counts=True)
    surface = np.unique(f[first[count == 1]])
    x[surface] /= np.linalg.norm(x[surface], axis=1, keepdims=True)
    for _ in range(2):  # drop flat ones, then the nodes that none uses
        e = x[tets[:, :3]] - x[tets[:, 3:]]
        s = np.linalg.svd(e, compute_uv=False)
        tets = tets[s[:, 0] < 30.0 * s[:, 2]]
    d = np.linalg.det(x[tets[:, :3]] - x[tets[:, 3:]])
    tets[d < 0] = tets[d < 0][:, [1, 0, 2, 3]]
    used = np.zeros(len(x), bool)
    used[tets.ravel()] = True
    new = np.cumsum(used) - 1
    x, tets = np.ascontiguousarray(x[used]), np.ascontiguousarray(new[tets].astype(np.int32))
    p = x[tets]
    det = np.abs(np.linalg.det(p[:, :3] - p[:, 3:]))
    area = [np.linalg.norm(np.cross(p[:, i] - p[:, k], p[:, j] - p[:, k]), axis=1)
            for i, j, k in ((0, 1, 2), (0, 1, 3), (0, 2, 3), (1, 2, 3))]
    sigma = np.full(len(x), np.inf)
    np.minimum.at(sigma, tets.ravel(), np.repeat(0.08 * det / np.max(area, axis=0), 4))
    return x, tets, sigma


def _ladder(case):
    """The mesh sizes of uneven cells (each cell's, the same for every seed)."""
    sizes = np.linspace(case["nodes"] / 40.0, case["nodes"], 24).astype(int)
    return sizes[np.arange(case["cells"]) * 7 % len(sizes)]


def _radial_regions(x, tets):
    r = np.linalg.norm(x[tets].mean(axis=1), axis=1)
    return np.where(r < 0.45, 1, np.where(r > 0.85, 2, 0)).astype(np.uint8)


def _host(case, seed):
    """The reference meshes: dict of CSR offsets, x, tets, regions (of the
    shared mesh alone where the cells share one)."""
    rng = np.random.default_rng(seed)
    C, n = case["cells"], case["nodes"]
    if case["mesh"] == "shared":
        balls, axes = [_ball(n)], np.ones((1, 3))
    elif case["mesh"] == "uneven":
        balls = [_ball(int(v)) for v in _ladder(case)]
        axes = rng.uniform(0.7, 1.3, (C, 3))
    else:
        balls = [_ball(n)] * C
        axes = rng.uniform(0.7, 1.3, (C, 3))
    if case["kind"] == "curve":
        # oblate on the axis of compression: such cells cannot roll
        axes = rng.uniform((1.05, 1.0, 0.75), (1.25, 1.2, 0.85), (C, 3))
    if case["kind"] in ("plate", "bptt"):
        axes = np.ones((C, 3))
    x = np.concatenate([b[0] * s for b, s in zip(balls, axes)])
    sigma = np.concatenate([b[2][:, None] * s for b, s in zip(balls, axes)])
    tets = np.concatenate([b[1] for b in balls])
    reg = None
    if case["regions"] > 1:
        reg = np.concatenate([_radial_regions(*b[:2]) for b in balls])
    return {"node_off": np.concatenate([[0], np.cumsum([len(b[0]) for b in balls])]),
            "tet_off": np.concatenate([[0], np.cumsum([len(b[1]) for b in balls])]),
            "x": x, "tets": tets, "sigma": sigma, "regions": reg}


def _options(case):
    return {"tile_tets": case["tile"] or None,
            "n_regions": case["regions"] if case["regions"] > 1 else None}


def _device_inputs(case, h, seed):
    """Positions, cotangents and parameters in the caller's node order
    (all cells, (N, 3) on the GPU)."""
    C = case["cells"]
    g = torch.Generator(device="cuda").manual_seed(int(seed))
    rng = np.random.default_rng([int(seed), 1])
    x, sigma = torch.from_numpy(h["x"]).cuda(), torch.from_numpy(h["sigma"]).cuda()
    counts = np.diff(h["node_off"])
    if case["mesh"] == "shared":
        x, sigma = x.repeat(C, 1), sigma.repeat(C, 1)
        counts = np.repeat(counts, C)
    cell = torch.repeat_interleave(torch.arange(C, device="cuda"),
                                   torch.from_numpy(counts).cuda())
    lam = 1.0 - rng.uniform(0.0, 0.8, C)
    A = np.zeros((C, 3, 3))
    A[:, 0, 0] = A[:, 1, 1] = 1.0
    A[:, 0, 2] = rng.uniform(0.0, 0.5, C)
    A[:, 2, 2] = lam
    if case["kind"] in ("plate", "bptt", "curve"):
        y = x
    else:
        eta = torch.randn(x.shape, generator=g, device="cuda", dtype=torch.float32)
        y = torch.empty_like(x)
        At = torch.from_numpy(A).cuda()
        for s in range(0, len(x), 1 << 20):
            c = cell[s:s + (1 << 20)]
            xs = x[s:s + (1 << 20)] + sigma[s:s + (1 << 20)] * eta[s:s + (1 << 20)].double()
            y[s:s + (1 << 20)] = (At[c] * xs[:, None, :]).sum(-1)
    fbar = torch.randn(x.shape, generator=g, device="cuda", dtype=torch.float32)
    n_mat = C * case["regions"]
    mu = rng.uniform(0.5, 2.0, n_mat)
    theta = np.stack([mu, mu * rng.uniform(5.0, 50.0, n_mat), rng.uniform(0.0, 1.0, n_mat)], 1)
    ebar = rng.normal(size=C)
    return {"y": y.float(), "fbar": fbar, "theta": theta, "ebar": ebar, "cell": cell}


def _targets(case, seed):
    return np.random.default_rng([int(seed), 2]).uniform(0.0, 20.0, (case["steps"], case["cells"]))


def _plates(case):
    n = case["steps"]
    return 1.0 - 2.0 * 0.2 * np.arange(n) / 200.0 - 0.02, -0.98


def prepare(case, seed):
    h = _host(case, seed)
    opt = _options(case)
    if case["mesh"] == "shared":
        cb = CellBatch.template(case["cells"], h["x"], h["tets"], regions=h["regions"], **opt)
    else:
        cb = CellBatch(h["node_off"], h["tet_off"], h["x"], h["tets"], regions=h["regions"], **opt)
    d = _device_inputs(case, h, seed)
    order = torch.from_numpy(cb.new_to_old).cuda()
    s = {"kind": case["kind"], "cb": cb,
         "y": d["y"][order].t().contiguous().reshape(-1),
         "fbar": d["fbar"][order].t().contiguous().reshape(-1),
         "ebar": torch.from_numpy(d["ebar"]).cuda(),
         "theta": torch.from_numpy(d["theta"]).cuda()}
    cb.set_params(*d["theta"].T.copy())
    kind = case["kind"]
    if kind == "autograd":
        s["y"].requires_grad_(True)
        s["theta"].requires_grad_(True)
    elif kind == "graph":
        s["out"] = (cb.empty_nodes(), torch.empty(cb.n_cells, dtype=torch.float64, device="cuda"),
                    cb.empty_nodes(), torch.empty(3 * cb.n_mat, dtype=torch.float64, device="cuda"))
        f, e, yb, tb = s["out"]
        s["stream"] = torch.cuda.Stream()
        torch.cuda.synchronize()
        cb.graph_capture(6, s["y"], f, e, fbar=s["fbar"], ebar=s["ebar"], ybar=yb, thetabar=tb,
                         stream=s["stream"])
    elif kind in ("plate", "bptt"):
        top, bottom = _plates(case)
        s["pc"] = PlateCompression(cb, top, bottom, K_PLATE, MOBILITY, checkpoint=10)
        s["target"] = torch.from_numpy(_targets(case, seed)).cuda()
    elif kind == "curve":
        s["qs"] = QuasiStaticCompression(cb, K_PLATE)
        z = d["y"][:, 2].double()
        lo = torch.full((cb.n_cells,), math.inf, device="cuda", dtype=torch.float64)
        hi = -lo
        lo.scatter_reduce_(0, d["cell"], z, "amin")
        hi.scatter_reduce_(0, d["cell"], z, "amax")
        lo, hi = lo.cpu().numpy(), hi.cpu().numpy()
        at = np.linspace(0.04, 0.2, case["steps"])
        s["tops"] = hi[None] - at[:, None] * (hi - lo)[None]
        s["bottom"] = lo
    elif kind == "shape":
        s["d_ref"] = torch.full((cb.n_cells,), 2.0, dtype=torch.float64, device="cuda")
    torch.cuda.synchronize()
    return s


def run(s):
    kind, cb = s["kind"], s["cb"]
    if kind == "forces":
        f, e = cb.forces(s["y"])
        return {"f": f, "energy": e}
    if kind == "backward":
        yb, tb = cb.backward(s["y"], s["fbar"], s["ebar"])
        return {"ybar": yb, "thetabar": tb}
    if kind == "step":
        f, e, yb, tb = cb.forces_and_backward(s["y"], s["fbar"], s["ebar"])
        return {"f": f, "energy": e, "ybar": yb, "thetabar": tb}
    if kind == "graph":
        cb.graph_launch()
        f, e, yb, tb = s["out"]
        return {"f": f, "energy": e, "ybar": yb, "thetabar": tb}
    if kind == "autograd":
        f, e = mr_forces(s["y"], s["theta"], cb)
        yb, tb = torch.autograd.grad((f, e), (s["y"], s["theta"]), (s["fbar"], s["ebar"]))
        return {"f": f, "energy": e, "ybar": yb, "thetabar": tb}
    if kind == "plate":
        force, y, _ = s["pc"].forward(s["y"])
        return {"force": force, "y": y}
    if kind == "bptt":
        loss, grad, force = s["pc"].gradient(s["y"], s["target"], 1e-3)
        return {"loss": loss, "grad": grad, "force": force}
    if kind == "shape":
        return {"shape": cb.shape(s["y"], s["d_ref"])}
    top, bottom, _, y = s["qs"].curve(s["y"], s["tops"], s["bottom"])
    return {"top": top, "bottom": bottom, "y": y}


# ------------------------------------------------------- the same in 64 bits
class _Reference:
    """Mooney-Rivlin energy and forces of the meshes in float64 (torch), in
    the caller's node order."""

    def __init__(self, case, h):
        C = case["cells"]
        x = torch.from_numpy(h["x"]).cuda()
        m, n = len(h["tets"]), len(h["x"])
        tets = torch.from_numpy(h["tets"]).cuda().long()
        if case["mesh"] != "shared":
            tets = tets + torch.repeat_interleave(
                torch.from_numpy(h["node_off"][:-1]).cuda(),
                torch.from_numpy(np.diff(h["tet_off"])).cuda())[:, None]
        e = x[tets[:, :3]] - x[tets[:, 3:]]             # rows: reference edges
        self.B = torch.linalg.inv(e.transpose(1, 2))    # J = columns of edges
        self.V = torch.linalg.det(e).abs() / 6.0
        reg = torch.zeros(m, dtype=torch.long, device="cuda") if h["regions"] is None \
            else torch.from_numpy(h["regions"]).cuda().long()
        if case["mesh"] == "shared":
            cell = torch.zeros(m, dtype=torch.long, device="cuda")
        else:
            cell = torch.repeat_interleave(torch.arange(C, device="cuda"),
                                           torch.from_numpy(np.diff(h["tet_off"])).cuda())
        self.tets, self.cell, self.reg = tets, cell, reg
        self.R, self.C, self.n, self.shared = case["regions"], C, n, case["mesh"] == "shared"

    def energy(self, y, theta, tets, B, V, cell, reg, C):
        p = y[tets]
        F = (p[:, :3] - p[:, 3:]).transpose(1, 2) @ B
        Cg = F.transpose(1, 2) @ F
        J = torch.linalg.det(F)
        t = theta[cell * self.R + reg]
        mu, kappa, w = t[:, 0], t[:, 1], t[:, 2]
        TC = Cg.diagonal(dim1=1, dim2=2).sum(1)
        I2 = 0.5 * (TC ** 2 - (Cg * Cg).sum((1, 2)))
        r2 = J.abs() ** (-2.0 / 3.0)
        U = (0.5 * w * mu * (TC * r2 - 3.0) + 0.5 * (1.0 - w) * mu * (I2 * r2 * r2 - 3.0)
             + 0.5 * kappa * (J - 1.0) ** 2)
        return torch.zeros(C, dtype=torch.float64, device=y.device).index_add(0, cell, V * U)

    def groups(self):
        """(cells, nodes, tets, B, V, cell, reg) of groups of cells that fit
        the memory; the tables of a shared mesh are repeated here."""
        if not self.shared:
            yield 0, self.C, 0, None, self.tets, self.B, self.V, self.cell, self.reg
            return
        step = max(1, 2_000_000 // len(self.tets))
        for c0 in range(0, self.C, step):
            k = min(step, self.C - c0)
            off = torch.arange(k, device="cuda")
            yield (c0, k, c0 * self.n, (c0 + k) * self.n,
                   (self.tets[None] + (off * self.n)[:, None, None]).reshape(-1, 4),
                   self.B.repeat(k, 1, 1), self.V.repeat(k),
                   (self.cell[None] + off[:, None]).reshape(-1), self.reg.repeat(k))

    def evaluate(self, y, theta, fbar=None, ebar=None):
        f, E = torch.zeros_like(y), torch.zeros(self.C, dtype=torch.float64, device="cuda")
        yb, tb = torch.zeros_like(y), torch.zeros_like(theta)
        for c0, k, n0, n1, *tables in self.groups():
            yy = y[n0:n1].clone().requires_grad_(True)
            th = theta[c0 * self.R:(c0 + k) * self.R].clone().requires_grad_(True)
            e = self.energy(yy, th, *tables, k)
            g, = torch.autograd.grad(e.sum(), yy, create_graph=fbar is not None)
            f[n0:n1], E[c0:c0 + k] = -g.detach(), e.detach()
            if fbar is not None:
                loss = -(g * fbar[n0:n1]).sum() + (e * ebar[c0:c0 + k]).sum()
                a, b = torch.autograd.grad(loss, (yy, th))
                yb[n0:n1], tb[c0 * self.R:(c0 + k) * self.R] = a, b
        return f, E, yb, tb

    def plate_steps(self, y, theta, cell, tops, bottom, graph):
        """Top-plate forces of every step and the last positions."""
        force = []
        (c0, k, n0, n1, *tables), = self.groups()
        for top in tops:
            yy = y if graph else y.detach().requires_grad_(True)
            e = self.energy(yy, theta, *tables, k)
            g, = torch.autograd.grad(e.sum(), yy, create_graph=graph)
            dt, db = (yy[:, 2] - top).clamp(min=0.0), (bottom - yy[:, 2]).clamp(min=0.0)
            force.append(torch.zeros(k, dtype=torch.float64, device="cuda").index_add(
                0, cell, K_PLATE * dt ** 2))
            p = torch.zeros_like(yy)
            p[:, 2] = K_PLATE * (db ** 2 - dt ** 2)
            y = yy + MOBILITY * (-g + p)
            if not graph:
                y, force[-1] = y.detach(), force[-1].detach()
        return torch.stack(force), y


def _exact_shape(case, h, d):
    ref = _Reference(case, h)
    C, y = case["cells"], d["y"].double()
    out = torch.zeros(C, 10, dtype=torch.float64, device="cuda")
    for c0, k, n0, n1, tets, _, _, cell, _ in ref.groups():
        yy = y[n0:n1]
        x = torch.from_numpy(h["x"]).cuda()
        x = x.repeat(k, 1) if case["mesh"] == "shared" else x
        p = yy[tets]
        sign = torch.sign(torch.linalg.det(x[tets[:, :3]] - x[tets[:, 3:]]))
        V = sign * torch.linalg.det(p[:, :3] - p[:, 3:]) / 6.0
        r = p.mean(1)
        M = torch.zeros(k, dtype=torch.float64, device="cuda").index_add(0, cell, V)
        com = torch.zeros(k, 3, dtype=torch.float64, device="cuda").index_add(
            0, cell, V[:, None] * r) / M[:, None]
        q = r - com[cell]
        S = torch.zeros(k, 9, dtype=torch.float64, device="cuda").index_add(
            0, cell, (V[:, None, None] * q[:, :, None] * q[:, None, :]).reshape(-1, 9)).reshape(-1, 3, 3)
        tr = S.diagonal(dim1=1, dim2=2).sum(1)
        inertia = tr[:, None, None] * torch.eye(3, device="cuda", dtype=torch.float64) - S
        t = torch.linalg.eigvalsh(inertia.cpu()).cuda().flip(1)
        fac = (2.5 / M)[:, None]
        a = torch.stack([-t[:, 0] + t[:, 1] + t[:, 2], t[:, 0] - t[:, 1] + t[:, 2],
                         t[:, 0] + t[:, 1] - t[:, 2]], 1).mul(fac).clamp(min=0.0).sqrt()
        o = out[c0:c0 + k]
        o[:, 0], o[:, 1:4], o[:, 4:7] = M, com, a
        o[:, 7] = (a[:, 2] - a[:, 0]) / (a[:, 2] + a[:, 0])
    off = h["node_off"] if case["mesh"] != "shared" else np.arange(C + 1) * len(h["x"])
    for c in range(C):
        p = y[off[c]:off[c + 1]]
        best = 0.0
        for s in range(0, len(p), 2048):
            best = max(best, float(((p[s:s + 2048, None] - p[None]) ** 2).sum(-1).max()))
        out[c, 8] = math.sqrt(best)
    out[:, 9] = (out[:, 8] - 2.0) / 2.0
    return {"shape": out}


def exact(case, seed):
    """What run gives, in float64 from the same inputs.  Only the numbering
    of the nodes comes from the framework (its documented permutation; a
    wrong one would put every force on another node than here)."""
    kind = case["kind"]
    if kind == "curve":
        return None  # equilibria are as exact as the solver's tolerance
    h = _host(case, seed)
    d = _device_inputs(case, h, seed)
    if kind == "shape":
        return _exact_shape(case, h, d)
    opt = _options(case)
    if case["mesh"] == "shared":
        # every copy has the numbering of one
        one = HostLayout(h["node_off"], h["tet_off"], h["x"], h["tets"], tile_tets=opt["tile_tets"],
                         regions=h["regions"], n_regions=opt["n_regions"]).new_to_old
        order = (np.arange(case["cells"])[:, None] * len(one) + one[None]).reshape(-1)
    else:
        order = HostLayout(h["node_off"], h["tet_off"], h["x"], h["tets"], regions=h["regions"],
                           **opt).new_to_old
    order = torch.from_numpy(order).cuda()
    ref = _Reference(case, h)
    y, theta = d["y"].double(), torch.from_numpy(d["theta"]).cuda()

    def soa(v):
        return v[order].t().contiguous().reshape(-1)

    if kind in ("plate", "bptt"):
        if case["mesh"] == "shared" and case["cells"] * len(h["tets"]) > 2_000_000:
            return None
        # back-propagation keeps every step's tensors
        if kind == "bptt" and case["steps"] * case["cells"] * case["nodes"] > 2_500_000:
            return None
        tops, bottom = _plates(case)
        if kind == "plate":
            force, yn = ref.plate_steps(y, theta, d["cell"], tops, bottom, False)
            return {"force": force, "y": soa(yn)}
        theta.requires_grad_(True)
        force, _ = ref.plate_steps(y.requires_grad_(True), theta, d["cell"], tops, bottom, True)
        loss = 1e-3 * ((force - torch.from_numpy(_targets(case, seed)).cuda()) ** 2).sum()
        grad, = torch.autograd.grad(loss, theta)
        return {"loss": float(loss), "grad": grad, "force": force.detach()}
    if kind == "forces":
        f, e, _, _ = ref.evaluate(y, theta)
        return {"f": soa(f), "energy": e}
    f, e, yb, tb = ref.evaluate(y, theta, d["fbar"].double(), torch.from_numpy(d["ebar"]).cuda())
    tb = tb if kind == "autograd" else tb.reshape(-1)
    if kind == "backward":
        return {"ybar": soa(yb), "thetabar": tb}
    return {"f": soa(f), "energy": e, "ybar": soa(yb), "thetabar": tb}


# ---------------------------------------------------------------------- work
def work(case):
    """Least bytes and flops of a pass: per tetrahedron its 4 vertex numbers,
    inverse edge matrix and volume (56 B; a shared mesh once), per node the
    positions and what is read and written with them; 350 flops a
    tetrahedron forward, 900 backward, 1,060 both at once."""
    C = case["cells"]
    if case["mesh"] == "uneven":
        sizes = [(len(x), len(t)) for x, t, _ in (_ball(int(v)) for v in _ladder(case))]
        n, m = (float(np.sum(v)) for v in zip(*sizes))
    else:
        x, t, _ = _ball(case["nodes"])
        n, m = C * len(x), C * len(t)
    mesh = 56.0 * (m / C if case["mesh"] == "shared" else m)
    s = case["steps"]
    kind = case["kind"]
    if kind == "forces":
        return {"bytes": mesh + 24.0 * n, "flops": 350.0 * m}
    if kind == "backward":
        return {"bytes": mesh + 36.0 * n, "flops": 900.0 * m}
    if kind in ("step", "graph"):
        return {"bytes": mesh + 48.0 * n, "flops": 1060.0 * m}
    if kind == "autograd":
        return {"bytes": 2 * mesh + 60.0 * n, "flops": 1250.0 * m}
    if kind == "plate":
        return {"bytes": s * (mesh + 24.0 * n), "flops": s * 350.0 * m}
    if kind == "bptt":
        return {"bytes": s * (2 * mesh + 60.0 * n), "flops": s * 1250.0 * m}
    if kind == "shape":
        return {"bytes": 16.0 * (m / C if case["mesh"] == "shared" else m) + 12.0 * n,
                "flops": 80.0 * m}
    # a few Newton steps a position and some tens of Hessian products a step
    return {"bytes": s * 200.0 * (mesh + 60.0 * n), "flops": s * 200.0 * 900.0 * m}
