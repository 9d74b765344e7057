"""The workloads the library's speed is judged by.

Each case is one call (or one short sequence of calls) as a program that uses
the package makes it: a smooth of a device-resident mesh, a few more sweeps
on a mesh handle, several handles swept together, a batch of host meshes, or
the adjacency of a bare triangle list.  The meshes are those of the
repository's benchmark and tests: jittered grids with random or Union-Jack
diagonals, annuli, randomly relabelled grids, and grids refined at random
triangles (valence 3 to about 15, like the Delaunay meshes of random points).
They are made from the seed with plain torch on the GPU.

A server's requests run the kernels that the batched cases time; its latency
depends on when requests arrive, so it has no case of its own.
"""
import math
import random
import types

import numpy as np
import torch

import paper_1502_00355_amd as sl

DEV = "cuda"


def _case(name, kind, **kw):
    c = dict(name=name, kind=kind, mesh="grid", nx=64, ny=64, diag="random", jitter=0.4, refine=0.0, shuffled=False,
             form="jacobi", precision="f64", layout="aos", accept="ge", sweeps=100, tol=0.0, count=1)
    c.update(kw)
    return c


def listed():
    return [
        # one small mesh, a few sweeps: the call's latency (checks, ordering,
        # tiles, sweeps, results) is what counts
        _case("device_a_64", "device", nx=64, ny=64, diag="unionjack", jitter=0.3, sweeps=10),
        # Form B on a mesh of a thousand nodes, as the smallest mesh of the
        # paper's tables
        _case("device_b_1k", "device", nx=25, ny=25, refine=0.35, form="colored", sweeps=100),
        # a mesh of the paper's sizes run to convergence (largest displacement
        # of a sweep below 1e-9), irregular valence
        _case("device_a_30k_tol", "device", nx=131, ny=137, refine=0.35, shuffled=True, sweeps=10000, tol=1e-9),
        # Form B on the largest mesh of the paper's tables
        _case("device_b_100k", "device", nx=243, ny=239, refine=0.35, shuffled=True, form="colored", sweeps=50),
        # an interactive program: a mesh kept on the device, a few more sweeps
        # and the positions back each frame
        _case("handle_a_100k", "handle", nx=317, ny=311, sweeps=10),
        # an application's meshes of uneven size, kept on the device, swept
        # together: what a batch or a server step does
        _case("handles_a_40", "handles", nx=24, ny=450, jitter=0.35, sweeps=16, count=40),
        # a million nodes in arbitrary numbering, as a mesh file holds them
        _case("device_a_1024", "device", nx=1024, ny=1024, shuffled=True, sweeps=100),
        # single precision on a curved domain of ragged size
        _case("device_f32_annulus", "device", mesh="annulus", nx=1500, ny=2049, precision="f32", sweeps=100),
        # Form B on a large mesh
        _case("device_b_1500", "device", nx=1500, ny=1499, form="colored", sweeps=30),
        # a mesh that comes as a triangle list: neighbours, incidences, boundary
        _case("adjacency_1m", "adjacency", nx=1021, ny=997, shuffled=True, sweeps=0),
        # host arrays in and out, many meshes in one call
        _case("host_batch_40", "host", nx=24, ny=450, jitter=0.35, sweeps=50, count=40),
        # the largest: the benchmark's mesh, 16.8M nodes
        _case("device_a_4096", "device", nx=4096, ny=4096, sweeps=100),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _shape(rng, lo, hi):
    """Grid sides of lo..hi nodes in all, an aspect ratio of up to two."""
    n, asp = _log(rng, lo, hi), math.exp(rng.uniform(-0.35, 0.35))
    return max(8, round(math.sqrt(n) * asp)), max(8, round(math.sqrt(n) / asp))


def draw(rng):
    kind = rng.choice(["device", "device", "device", "device", "handle", "handles", "adjacency", "host"])
    c = _case(None, kind)
    del c["name"]
    c["jitter"] = rng.choice([0.3, 0.35, 0.4])
    c["shuffled"] = rng.random() < 0.4
    c["refine"] = rng.choice([0.0, 0.0, 0.35])
    c["diag"] = rng.choice(["random", "random", "random", "unionjack"])
    if kind == "device":
        c["form"] = rng.choice(["jacobi", "jacobi", "colored"])
        c["nx"], c["ny"] = _shape(rng, 500, 6e6 if c["form"] == "jacobi" else 2e6)
        if c["form"] == "jacobi" and rng.random() < 0.25:
            c["precision"] = "f32"
        if rng.random() < 0.2:
            c["mesh"], c["refine"] = "annulus", 0.0
        c["layout"] = rng.choice(["aos", "aos", "aos", "soa"])
        c["accept"] = rng.choice(["ge", "ge", "ge", "gt"])
        if c["precision"] == "f64" and c["nx"] * c["ny"] < 2e6 and rng.random() < 0.35:
            c["sweeps"], c["tol"] = 300, rng.choice([1e-6, 1e-8, 1e-9])
        else:
            c["sweeps"] = round(_log(rng, 10, 100)) if c["form"] == "jacobi" else round(_log(rng, 10, 60))
    elif kind == "handle":
        c["nx"], c["ny"] = _shape(rng, 500, 4e6)
        c["form"] = rng.choice(["jacobi", "jacobi", "jacobi", "colored"])
        c["sweeps"] = round(_log(rng, 1, 64))
    elif kind == "handles":
        c["nx"], c["ny"] = 24, rng.randint(120, 450)
        c["count"], c["sweeps"], c["refine"] = rng.randint(4, 60), rng.randint(4, 40), 0.0
    elif kind == "adjacency":
        c["nx"], c["ny"] = _shape(rng, 1000, 4e6)
        c["sweeps"] = 0
    else:
        c["count"], c["sweeps"], c["refine"] = rng.randint(1, 40), round(_log(rng, 10, 100)), 0.0
        c["nx"], c["ny"] = 24, rng.randint(120, 450)
    return c


# ------------------------------------------------------------------ meshes --

def _grid_tris(nx, ny, diag, periodic, gen):
    """CCW triangles, two per cell, node (i, j) with id j * nx + i."""
    ncx, ncy = nx - 1, ny if periodic else ny - 1
    j = torch.arange(ncy, device=DEV)[:, None]
    i = torch.arange(ncx, device=DEV)[None, :]
    jn = (j + 1) % ny
    a, b, c, d = j * nx + i, j * nx + i + 1, jn * nx + i + 1, jn * nx + i
    if diag == "unionjack":
        slash = (i + j) % 2 == 0
    else:
        slash = torch.rand((ncy, ncx), device=DEV, generator=gen) < 0.5
    slash = slash[..., None]
    t1 = torch.where(slash, torch.stack([a, b, c], -1), torch.stack([a, b, d], -1))
    t2 = torch.where(slash, torch.stack([a, c, d], -1), torch.stack([b, c, d], -1))
    return torch.stack([t1, t2], 2).reshape(-1, 3)


def _points(case, nx, ny, gen):
    """Jittered positions and the mask of the nodes on a boundary."""
    J = case["jitter"]
    i = torch.arange(nx, device=DEV).repeat(ny)
    j = torch.arange(ny, device=DEV).repeat_interleave(nx)
    jit = (torch.rand((nx * ny, 2), device=DEV, dtype=torch.float64, generator=gen) * 2 - 1) * J
    if case["mesh"] == "annulus":
        edge = (i == 0) | (i == nx - 1)
        jit[edge] = 0
        r = 0.3 + 0.7 * (i + jit[:, 0]) / (nx - 1)
        th = 2 * math.pi * (j + jit[:, 1]) / ny
        return torch.stack([r * torch.cos(th), r * torch.sin(th)], 1), edge
    edge = (i == 0) | (i == nx - 1) | (j == 0) | (j == ny - 1)
    jit[edge] = 0
    h = 1.0 / (max(nx, ny) - 1)
    return torch.stack([(i + jit[:, 0]) * h, (j + jit[:, 1]) * h], 1), edge


def _adjacency(n, tris):
    """Node->neighbour rows (in order of first appearance, triangle by
    triangle) and node->triangle rows (ascending) of a triangle list."""
    inc = torch.sort(tris.reshape(-1), stable=True)
    node, slot = inc.values, inc.indices
    t, k = slot // 3, slot % 3
    tri_ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    tri_ptr[1:] = torch.cumsum(torch.bincount(node, minlength=n), 0)
    v = tris[t]
    u0 = torch.where(k == 0, v[:, 1], v[:, 0])
    u1 = torch.where(k == 2, v[:, 1], v[:, 2])
    key = (node[:, None] * n + torch.stack([u0, u1], 1)).reshape(-1)
    del v, u0, u1, k
    s = torch.sort(key, stable=True)
    first = torch.ones_like(s.values, dtype=torch.bool)
    first[1:] = s.values[1:] != s.values[:-1]
    keep = key[torch.sort(s.indices[first]).values]
    nbr_ptr = torch.zeros(n + 1, dtype=torch.int64, device=DEV)
    nbr_ptr[1:] = torch.cumsum(torch.bincount(keep // n, minlength=n), 0)
    return nbr_ptr.int(), (keep % n).int(), tri_ptr.int(), t.int()


def _mesh(case, nx, ny, seed, rows=True):
    """Device tensors of one mesh; without `rows` the points and triangles only."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    tris = _grid_tris(nx, ny, case["diag"], case["mesh"] == "annulus", gen)
    pts, edge = _points(case, nx, ny, gen)
    if case["refine"] > 0:
        # the chosen triangles are split in three at an inner point
        order = torch.randperm(tris.shape[0], device=DEV, generator=gen)
        k = round(case["refine"] * tris.shape[0])
        old, rest = tris[order[:k]], tris[torch.sort(order[k:]).values]
        w = torch.rand((old.shape[0], 3), device=DEV, dtype=torch.float64, generator=gen) + 0.5
        w = w / w.sum(1, keepdim=True)
        new = (pts[old] * w[:, :, None]).sum(1)
        m = torch.arange(old.shape[0], device=DEV) + pts.shape[0]
        a, b, c = old[:, 0], old[:, 1], old[:, 2]
        tris = torch.cat([rest, torch.stack([a, b, m], 1), torch.stack([b, c, m], 1), torch.stack([c, a, m], 1)])
        pts = torch.cat([pts, new])
        edge = torch.cat([edge, torch.zeros(new.shape[0], dtype=torch.bool, device=DEV)])
    n = pts.shape[0]
    if case["shuffled"]:
        to = torch.randperm(n, device=DEV, generator=gen)
        p, e = torch.empty_like(pts), torch.empty_like(edge)
        p[to], e[to] = pts, edge
        pts, edge = p, e
        tris = to[tris[torch.randperm(tris.shape[0], device=DEV, generator=gen)]]
    m = types.SimpleNamespace(coords=pts.contiguous(), tris=tris.int().contiguous(), boundary=edge.to(torch.uint8), n=n)
    if rows:
        m.nbr_ptr, m.nbr_idx, m.tri_ptr, m.tri_idx = _adjacency(n, tris)
    return m


def _sides(case):
    """Grid sides of a batch, spread over their logarithm (the same for every seed)."""
    r = random.Random(case["count"] * 1000 + case["ny"])
    return [round(_log(r, case["nx"], case["ny"])) for _ in range(case["count"])]


def _meshes(case, seed):
    return [_mesh(case, n, n, seed * 101 + i) for i, n in enumerate(_sides(case))]


def _tensors(m):
    return (m.coords, m.nbr_ptr, m.nbr_idx, m.tri_ptr, m.tri_idx, m.tris.reshape(-1), m.boundary)


def _opts(case):
    return dict(form=case["form"], precision=case["precision"], layout=case["layout"], accept=case["accept"])


# -------------------------------------------------------------- the passes --

def prepare(case, seed):
    kind = case["kind"]
    if kind == "adjacency":
        m = _mesh(case, case["nx"], case["ny"], seed, rows=False)
        return dict(case=case, tris=m.tris, n=m.n)
    if kind == "handles":
        ms = _meshes(case, seed)
        hs = [sl.Mesh.from_device(_tensors(m), **_opts(case)) for m in ms]
        return dict(case=case, handles=hs, out=[torch.empty_like(m.coords) for m in ms])
    if kind == "host":
        f = ("coords", "nbr_ptr", "nbr_idx", "tri_ptr", "tri_idx", "tris", "boundary")
        return dict(case=case, meshes=[types.SimpleNamespace(**{k: getattr(m, k).cpu().numpy() for k in f})
                                       for m in _meshes(case, seed)])
    m = _mesh(case, case["nx"], case["ny"], seed)
    if kind == "handle":
        return dict(case=case, handle=sl.Mesh.from_device(_tensors(m), **_opts(case)), out=torch.empty_like(m.coords))
    return dict(case=case, mesh=_tensors(m))


def run(state):
    case = state["case"]
    kind, k, tol = case["kind"], case["sweeps"], case["tol"]
    if kind == "device":
        # the call smooths in place; the caller keeps its input positions
        x = state["mesh"][0].clone()
        rep = sl.smooth_mesh_device(x, *state["mesh"][1:], iterations=k, tol=tol, **_opts(case))
        return {"coords": x, "sweeps": rep.iterations_run, "accepted": rep.accepted_total}
    if kind == "handle":
        state["handle"].smooth_async(k)
        state["handle"].download_device(state["out"])
        return {"coords": state["out"]}
    if kind == "handles":
        sl.smooth_batch_async(state["handles"], k)
        for h, x in zip(state["handles"], state["out"]):
            h.download_device(x)
        return {"coords": state["out"]}
    if kind == "adjacency":
        return dict(zip(("nbr_ptr", "nbr_idx", "tri_ptr", "tri_idx", "boundary"),
                        sl.build_adjacency_device(state["tris"], state["n"])))
    ms = state["meshes"]
    if len(ms) == 1:
        m = ms[0]
        x, rep, _ = sl.smooth_mesh(m.coords, m.nbr_ptr, m.nbr_idx, m.tri_ptr, m.tri_idx, m.tris, m.boundary, k, tol,
                                   **_opts(case))
        return {"coords": [x], "sweeps": np.array([rep.iterations_run])}
    xs, reps, _ = sl.batch_smooth(ms, k, tol, **_opts(case))
    return {"coords": xs, "sweeps": np.array([r.iterations_run for r in reps])}


def _counts(case, nx, ny):
    """Nodes and triangles of a mesh."""
    t = 2 * (nx - 1) * (ny if case["mesh"] == "annulus" else ny - 1)
    split = round(case["refine"] * t)
    return nx * ny + split, t + 2 * split


def work(case):
    """Inputs read once, outputs written once; per node and sweep one
    neighbour sum (12 adds, 2 divisions), 2 old qualities of 21 operations
    (one per triangle) and 6 candidate qualities of 20.  A run to a
    tolerance takes about 80 sweeps."""
    kind = case["kind"]
    sizes = [(n, n) for n in _sides(case)] if kind in ("handles", "host") else [(case["nx"], case["ny"])]
    n = t = 0.0
    for nx, ny in sizes:
        a, b = _counts(case, nx, ny)
        n, t = n + a, t + b
    rows = 4 * (6 * n) + 4 * n + 4 * (3 * t) + 4 * n   # the two CSR arrays
    if kind == "adjacency":
        return {"bytes": 12 * t + rows + n, "flops": 0.0}
    sweeps = 80 if case["tol"] > 0 else case["sweeps"]
    flops = 176.0 * n * sweeps
    if kind in ("handle", "handles"):
        # the mesh is on the device already: positions read and written, the
        # connectivity (neighbour and triangle ids) read
        return {"bytes": 32 * n + 4 * (6 * n) + 12 * t, "flops": flops}
    return {"bytes": 16 * n + rows + 12 * t + n + 16 * n, "flops": flops}


# ------------------------------------------------- the same in plain torch --

def _padded(ptr, width):
    """Indices into a CSR array, one row of `width` per node, and their mask."""
    ptr = ptr.long()
    k = torch.arange(width, device=DEV)[None, :]
    deg = ptr[1:] - ptr[:-1]
    ok = k < deg[:, None]
    return torch.where(ok, ptr[:-1, None] + k, torch.zeros_like(k)), ok


def _q(x0, y0, x1, y1, x2, y2):
    ax, ay, bx, by, cx, cy = x1 - x0, y1 - y0, x2 - x0, y2 - y0, x2 - x1, y2 - y1
    cr = ax * by - bx * ay
    s = (ax * ax + ay * ay) + (cx * cx + cy * cy) + (bx * bx + by * by)
    return torch.where(s == 0, torch.zeros_like(s), (2 * math.sqrt(3.0) * cr) / s)


class _Plain:
    """The smoothing of one mesh as written in the paper, node by node."""

    def __init__(self, m, accept):
        self.gt = accept == "gt"
        self.x = m.coords.clone()
        deg, inc = (p[1:].long() - p[:-1].long() for p in (m.nbr_ptr, m.tri_ptr))
        at, self.nbr_ok = _padded(m.nbr_ptr, int(deg.max()))
        self.nbr = m.nbr_idx[at]
        at, self.tri_ok = _padded(m.tri_ptr, int(inc.max()))
        self.tri = m.tri_idx[at]
        self.tris, self.deg = m.tris.reshape(-1, 3), deg.double()
        self.free = torch.nonzero(m.boundary == 0).reshape(-1)

    def decide(self, nodes):
        """The next positions of `nodes`, from self.x."""
        out = torch.empty((nodes.numel(), 2), dtype=torch.float64, device=DEV)
        for b in range(0, nodes.numel(), 1 << 21):
            i = nodes[b:b + (1 << 21)]
            s = torch.zeros((i.numel(), 2), dtype=torch.float64, device=DEV)
            for k in range(self.nbr.shape[1]):
                s = torch.where(self.nbr_ok[i, k, None], s + self.x[self.nbr[i, k].long()], s)
            c, o = s / self.deg[i, None], self.x[i]
            old = torch.full((i.numel(),), math.inf, dtype=torch.float64, device=DEV)
            new = old.clone()
            for k in range(self.tri.shape[1]):
                v, ok = self.tris[self.tri[i, k].long()].long(), self.tri_ok[i, k]
                p = self.x[v]
                here = (v == i[:, None])[:, :, None]
                for pos, kind in ((p, 0), (torch.where(here, c[:, None, :], p), 1)):
                    q = _q(*(pos[:, j, a] for j in range(3) for a in range(2)))
                    q = torch.where(ok, q, torch.full_like(q, math.inf))
                    if kind:
                        new = torch.minimum(new, q)
                    else:
                        old = torch.minimum(old, q)
            yes = new > old if self.gt else new >= old
            out[b:b + (1 << 21)] = torch.where(yes[:, None], c, o)
        return out

    def smooth(self, sweeps, tol, classes=None):
        for _ in range(sweeps):
            before = self.x.clone() if tol > 0 else None
            for nodes in classes if classes is not None else [self.free]:
                self.x[nodes] = self.decide(nodes)
            if tol > 0 and float((self.x - before).square().sum(1).max()) < tol * tol:
                break
        return self.x

    def classes(self):
        """Greedy colouring of the free nodes in decreasing SplitMix64
        priority of the node id; the classes in increasing colour."""
        n = self.x.shape[0]

        def wrap(v):
            return v - (1 << 64) if v >= 1 << 63 else v

        def shr(z, b):
            return (z >> b) & ((1 << (64 - b)) - 1)

        z = torch.arange(n, device=DEV) + wrap(0x9E3779B97F4A7C15)
        z = (z ^ shr(z, 30)) * wrap(0xBF58476D1CE4E5B9)
        z = (z ^ shr(z, 27)) * wrap(0x94D049BB133111EB)
        z = (z ^ shr(z, 31)) ^ wrap(1 << 63)      # unsigned order as signed order
        color = torch.full((n,), -1, dtype=torch.int64, device=DEV)
        is_free = torch.zeros(n, dtype=torch.bool, device=DEV)
        is_free[self.free] = True
        left = self.free
        while left.numel():
            j = self.nbr[left].long()
            above = self.nbr_ok[left] & is_free[j] & (z[j] > z[left, None])
            ready = ~(above & (color[j] < 0)).any(1)
            used = torch.zeros((left.numel(), 1), dtype=torch.int64, device=DEV)
            bits = torch.where(above & (color[j] >= 0), 1 << color[j].clamp(min=0), torch.zeros_like(j))
            for k in range(bits.shape[1]):
                used = used | bits[:, k:k + 1]
            c = torch.zeros(left.numel(), dtype=torch.int64, device=DEV)
            for b in range(62, -1, -1):
                c = torch.where(shr(used[:, 0], b) & 1 == 0, torch.full_like(c, b), c)
            color[left[ready]] = c[ready]
            left = left[~ready]
        return [torch.nonzero(color == c).reshape(-1) for c in range(int(color.max()) + 1)]


def exact(case, seed):
    if case["kind"] == "adjacency":
        return None
    ms = _meshes(case, seed) if case["kind"] in ("handles", "host") else [_mesh(case, case["nx"], case["ny"], seed)]
    xs = []
    for m in ms:
        p = _Plain(m, case["accept"])
        xs.append(p.smooth(case["sweeps"], case["tol"], p.classes() if case["form"] == "colored" else None))
    if case["kind"] == "device":
        return {"coords": xs[0], "sweeps": None, "accepted": None}
    if case["kind"] == "handle":
        return {"coords": xs[0]}
    if case["kind"] == "handles":
        return {"coords": xs}
    return {"coords": [x.cpu().numpy() for x in xs], "sweeps": None}
