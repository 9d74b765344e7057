"""The one-launch path of small and medium meshes (tiles resident on the
device for all sweeps) against the oracle: at the edges of its tile sizes, the
meshes it hands on to the other kernels, and several calls at once.

Every operation is the oracle's, in its order, so equality is exact."""
import threading

import numpy as np
import pytest

import meshgen
import oracle
import paper_1502_00355_amd as sl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    torch.cuda.set_device(0)
    sl.lib()
    yield


def check(m, iters, tol=0.0, form="jacobi", accept="ge", **opts):
    import torch
    print("flow %s n=%d iters=%d tol=%g %s %s %s" % (m.name, m.n_nodes, iters, tol, form, accept, opts), flush=True)
    dev = sl.to_device(m, "cuda:0")
    nb = (m.n_nodes + 7) // 8
    flags = torch.zeros(iters * nb, dtype=torch.uint8, device="cuda:0")
    rep = sl.smooth_mesh_device(*dev, iterations=iters, tol=tol, flags=flags, form=form, accept=accept, **opts)
    ref = oracle.smooth(m, iters, tol=tol, accept_gt=accept == "gt", threads=oracle.max_threads(), form=form)
    k = ref.iterations_run
    assert rep.iterations_run == k
    assert (dev[0].cpu().numpy() == ref.coords).all()
    F = sl.unpack_flags(flags.cpu().numpy().reshape(iters, nb), m.n_nodes)
    assert (F[:k] == (ref.flags == 1)).all() and (F[k:] == 0).all()
    assert rep.accepted_total == int(ref.accepted.sum()) and rep.accepted_last == int(ref.accepted[-1])
    assert rep.max_disp_sq_last == ref.disp[-1]
    return rep


def grid(nx, ny, seed=1):
    """A jittered nx x ny grid (make_grid's meshes are square)."""
    m = meshgen.make_annulus(nx, ny, diag="random", jitter=0.3, seed=seed)
    m.name = "annulus%dx%d" % (nx, ny)
    return m


@pytest.mark.parametrize("form", ["jacobi", "colored"])
@pytest.mark.parametrize("nx,ny", [(3, 3), (3, 64), (3, 65), (10, 8), (10, 9), (66, 63), (128, 128), (129, 127),
                                   (130, 128), (128, 256), (129, 256), (257, 256), (256, 257), (500, 512), (502, 512)])
def test_tile_edges(nx, ny, form):
    """One free ring up to the largest mesh, full and ragged last tiles, each
    change of the tile size, and the first size beyond the path."""
    m = grid(nx, ny)
    sweeps = 12 if m.n_nodes < 40000 else 5
    rep = check(m, sweeps, form=form)
    if form == "jacobi":
        assert rep.kernel_used == sl.KERNELS["tile"]
    check(m, 3, form=form, accept="gt", layout="soa")


@pytest.mark.parametrize("form", ["jacobi", "colored"])
@pytest.mark.parametrize("tol,iters", [(1e-3, 40), (1e-9, 200), (1e-30, 1), (1e-30, 2), (1e-30, 7), (10.0, 5)])
def test_tolerance_stops(form, tol, iters):
    """Stops at the first sweep, inside a run and at the cap (the tiles run
    ahead of the decision by up to three sweeps)."""
    check(meshgen.make_delaunay(3000, 11), iters, tol=tol, form=form)
    check(meshgen.permute_mesh(meshgen.make_grid(90, "random", 0.4, 3), 5), iters, tol=tol, form=form)


def test_single_free_node_and_separate_parts():
    check(meshgen.star_mesh((0.1, 0.2), [(1, 0), (0, 1), (-1, 0), (0, -1)]), 6)
    check(meshgen.star_mesh((0.1, 0.2), [(1, 0), (0, 1), (-1, 0), (0, -1)]), 6, form="colored")
    # two meshes that share no node: tiles without anything to exchange
    a, b = meshgen.make_grid(12, "random", 0.3, 1), meshgen.make_grid(33, "random", 0.3, 2)
    tris = np.concatenate([a.tris, b.tris + a.n_nodes]).astype(np.int32)
    adj = meshgen.build_adjacency(a.n_nodes + b.n_nodes, tris)
    m = meshgen.Mesh(np.concatenate([a.coords, b.coords + 5.0]), tris, *adj, name="two parts")
    check(m, 20)
    check(m, 20, tol=1e-9, form="colored")


def hub_mesh(valence, seed=3):
    """A grid with, beside it, a free node of the given valence."""
    g = meshgen.make_grid(40, "random", 0.3, seed)
    th = 2 * np.pi * np.arange(valence) / valence
    s = meshgen.star_mesh((3.0, 0.1), np.stack([3 + np.cos(th), np.sin(th)], 1))
    tris = np.concatenate([g.tris, s.tris + g.n_nodes]).astype(np.int32)
    adj = meshgen.build_adjacency(g.n_nodes + s.n_nodes, tris)
    return meshgen.Mesh(np.concatenate([g.coords, s.coords]), tris, *adj, name="hub%d" % valence)


@pytest.mark.parametrize("form", ["jacobi", "colored"])
@pytest.mark.parametrize("valence", [17, 100, 127])
def test_long_rows(valence, form):
    """Rows longer than a read group, up to the valence limit (a tile with
    too many halo nodes goes to the other kernels)."""
    check(hub_mesh(valence), 6, form=form)


def test_rows_that_are_not_symmetric():
    """Form A takes them (on the other kernels); Form B refuses them."""
    m = meshgen.make_grid(50, "random", 0.3, 4)
    free = np.flatnonzero(m.boundary == 0)
    i, j = int(free[3]), int(free[-3])
    e = int(m.nbr_ptr[i + 1])
    m.nbr_idx = np.insert(m.nbr_idx, e, j).astype(np.int32)
    m.nbr_ptr = m.nbr_ptr.copy()
    m.nbr_ptr[i + 1:] += 1
    check(m, 8)
    check(m, 50, tol=1e-6)
    with pytest.raises(sl.SmartlapError):
        check(m, 8, form="colored")


def with_entries(m, pairs):
    """m with further entries (i, j) at the end of node i's row."""
    m = m.copy()
    for i, j in pairs:
        m.nbr_idx = np.insert(m.nbr_idx, int(m.nbr_ptr[i + 1]), j).astype(np.int32)
        m.nbr_ptr = m.nbr_ptr.copy()
        m.nbr_ptr[i + 1:] += 1
    return m


@pytest.mark.parametrize("size", [12, 90, 300, 600])
def test_neighbours_of_no_triangle(size):
    """Entries that no triangle explains: taken by Form B when both nodes
    list each other, or when the other is fixed; refused when one does not."""
    m = meshgen.make_grid(size, "random", 0.2, 5)
    free = np.flatnonzero(m.boundary == 0)
    i, j, f = int(free[2]), int(free[-2]), int(np.flatnonzero(m.boundary)[-1])
    check(with_entries(m, [(i, j), (j, i), (i, f)]), 2, form="colored")
    for pair in [(i, j), (j, i)]:
        with pytest.raises(sl.SmartlapError, match="not symmetric"):
            sl.smooth_mesh_device(*sl.to_device(with_entries(m, [pair]), "cuda:0"), iterations=2, form="colored")


def test_calls_at_once():
    """More calls at once, each on its own stream, than the device holds
    tiles for: some run on the other kernels, all give the same results."""
    import torch
    meshes = [grid(100 + 7 * k, 150 + 3 * k, seed=k) for k in range(6)]
    want = [oracle.smooth(m, 60, threads=oracle.max_threads()).coords for m in meshes]
    bad = []

    def work(k):
        torch.cuda.set_device(0)
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            for _ in range(4):
                dev = sl.to_device(meshes[k], "cuda:0")
                sl.smooth_mesh_device(*dev, iterations=60, stream=st)
                if not (dev[0].cpu().numpy() == want[k]).all():
                    bad.append(k)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(len(meshes))]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    assert not bad


def handle_check(m, calls, accept="ge", **opts):
    """A handle smoothed by several calls (sweeps, tolerance), against the
    oracle continued the same way."""
    h = sl.Mesh(m, accept=accept, **opts)
    X = m.copy()
    total = acc = 0
    for iters, tol in calls:
        print("handle %s n=%d iters=%d tol=%g %s" % (m.name, m.n_nodes, iters, tol, accept), flush=True)
        h.smooth_async(iters, tol)
        ref = oracle.smooth(X, iters, tol=tol, accept_gt=accept == "gt", threads=oracle.max_threads())
        X.coords = ref.coords
        total += ref.iterations_run
        acc += int(ref.accepted.sum())
        got, rep = h.download()
        assert (got == ref.coords).all()
        assert rep.iterations_run == total and rep.accepted_total == acc
        if ref.iterations_run:
            assert rep.accepted_last == int(ref.accepted[-1]) and rep.max_disp_sq_last == ref.disp[-1]
    assert rep.kernel_used == sl.KERNELS["tile"]
    h.close()


@pytest.mark.parametrize("nx,ny", [(3, 3), (10, 8), (10, 12), (66, 63), (130, 128), (129, 256), (257, 256), (500, 512),
                                   (502, 512)])
def test_handles(nx, ny):
    """Runs that follow each other (the exchange goes on where it was), with
    and without a tolerance, of one sweep (not on this path), of few tiles and
    sweeps (one work-group makes them) and beyond the path's size."""
    m = grid(nx, ny)
    long = 40 if m.n_nodes < 40000 else 9
    handle_check(m, [(2, 0.0), (3, 0.0), (1, 0.0), (4, 0.0), (long, 1e-9), (2, 1e-30), (5, 0.0), (2, 0.0), (0, 0.0)])
    handle_check(m, [(2, 1e-30), (2, 10.0), (7, 0.0)], accept="gt")


def test_handles_at_once():
    """More handles at work at once than the device holds tiles for; each
    gets its result, and the places pass from one to the next."""
    import torch
    ms = [grid(120 + 9 * k, 170, seed=k) for k in range(7)]
    hs = [sl.Mesh(m) for m in ms]
    sts = [torch.cuda.Stream() for _ in ms]
    for _ in range(3):
        for h, st in zip(hs, sts):
            h.smooth_async(12, stream=st)
    for h, m in zip(hs, ms):
        assert (h.download()[0] == oracle.smooth(m, 36, threads=oracle.max_threads()).coords).all()
    for h in hs:
        h.close()
