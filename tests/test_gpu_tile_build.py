"""The builds of the sweeps' tiles at their edges: rows and fans up to, at and
beyond the entries a work-item holds in registers, up to the valence limit,
last tiles of one node and full ones, vertices of every stored position.

Every operation is the oracle's, in its order, so equality is exact."""
import numpy as np
import pytest

import meshgen
import oracle
import paper_1502_00355_amd as sl

pytestmark = pytest.mark.gpu


def wheels(valence, size, seed):
    """A grid of size x size nodes and, beside it, a free node of the given
    valence within two rings of which the inner one is free; nodes, triangles
    and the triangles' first vertices in arbitrary order."""
    g = meshgen.make_grid(size, "random", 0.3, seed)
    k, z = np.arange(valence), g.n_nodes
    th = 2 * np.pi * k / valence
    ring = np.stack([np.cos(th), np.sin(th)], 1)
    nxt = (k + 1) % valence
    hub = np.stack([np.full(valence, z), z + 1 + k, z + 1 + nxt], 1)
    inner = np.stack([z + 1 + k, z + 1 + valence + k, z + 1 + valence + nxt], 1)
    outer = np.stack([z + 1 + k, z + 1 + valence + nxt, z + 1 + nxt], 1)
    xy = np.concatenate([g.coords, [[3.1, 0.05]], [3.0, 0.0] + 0.5 * ring, [3.0, 0.0] + ring])
    rng = np.random.default_rng(seed)
    order = rng.permutation(len(xy))
    label = np.empty(len(xy), np.int64)
    label[order] = np.arange(len(xy))
    tris = label[np.concatenate([g.tris, hub, inner, outer])]
    tris = np.stack([np.roll(t, r) for t, r in zip(tris, rng.integers(0, 3, len(tris)))])
    tris = tris[rng.permutation(len(tris))].astype(np.int32)
    return meshgen.Mesh(xy[order], tris, *meshgen.build_adjacency(len(xy), tris), name="wheel%d" % valence)


@pytest.mark.parametrize("form", ["jacobi", "colored"])
@pytest.mark.parametrize("tile_nodes", [256, 512])
@pytest.mark.parametrize("valence,size", [(3, 3), (7, 18), (8, 24), (9, 34), (17, 40), (127, 48)])
def test_build_edges(valence, size, tile_nodes, form):
    m = wheels(valence, size, 10 * valence + size)
    dev = sl.to_device(m, "cuda:0")
    rep = sl.smooth_mesh_device(*dev, iterations=4, form=form, kernel="tile", tile_nodes=tile_nodes)
    ref = oracle.smooth(m, 4, threads=oracle.max_threads(), form=form)
    assert rep.kernel_used == 2 and rep.tile_nodes == tile_nodes
    assert (dev[0].cpu().numpy() == ref.coords).all()
    assert rep.accepted_total == int(ref.accepted.sum())


@pytest.mark.parametrize("nx,ny", [(18, 18), (18, 34), (34, 18), (27, 43), (3, 3)])
def test_last_tiles(nx, ny):
    """Free nodes a multiple of the tile, one more, one tile not full."""
    m = meshgen.make_annulus(nx, ny, diag="random", jitter=0.3, seed=nx + ny)
    for tile_nodes in (256, 512):
        dev = sl.to_device(m, "cuda:0")
        rep = sl.smooth_mesh_device(*dev, iterations=5, kernel="tile", tile_nodes=tile_nodes)
        ref = oracle.smooth(m, 5, threads=oracle.max_threads())
        assert rep.kernel_used == 2 and (dev[0].cpu().numpy() == ref.coords).all()
