"""The node kernels at the edges of their row lengths (one work-item per node
up to 8 entries, then 2, 4 and 8), and Form B's folds, which wait from class
to class for the sweep's last launch.

Every operation is the oracle's, in its order, so equality is exact."""
import numpy as np
import pytest

import meshgen
import oracle
import paper_1502_00355_amd as sl
from test_gpu_tile_build import wheels

pytestmark = pytest.mark.gpu


def check(m, iters, form, tol=0.0, **opts):
    import torch
    dev = sl.to_device(m, "cuda:0")
    nb = (m.n_nodes + 7) // 8
    flags = torch.zeros(iters * nb, dtype=torch.uint8, device="cuda:0")
    rep = sl.smooth_mesh_device(*dev, iterations=iters, tol=tol, flags=flags, form=form, kernel="node", **opts)
    ref = oracle.smooth(m, iters, tol=tol, threads=oracle.max_threads(), form=form)
    k = ref.iterations_run
    assert rep.iterations_run == k and rep.kernel_used == 1
    assert (dev[0].cpu().numpy() == ref.coords).all()
    F = sl.unpack_flags(flags.cpu().numpy().reshape(iters, nb), m.n_nodes)
    assert (F[:k] == (ref.flags == 1)).all() and (F[k:] == 0).all()
    assert rep.accepted_total == int(ref.accepted.sum()) and rep.accepted_last == int(ref.accepted[-1])
    assert rep.max_disp_sq_last == ref.disp[-1]


@pytest.mark.parametrize("layout", ["aos", "soa"])
@pytest.mark.parametrize("form", ["jacobi", "colored"])
@pytest.mark.parametrize("valence,size", [(8, 3), (8, 60), (9, 60), (16, 33), (17, 60), (32, 40), (33, 60), (127, 24)])
def test_row_lengths(valence, size, form, layout):
    check(wheels(valence, size, valence + size), 6, form, layout=layout)


@pytest.mark.parametrize("form", ["jacobi", "colored"])
def test_to_convergence(form):
    check(wheels(9, 20, 5), 400, form, tol=1e-4)


@pytest.mark.parametrize("block_size", [64, 128, 256])
def test_folds_over_classes(block_size):
    """Classes of many work-groups and of few, sweep after sweep."""
    m = meshgen.make_grid(300, "random", 0.3, 8)
    check(m, 5, "colored", block_size=block_size)


def test_arbitrary_numbering():
    """More nodes than are coloured at the same time, neighbours far apart."""
    g = meshgen.make_grid(900, "random", 0.3, 9)
    rng = np.random.default_rng(9)
    order = rng.permutation(g.n_nodes)
    label = np.empty(g.n_nodes, np.int64)
    label[order] = np.arange(g.n_nodes)
    tris = label[g.tris][rng.permutation(len(g.tris))].astype(np.int32)
    m = meshgen.Mesh(g.coords[order], tris, *meshgen.build_adjacency(g.n_nodes, tris), name="shuffled900")
    check(m, 2, "colored")
