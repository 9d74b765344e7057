"""Meshes most of whose nodes are fixed (a local smooth in a large mesh), and
meshes whose nodes crowd into few cells of the node order: results against the
oracle, and the setup's time, which must not queue on a few counters."""
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


def setup_ms(m, form):
    out = []
    for _ in range(7):
        dev = sl.to_device(m, "cuda:0")
        rep = sl.smooth_mesh_device(*dev, iterations=2, form=form)
        out.append(rep.setup_ms)
    ref = oracle.smooth(m, 2, threads=oracle.max_threads(), form=form)
    assert (dev[0].cpu().numpy() == ref.coords).all()
    return float(np.median(out))


@pytest.mark.parametrize("form", ["jacobi", "colored"])
@pytest.mark.parametrize("shuffled", [False, True])
@pytest.mark.parametrize("free", [20, 60, 300])
def test_mostly_fixed(free, shuffled, form):
    """free x free nodes of 1100 x 1100 may move."""
    size = 1100
    m = meshgen.make_grid(size, "random", 0.3, 5)
    if shuffled:
        m = meshgen.permute_mesh(m, 2)
    whole = setup_ms(m, form)
    k = np.argsort(np.abs(m.coords - 0.5).max(axis=1))[: free * free]
    m.boundary = np.ones_like(m.boundary)
    m.boundary[k] = 0
    local = setup_ms(m, form)
    print("%s free %d shuffled %s: setup %.3f ms, of the whole mesh %.3f ms" % (form, free * free, shuffled, local, whole),
          flush=True)
    assert local < 1.25 * whole


@pytest.mark.parametrize("form", ["jacobi", "colored"])
def test_crowded_cells(form):
    m = meshgen.make_grid(600, "random", 0.3, 6)
    plain = setup_ms(m, form)
    m.coords = m.coords ** 6
    crowded = setup_ms(m, form)
    print("%s: setup %.3f ms, crowded %.3f ms" % (form, plain, crowded), flush=True)
    assert crowded < 3 * plain
