"""Adjacency of nodes that are in no triangle: no triangle array at all (a
null pointer), and isolated nodes beside a mesh."""
import numpy as np
import pytest

import meshgen
import paper_1502_00355_amd as sl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    torch.cuda.set_device(0)
    sl.lib()
    yield


@pytest.mark.parametrize("n", [1, 5, 257, 70000])
def test_no_triangles(n):
    import torch
    print("adjacency of %d nodes, no triangles" % n, flush=True)
    tris = torch.empty((0, 3), dtype=torch.int32, device="cuda:0")
    got = [x.cpu().numpy() for x in sl.build_adjacency_device(tris, n)]
    host = sl.build_adjacency(n, np.empty((0, 3), np.int32))
    for nbr_ptr, nbr_idx, tri_ptr, tri_idx, boundary in (got, host):
        assert nbr_ptr.shape == tri_ptr.shape == (n + 1,) and not nbr_ptr.any() and not tri_ptr.any()
        assert nbr_idx.size == tri_idx.size == 0 and (boundary == 1).all()


def test_isolated_nodes():
    import torch
    m = meshgen.make_grid(20, "random", 0.3, 1)
    tris = torch.from_numpy(np.ascontiguousarray(m.tris)).to("cuda:0")
    want = meshgen.build_adjacency(m.n_nodes + 300, m.tris)
    for g, w in zip(sl.build_adjacency_device(tris, m.n_nodes + 300), want):
        assert (g.cpu().numpy() == w).all()
