"""Device adjacency at the sizes where its binning changes: one bin, a last
bin of one node, several nodes per work-item, and nodes in more triangles than
the registers hold -- against the plain builder of the generators (index for
index: the results are whole numbers)."""
import numpy as np
import pytest

import meshgen
import paper_1502_00355_amd as sl

pytestmark = pytest.mark.gpu


def fan(k, extra=0):
    """A hub in k triangles around it (hub id 0), plus `extra` unused nodes."""
    t = np.array([[0, 1 + q, 1 + (q + 1) % k] for q in range(k)], np.int32)
    return k + 1 + extra, t


def shuffled_grid(nx, ny, seed):
    m = meshgen.permute_mesh(meshgen.make_annulus(nx, ny, seed=seed), seed)
    return m.n_nodes, m.tris


CASES = [fan(3), fan(8), fan(9), fan(16), fan(17), fan(200), fan(63 - 1), fan(64 - 1), fan(64), fan(5, extra=300),
         shuffled_grid(5, 7, 1), shuffled_grid(181, 181, 2), shuffled_grid(256, 128, 3), shuffled_grid(257, 128, 4),
         shuffled_grid(700, 511, 5)]


@pytest.mark.parametrize("n,tris", CASES, ids=["%d-%d" % (n, len(t)) for n, t in CASES])
def test_equals_the_plain_builder(n, tris):
    import torch
    torch.cuda.set_device(0)
    print("adjacency n=%d tris=%d" % (n, len(tris)), flush=True)
    want = meshgen.build_adjacency(n, tris)
    got = sl.build_adjacency(n, tris)
    dev = sl.build_adjacency_device(torch.from_numpy(np.ascontiguousarray(tris, dtype=np.int32)).cuda(), n)
    for w, g, d in zip(want, got, dev):
        assert (g == w).all() and (d.cpu().numpy() == w).all()
