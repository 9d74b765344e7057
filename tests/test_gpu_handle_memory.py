"""Device memory of mesh handles, and what a call with a tolerance adds."""
import pytest

import meshgen
import paper_1502_00355_amd as sl

pytestmark = pytest.mark.gpu


def test_bytes_per_node():
    import torch
    torch.cuda.set_device(0)
    m = meshgen.make_grid(500, "random", 0.3, 1)
    count = 16

    def used():
        torch.cuda.synchronize()
        sl.release_cached_memory()
        free, total = torch.cuda.mem_get_info()
        return total - free

    sl.Mesh(m).close()   # (the pools' first allocations)
    base = used()
    hs = [sl.Mesh(m) for _ in range(count)]
    made = (used() - base) / (count * m.n_nodes)
    for h in hs:
        h.smooth_async(20)
    swept = (used() - base) / (count * m.n_nodes)
    for h in hs:
        h.smooth_async(20, 1e-30)
    tol = (used() - base) / (count * m.n_nodes)
    print("bytes a node: made %.0f, swept %.0f, with a tolerance %.0f" % (made, swept, tol), flush=True)
    assert made < 300 and swept < 300 and tol < 365
    for h in hs:
        h.close()
    assert used() - base < 64 << 20
