"""Tile sweeps without a tolerance, which the run's last sweep closes
together: run lengths around the graph's chunks, few and many work-groups,
one call after another.

Every operation is the oracle's, in its order, so equality is exact."""
import pytest

import meshgen
import oracle
import paper_1502_00355_amd as sl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size,iters", [(5, 1), (5, 2), (5, 3), (60, 31), (60, 63), (60, 64), (60, 65), (60, 68),
                                        (60, 100), (200, 36), (200, 68), (450, 7)])
def test_run_lengths(size, iters):
    """Displacement and counts of the last sweep, and the total over all."""
    m = meshgen.make_grid(size, "random", 0.35, size + iters)
    ref = oracle.smooth(m, iters, threads=oracle.max_threads())
    for tile_nodes in (256, 512):
        dev = sl.to_device(m, "cuda:0")
        rep = sl.smooth_mesh_device(*dev, iterations=iters, kernel="tile", tile_nodes=tile_nodes)
        assert rep.iterations_run == iters and rep.kernel_used == sl.KERNELS["tile"]
        assert (dev[0].cpu().numpy() == ref.coords).all()
        assert rep.accepted_total == int(ref.accepted.sum()) and rep.accepted_last == int(ref.accepted[-1])
        assert rep.max_disp_sq_last == ref.disp[-1]


def test_handle_calls():
    """A handle's calls of few sweeps (closed together) and of a chunk and
    more, from either buffer."""
    m = meshgen.make_grid(140, "random", 0.35, 3)
    h = sl.Mesh(m, kernel="tile", tile_nodes=256)
    total = 0
    for calls in ([1], [2, 1], [5], [31], [32, 3], [33], [65, 7]):
        for k in calls:
            h.smooth_async(k)
            total += k
        x, rep = h.download()
        ref = oracle.smooth(m, total, threads=oracle.max_threads())
        assert (x == ref.coords).all() and rep.iterations_run == total
        assert rep.accepted_total == int(ref.accepted.sum()) and rep.accepted_last == int(ref.accepted[-1])
        assert rep.max_disp_sq_last == ref.disp[-1]
    h.close()
