"""Scans of more values than their tiles add up in place (2^27): the offsets of
an adjacency and of a mesh of that size, and the time of the largest."""
import time

import pytest

import paper_1502_00355_amd as sl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    torch.cuda.set_device(0)
    sl.lib()
    yield
    torch.cuda.empty_cache()
    sl.release_cached_memory()


@pytest.mark.parametrize("n", [(1 << 27) - 3, (1 << 27) + 5, 300_000_001])
def test_adjacency_offsets(n):
    """Separate triangles at far ends of the numbering."""
    import torch
    print("adjacency of %d nodes" % n, flush=True)
    at = torch.tensor([0, 4093, 4096 * 100, n // 3, n // 2 + 1, n - 4], device="cuda:0")
    tris = (at[:, None] + torch.arange(3, device="cuda:0")[None]).to(torch.int32)
    nbr_ptr, nbr_idx, tri_ptr, tri_idx, boundary = sl.build_adjacency_device(tris.contiguous(), n)
    assert bool((boundary == 1).all()) and nbr_idx.numel() == 36 and tri_idx.numel() == 18
    nodes = tris.flatten().sort().values
    for ptr, each in ((nbr_ptr, 2), (tri_ptr, 1)):
        # the offset of node v: `each` per listed node below v
        steps = torch.nonzero(ptr[1:] != ptr[:-1]).flatten()
        assert bool((steps == nodes).all()) and int(ptr[0]) == 0 and int(ptr[-1]) == each * 18
        assert bool(((ptr[nodes.long() + 1] - ptr[nodes.long()]) == each).all())


def test_time_grows_with_the_size():
    """10^9 nodes take per node at most a third more than 130M (twice as long
    each when every tile added up all earlier ones: 0.047 ns against 0.033)."""
    import torch
    tri = torch.tensor([[0, 1, 2]], dtype=torch.int32, device="cuda:0")

    def ns(n):
        out = []
        for _ in range(5):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            sl.build_adjacency_device(tri, n)
            torch.cuda.synchronize()
            out.append(1e9 * (time.perf_counter() - t0) / n)
        return min(out)

    a, b = ns(130_000_000), ns(1_000_000_000)
    print("%.4f ns a node at 130M, %.4f at 10^9" % (a, b), flush=True)
    assert b < 1.33 * a


def grid(nx, ny):
    import torch
    j = torch.arange(ny - 1, device="cuda:0", dtype=torch.int32)[:, None]
    i = torch.arange(nx - 1, device="cuda:0", dtype=torch.int32)[None, :]
    a = j * nx + i
    return torch.stack([a, a + 1, a + nx + 1, a, a + nx + 1, a + nx], -1).reshape(-1, 3)


def test_mesh_offsets():
    """A grid of more than 2^27 free nodes: one sweep gives what it gives on
    each half (with a row of the other half, fixed there)."""
    import torch
    nx, ny = 11700, 11500
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    x = torch.empty((ny, nx, 2), dtype=torch.float64, device="cuda:0")
    x[..., 0] = torch.arange(nx, device="cuda:0", dtype=torch.float64)[None, :]
    x[..., 1] = torch.arange(ny, device="cuda:0", dtype=torch.float64)[:, None]
    x[1:-1, 1:-1] += 0.3 * (2 * torch.rand((ny - 2, nx - 2, 2), dtype=torch.float64, device="cuda:0", generator=gen) - 1)

    def sweep(y):
        rows = y.shape[0]
        y = y.clone().reshape(-1, 2)
        tris = grid(nx, rows)
        adj = sl.build_adjacency_device(tris, y.shape[0])
        rep = sl.smooth_mesh_device(y, *adj[:4], tris.reshape(-1), adj[4], iterations=1)
        return y.reshape(rows, nx, 2), rep

    half = ny // 2
    lower, r0 = sweep(x[: half + 1])
    upper, r1 = sweep(x[half - 1:])
    print("halves accepted %d, %d" % (r0.accepted_total, r1.accepted_total), flush=True)
    whole, r = sweep(x)
    assert r.accepted_total == r0.accepted_total + r1.accepted_total
    assert bool((whole[:half] == lower[:half]).all()) and bool((whole[half:] == upper[1:]).all())
    assert bool((whole != x).any())
