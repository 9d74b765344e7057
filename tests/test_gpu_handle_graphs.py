"""A handle's calls captured into a caller's graph, replayed between eager
calls.  A graph keeps the buffers it was captured with; with even numbers of
sweeps in every call they stay the right ones.

Every operation is the oracle's, in its order, so equality is exact."""
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


def positions(h, st):
    import torch
    x = torch.empty((h.n_nodes, 2), dtype=torch.float64, device="cuda:0")
    h.download_device(x, stream=st)
    st.synchronize()
    return x.cpu().numpy()


@pytest.mark.parametrize("with_download", [False, True])
@pytest.mark.parametrize("size", [20, 110, 300])
def test_replays_between_eager_calls(size, with_download):
    import torch
    m = meshgen.make_grid(size, "random", 0.35, 7)
    st = torch.cuda.Stream()
    h = sl.Mesh(m)
    out = torch.zeros((m.n_nodes, 2), dtype=torch.float64, device="cuda:0")
    print("capture size=%d download=%s" % (size, with_download), flush=True)
    h.smooth_async(10, stream=st)
    st.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        h.smooth_async(6, stream=st)
        if with_download:
            h.download_device(out, stream=st)
    total = 10
    for eager in (0, 10, 4, 2):
        if eager:
            h.smooth_async(eager, stream=st)
            total += eager
        for _ in range(2):
            with torch.cuda.stream(st):
                g.replay()
            total += 6
            st.synchronize()
            want = oracle.smooth(m, total, threads=oracle.max_threads()).coords
            if with_download:
                assert (out.cpu().numpy() == want).all()
            assert (positions(h, st) == want).all()
    h.close()


@pytest.mark.parametrize("size", [20, 110])
def test_captured_download_follows_eager_sweeps(size):
    import torch
    m = meshgen.make_grid(size, "random", 0.35, 8)
    st = torch.cuda.Stream()
    h = sl.Mesh(m)
    out = torch.zeros((m.n_nodes, 2), dtype=torch.float64, device="cuda:0")
    h.smooth_async(4, stream=st)
    st.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        h.download_device(out, stream=st)
    for more, k in ((0, 4), (10, 14), (2, 16), (30, 46)):
        if more:
            h.smooth_async(more, stream=st)
        with torch.cuda.stream(st):
            g.replay()
        st.synchronize()
        assert (out.cpu().numpy() == oracle.smooth(m, k, threads=oracle.max_threads()).coords).all()
    h.close()


def test_other_handles_run_beside_a_capture():
    """Two handles whose tiles do not fit the device together: while one's
    call is being captured, the other takes the room that the first one's
    earlier, finished call had, and the capture stays whole."""
    import torch
    m = meshgen.make_grid(470, "random", 0.35, 9)
    st, st2 = torch.cuda.Stream(), torch.cuda.Stream()
    h, h2 = sl.Mesh(m), sl.Mesh(m)
    h.smooth_async(4, stream=st)
    st.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st, capture_error_mode="relaxed"):
        h.smooth_async(6, stream=st)
        h2.smooth_async(8, stream=st2)
    with torch.cuda.stream(st):
        g.replay()
    st.synchronize()
    st2.synchronize()
    assert (positions(h, st) == oracle.smooth(m, 10, threads=oracle.max_threads()).coords).all()
    assert (h2.download()[0] == oracle.smooth(m, 8, threads=oracle.max_threads()).coords).all()
    h.close()
    h2.close()
