"""One-call smooths, handles, a batch, a server and adjacencies on threads of
one process at once: every result as if alone, and nothing held up for long.

Every operation is the oracle's, in its order, so equality is exact."""
import threading
import time

import numpy as np
import pytest

import meshgen
import oracle
import paper_1502_00355_amd as sl

pytestmark = pytest.mark.gpu

SWEEPS = (3, 10, 25)
SECONDS = 6.0


def test_everything_at_once():
    import torch
    torch.cuda.set_device(0)
    ms = [meshgen.make_grid(s, "random", 0.35, s) for s in (12, 50, 120, 200, 300, 420, 480, 600)]
    want = {(i, f): [oracle.smooth(m, k, threads=oracle.max_threads(), form=f).coords for k in SWEEPS]
            for i, m in enumerate(ms) for f in ("jacobi", "colored")}
    bad, count, t0 = [], {}, time.time()

    def running():
        return time.time() - t0 < SECONDS

    def smooths(rng):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            devs = [sl.to_device(m, "cuda:0") for m in ms]
            start = [d[0].clone() for d in devs]
            while running():
                i, k, f = int(rng.integers(len(ms))), int(rng.integers(3)), ("jacobi", "colored")[int(rng.integers(2))]
                devs[i][0].copy_(start[i])
                sl.smooth_mesh_device(*devs[i], iterations=SWEEPS[k], form=f, stream=st)
                yield bool((devs[i][0].cpu().numpy() == want[i, f][k]).all())

    def handles(rng):
        sts = [torch.cuda.Stream() for _ in range(2)]
        while running():
            i = int(rng.integers(len(ms)))
            with sl.Mesh(ms[i]) as h:
                for a, b, k in ((3, 7, 1), (10, 5, 2)):
                    h.smooth_async(a, stream=sts[0])
                    h.smooth_async(b, stream=sts[1])
                    yield bool((h.download()[0] == want[i, "jacobi"][k]).all())

    def batch(rng):
        while running():
            outs = sl.batch_smooth(ms[:6], 10)[0]
            yield all((x == want[i, "jacobi"][1]).all() for i, x in enumerate(outs))

    def server(rng):
        with sl.Server() as s:
            while running():
                q = [(int(rng.integers(len(ms))), int(rng.integers(3))) for _ in range(12)]
                ids = [s.submit(ms[i], SWEEPS[k], 0.0) for i, k in q]
                for rid, (i, k) in zip(ids, q):
                    r = s.wait(rid)
                    yield r.status == sl.SL_OK and bool((r.coords == want[i, "jacobi"][k]).all())

    def adjacency(rng):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            tris = [torch.from_numpy(np.ascontiguousarray(m.tris.reshape(-1, 3))).to("cuda:0") for m in ms]
            while running():
                for t, m in zip(tris, ms):
                    yield bool((sl.build_adjacency_device(t, m.n_nodes, stream=st)[1].cpu().numpy() == m.nbr_idx).all())

    def work(name, gen):
        torch.cuda.set_device(0)
        try:
            for ok in gen:
                count[name] = count.get(name, 0) + 1
                if not ok:
                    bad.append(name + ": wrong result")
        except Exception as e:
            bad.append("%s: %s" % (name, e))

    sl.lib().sl_one_launch_wait(-1.0)
    ts = [threading.Thread(target=work, args=(f.__name__ + str(k), f(np.random.default_rng(k))))
          for k, f in enumerate([smooths, smooths, smooths, handles, handles, batch, server, adjacency])]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    print("in %.0f s: %s" % (SECONDS, count), flush=True)
    assert not bad, bad[:5]
    # 500 a second each; 65 to 150 when runs waited seconds for places on the device
    assert all(count["smooths%d" % k] > 100 * SECONDS for k in range(3))
