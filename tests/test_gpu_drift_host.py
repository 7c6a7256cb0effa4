"""A drift schedule in host memory is read during the call, also into a buffer that is kept from the
one before it and behind iterations still queued: the caller may reuse the memory at once."""
import numpy as np
import pytest
import torch

import paper_2003_09956_amd as P
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pinned", [False, True])
@pytest.mark.parametrize("n,T", [(4096, 300), (4097, 300), (4096, 2), (4099, 2)])
def test_host_schedule_may_be_reused_at_once(n, T, pinned):
    w = W.gaussian(n, 8192, seed=n, dtype="f32")
    prm = P.params(lam=0.02, eps=1e-9, track=True)
    want = W.drift(n, T, sigma=1e-3, seed=7)
    V = torch.zeros((T, n), dtype=torch.float64, pin_memory=pinned).numpy()
    ends = []
    for reuse in (False, True):
        with P.Solver(0) as s:
            s.set_system(w.A, w.b, x0=w.z + 0.3, dtype="f32")
            s.set_drift(W.drift(n, T, sigma=1e-3, seed=8))
            s.iterate(1000, prm, stats=False)       # tens of milliseconds
            V[:] = want
            s.set_drift(V)
            if reuse:
                V[:] = 1.0
            s.iterate(T, prm, stats=False)
            x, b, q = s.query(want_b=True)
            ends.append((x, b, q.iters))
    assert np.array_equal(ends[0][0], ends[1][0]) and np.array_equal(ends[0][1], ends[1][1])
    assert ends[0][2] == ends[1][2]


def test_schedules_are_refused_under_capture():
    """And the capture, the schedule before it and the context go on."""
    w = W.gaussian(600, 900, seed=1, dtype="f32")
    V = W.drift(600, 5, sigma=1e-3, seed=1)
    prm = P.params(lam=0.02, track=True)
    side = torch.cuda.Stream()
    with P.Solver(0, stream=side.cuda_stream) as s:
        s.set_system(w.A, w.b, x0=w.z + 0.3, dtype="f32")
        done = 0
        for what in (V, None, torch.from_numpy(V).cuda()):
            for before in (None, V):
                s.set_drift(before)
                graph = torch.cuda.CUDAGraph()
                torch.cuda.synchronize()
                with torch.cuda.graph(graph, stream=side):
                    with pytest.raises(P.ModapError, match="E_DEVICE"):
                        s.set_drift(what)
                    s.iterate(2, prm, stats=False)
                with torch.cuda.stream(side):
                    graph.replay()
                done += 2
                assert s.query()[2].sweeps == done
