"""The numbers that tell the words of one resident iteration from another's: a captured launch that
is replayed uses the same ones again, and 32 bits of them come round."""
import numpy as np
import pytest
import torch

import paper_2003_09956_amd as P
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,n,m", [("f64", 64, 250), ("f64", 128, 600), ("f32", 256, 1024)])
@pytest.mark.parametrize("k", [1, 2, 3, 6])
def test_replayed_launches_follow_eager_ones(dtype, n, m, k):
    """(up to eight workgroups, more, and more with the sums in two trips)"""
    w = W.gaussian(n, m, seed=n + k, dtype=dtype)
    V = W.drift(n, 100, sigma=1e-3, seed=k)
    prm = P.params(lam=0.02, eps=1e-9, track=True)
    side = torch.cuda.Stream()
    with P.Solver(0) as eager, P.Solver(0, stream=side.cuda_stream) as s:
        for c in (eager, s):
            c.set_system(w.A, w.b, x0=w.z + 0.3, dtype=dtype)
            c.set_drift(V)
        assert eager.iterate(k, prm).resident == 1
        s.iterate(k, prm)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            s.iterate(k, prm, stats=False)
        for i in range(7):
            print(dtype, n, m, k, "pass", i, flush=True)
            if i % 3 == 2:      # the program's own work between the replays
                s.iterate(k, prm)
                torch.cuda.synchronize()
            else:
                with torch.cuda.stream(side):
                    graph.replay()
            e = eager.iterate(k, prm)
            (x0, b0, _), (x1, b1, q) = eager.query(want_b=True), s.query(want_b=True)
            assert np.array_equal(x0, x1) and np.array_equal(b0, b1)
            assert (q.iters, q.sweeps, q.h, q.max_viol) == (e.iters, e.sweeps, e.h, e.max_viol)


def test_numbers_come_round():
    """A launch of 2^20 iterations uses up as many numbers however soon it stops: after 4096 of them
    words of the first launch would carry the numbers that the next one looks for."""
    n, m, K = 64, 300, 1 << 20
    w = W.gaussian(n, m, seed=1, dtype="f64")
    b = w.A @ w.z + 1.0
    prm = P.params(lam=0.5, eps=1e-9, certify=False)
    near, far = w.z + 1.2 * w.A[0], w.z + np.random.default_rng(3).normal(scale=4.0, size=n)
    ends = []
    with P.Solver(0) as s:
        s.set_system(w.A, b, x0=near, dtype="f64")
        q = s.iterate(K, prm)
        assert q.resident == 1 and (q.iters, q.sweeps) == (1, 2)     # words numbered 1 and 2
        for i in range(4095):                                       # one check each
            s.iterate(K, prm, stats=False)
        for _ in range(2):
            s.set_x(far)
            q = s.iterate(K, prm)
            ends.append((s.query()[0], q.iters, q.sweeps, q.max_viol))
    assert ends[0][1] > 5
    assert np.array_equal(ends[0][0], ends[1][0]) and ends[0][1:] == ends[1][1:]
