"""Inputs in pinned host memory are the caller's again when a call returns, also behind iterations
still queued (a copy from pinned memory is made only when the stream comes to it)."""
import numpy as np
import pytest
import torch

import paper_2003_09956_amd as P
import workloads as W

pytestmark = pytest.mark.gpu
N, M = 4100, 8192


def host(a, pinned):
    """A copy of `a`, in pinned or in pageable memory."""
    t = torch.empty(a.shape, dtype=getattr(torch, a.dtype.name), pin_memory=pinned).numpy()
    t[...] = a
    return t


@pytest.mark.parametrize("pinned", [False, True])
@pytest.mark.parametrize("what", ["x", "rows", "new_b", "translate"])
def test_context_inputs_may_be_reused_at_once(what, pinned):
    w = W.gaussian(N, M, seed=3, dtype="f32")
    prm = P.params(lam=0.02, eps=1e-9, track=True)
    rng = np.random.default_rng(5)
    rows = np.arange(0, M, 50, dtype=np.int64)
    new = rng.standard_normal((len(rows), N)).astype(np.float32)
    v = 1e-2 * rng.standard_normal(N)
    ends = []
    for reuse in (False, True):
        with P.Solver(0) as s:
            s.set_system(w.A, w.b, x0=w.z + 0.3, dtype="f32")
            s.iterate(1000, prm, stats=False)       # tens of milliseconds
            if what == "x":
                a = host(w.z + 0.2, pinned)
                s.set_x(a)
            elif what == "translate":
                a = host(v, pinned)
                s.update_coeffs(translate=a)
            else:
                A2, b2 = host(new, pinned), host(new.astype(np.float64) @ w.z + 0.5, pinned)
                s.update_coeffs(rows=rows, new_rows=A2, new_b=b2)
                a = A2 if what == "rows" else b2
            if reuse:
                a[...] = 1.0
            s.iterate(20, prm, stats=False)
            x, b, q = s.query(want_b=True)
            ends.append((x, b, q.iters))
    assert np.array_equal(ends[0][0], ends[1][0]) and np.array_equal(ends[0][1], ends[1][1])
    assert ends[0][2] == ends[1][2]


@pytest.mark.parametrize("pinned", [False, True])
def test_batch_schedule_may_be_reused_at_once(pinned):
    w = [W.gaussian(900 + 10 * k, 6000, seed=k, dtype="f32") for k in range(16)]
    prm = P.params(lam=0.02, eps=1e-9, track=True)
    want = W.drift(900, 200, sigma=1e-3, seed=7)
    ends = []
    for reuse in (False, True):
        with P.Batch("f32") as B:
            ids = [B.add(s.A, s.b, x0=s.z + 0.3) for s in w]
            B.iterate(1000, prm, stats=False)
            V = host(want, pinned)
            B.set_drift(ids[0], V)
            if reuse:
                V[...] = 1.0
            B.iterate(200, prm)
            x, b, q = B.query(ids[0], want_b=True)
            ends.append((x, b, q.iters))
    assert np.array_equal(ends[0][0], ends[1][0]) and np.array_equal(ends[0][1], ends[1][1])
    assert ends[0][2] == ends[1][2]
