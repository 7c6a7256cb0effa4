"""What comes in from device memory: drift schedules (copied, padded and checked by one kernel into
a buffer that is kept) and server requests (whose matrix is handed over, not copied again) give
the same bits as the same data from host memory; what is not finite is refused and leaves no
schedule behind."""
import numpy as np
import pytest
import torch

import paper_2003_09956_amd as P
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,n", [("f64", 255), ("f32", 257), ("f32", 1001), ("f64", 9001)])
def test_device_schedules_match_host_ones(dtype, n):
    sys_ = W.gaussian(n, 300, seed=n, dtype=dtype)
    prm = P.params(lam=0.02, track=True)
    out = []
    for dev in (False, True):
        with P.Solver(0) as s:
            s.set_system(sys_.A, sys_.b, x0=sys_.z + 0.1, dtype=dtype)
            for T in (1, 7, 300, 2, 65, 66, 0, 3):   # grown, shrunk, kept, given back
                V = W.drift(n, max(T, 1), sigma=1e-3, seed=T)[:T]
                print(dtype, n, dev, T, flush=True)
                s.set_drift((torch.from_numpy(V).cuda() if dev else V) if T else None)
                s.iterate(2, prm)                     # a row of the schedule is still due
            x, b, q = s.query(want_b=True)
            out += [x, b, np.array([q.iters, q.h, q.max_viol])]
    for a, c in zip(out[:3], out[3:]):
        assert np.array_equal(a, c)


def test_a_bad_device_schedule_leaves_none():
    sys_ = W.gaussian(300, 500, seed=2, dtype="f32")
    prm = P.params(lam=0.02, track=True)
    with P.Solver(0) as s:
        s.set_system(sys_.A, sys_.b, x0=sys_.z + 0.1, dtype="f32")
        for at in ((0, 0), (4, 299), (2, 150)):
            V = W.drift(300, 5, sigma=1e-3, seed=3)
            s.set_drift(torch.from_numpy(V).cuda())
            V[at] = np.inf
            with pytest.raises(P.ModapError):
                s.set_drift(torch.from_numpy(V).cuda())
            b = s.query(want_b=True)[1]
            s.iterate(3, prm)
            assert np.array_equal(s.query(want_b=True)[1], b)
        V[at] = 0.0
        s.set_drift(torch.from_numpy(V).cuda())
        s.iterate(3, prm)
        assert not np.array_equal(s.query(want_b=True)[1], b)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_device_requests_match_host_ones(dtype):
    """Rows of a whole number of 16-byte vectors and ragged ones, batched and in contexts of their
    own (two at once, one after the other: the stream is kept), with and without x0 and drift."""
    shapes = [(64, 300), (333, 900), (1001, 1500), (4999, 400), (5002, 400), (2500, 300)]
    prm = P.params(lam=0.3, eps=1e-3)
    res = []
    for dev in (False, True):
        put = (lambda a: torch.from_numpy(a).cuda()) if dev else (lambda a: a)
        with P.Server(dtype, prm=prm, iters_per_round=4) as s:
            tickets = []
            for k, (n, m) in enumerate(shapes):
                w = W.gaussian(n, m, seed=n, dtype=dtype)
                x0 = put(w.z + 0.2) if k % 2 == 0 else None
                V = put(W.drift(n, 3, sigma=1e-3, seed=k)) if k % 3 == 0 else None
                tickets.append(s.submit(put(w.A), put(w.b), x0=x0, V=V))
            for r in range(400):
                if s.round(float(r)) == 0:
                    break
            print(dtype, dev, r, flush=True)
            res.append([(s.result(t), s.info(t)) for t in tickets])
    for (xa, ia), (xb, ib) in zip(*res):
        assert np.array_equal(xa, xb)
        assert all(ia[k] == ib[k] for k in ("status", "iters", "sweeps", "max_viol"))
