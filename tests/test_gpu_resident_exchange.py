"""The exchange between the workgroups of a resident launch at the edges of its forms: up to eight
workgroups and more, sums in one trip (rows of up to 128 columns, with workgroups that fill the
threads' shares and not) and in two (longer rows, with workgroups that own columns and not).
The first steps against the oracle, and many iterations in one launch against single calls."""
import numpy as np
import pytest

import oracle
import paper_2003_09956_amd as P
import workloads as W
from parity import TOL, weighted_abs_rows

pytestmark = pytest.mark.gpu
# 32 rows a workgroup: 1, 8, 9, 15, 16, 17, 25, 31 and 32 of them
SHAPES = [(64, 20), (64, 256), (65, 257), (128, 480), (120, 512), (128, 513), (100, 800), (127, 1024), (129, 256),
          (129, 257), (191, 480), (192, 990), (256, 1024), (300, 545), (511, 330)]


@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
def test_exchange_forms(dtype):
    lam = 0.05
    prm, trk = P.params(lam=lam, eps=1e-9), P.params(lam=lam, eps=1e-9, track=True)
    for n, m in SHAPES:
        print(dtype, n, m, flush=True)
        w = W.gaussian(n, m, seed=n + m, dtype=dtype)
        V = W.drift(n, 40, sigma=1e-3, seed=m)
        ends = []
        for calls in ([1] * 12, [12], [5, 7]):
            with P.Solver(0) as s:
                s.set_system(w.A, w.b, x0=w.z + 0.3, dtype=dtype)
                s.set_drift(V)
                x, b = w.z + 0.3, np.array(w.b, dtype=np.float64)
                for i, k in enumerate(calls):
                    q = s.iterate(k, trk)
                    assert q.resident == 1
                    if k == 1 and i < 2:
                        if i == 1:
                            b = oracle.translate(w.A, dtype, b, V[0])
                        o = oracle.sweep(w.A, dtype, b, x)
                        xo, status = oracle.step(o.y, o.h, 0, lam, x)
                        x1 = s.query()[0]
                        assert status == 0 and abs(q.h - o.h) <= (np.abs(o.r) <= TOL[dtype] * o.t).sum()
                        near = o.r > -TOL[dtype] * o.t
                        s_y = np.linalg.norm(weighted_abs_rows(w.A, dtype, np.where(near, o.t / o.nu, 0)))
                        bound = TOL[dtype] * (np.linalg.norm(x) + lam * s_y / np.linalg.norm(o.y))
                        assert np.linalg.norm(x1 - xo) <= bound, (n, m, i)
                        x = x1
                x1, b1, q = s.query(want_b=True)
                ends.append((x1, b1, q.iters, q.h, q.max_viol, q.y_norm))
        for e in ends[1:]:
            assert np.array_equal(e[0], ends[0][0]) and np.array_equal(e[1], ends[0][1]) and e[2:] == ends[0][2:]
