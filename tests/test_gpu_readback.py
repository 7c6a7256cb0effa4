"""Results read back by the host: staged through mapped memory by one workgroup
or many, or copied when they are large; host and device outputs the same bits."""
import numpy as np
import pytest

import paper_2003_09956_amd as P
import workloads as W

pytestmark = pytest.mark.gpu


# (m, n): x and b together below, at and above the one-workgroup limit of 4096
# doubles, and above the staging limit of 2^20
@pytest.mark.parametrize("m,n", [(1, 1), (3, 2), (4000, 95), (4000, 96), (4000, 97), (40000, 8), (1 << 20, 2)])
def test_query_and_eval_host_equal_device(m, n):
    import torch
    rng = np.random.default_rng(m + n)
    A = rng.standard_normal((m, n))
    b = rng.standard_normal(m)
    x0 = rng.standard_normal(n)
    with P.Solver(0) as s:
        s.set_system(A, b, x0, dtype="f64")
        for _ in range(2):      # the staging memory is there the second time
            x, bb, st = s.query(want_b=True)
            assert np.array_equal(x, x0) and np.array_equal(bb, b) and st.iters == 0
            host = s.eval_sweep(x0)
            dev = s.eval_sweep(torch.from_numpy(x0).cuda())
            assert np.array_equal(host.y, dev.y.cpu().numpy()) and np.array_equal(host.r, dev.r.cpu().numpy())
            assert (host.h, host.max_viol) == (dev.h, dev.max_viol)
            t = np.abs(A) @ np.abs(x0) + np.abs(b)
            assert np.all(np.abs(host.r - (A @ x0 - b)) <= 1e-12 * t)
    with P.Batch("f64") as q:
        i = q.add(A, b, x0)
        for _ in range(2):
            x, bb, _ = q.query(i, want_b=True)
            assert np.array_equal(x, x0) and np.array_equal(bb, b)


@pytest.mark.parametrize("reload", [False, True])
def test_solves_in_a_row_stop_where_the_first_did(reload):
    """The word that tells the host how far a solve has come is fresh in every solve: the same
    solve from the same start, in one context and after another system, takes the same steps."""
    big = W.gaussian(60, 400, seed=1, dtype="f32")
    one = W.gaussian(1200, 2000, seed=2, dtype="f32")
    x0 = one.z + 0.02 * np.random.default_rng(0).standard_normal(one.n)
    prm = P.params(lam=0.01, eps=1e-4, max_iters=400)
    with P.Solver(0) as s:
        got = []
        s.set_system(one.A, one.b, x0, dtype="f32")
        for _ in range(3):
            if reload:
                s.set_system(big.A, big.b, dtype="f32")
                s.solve(prm, raise_on_stop=False)
                s.set_system(one.A, one.b, x0, dtype="f32")
            s.set_x(x0)
            st, code = s.solve(prm)
            got.append((st.iters, st.sweeps, s.query()[0].tobytes()))
        assert got[0] == got[1] == got[2] and got[0][0] > 0
    with P.Batch("f32") as q:
        ids = [q.add(one.A, one.b, x0), q.add(big.A, big.b)]
        out = q.solve(prm)
        st = q.query(ids[0])[2]
        assert out.running == 0 and st.state == 1 and st.certified == 1
        out = q.solve(prm)      # every system stands: one check each
        assert out.running == 0 and q.query(ids[0])[2].iters == st.iters
