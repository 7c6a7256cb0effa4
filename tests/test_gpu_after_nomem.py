"""A request that no device memory can hold (8 TB, refused by the allocator at once) leaves nothing
behind: the next call on the same thread works, and so does PyTorch's."""
import ctypes as C

import numpy as np
import pytest
import torch

import paper_2003_09956_amd as P
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("torch_first", [False, True])
def test_context_goes_on_after_too_large_a_system(torch_first):
    w = W.gaussian(50, 200, seed=1, dtype="f64")
    v = torch.zeros(64, device="cuda", dtype=torch.float64)
    with P.Solver(0) as s:
        for _ in range(2):
            # the matrix is never read: its copy is the first thing asked for
            st = P.lib().modap_set_system(s._ctx, 1 << 20, 1 << 20, 0, C.c_void_p(v.data_ptr()), 1 << 20,
                                          C.c_void_p(v.data_ptr()), None, 1)
            assert P.STATUS_NAMES[st] == "E_NOMEM"
            if torch_first:
                assert float((v + 1.0).sum()) == 64.0
            s.set_system(w.A, w.b, dtype="f64")
            assert s.eval_sweep(w.z).h == 0


@pytest.mark.parametrize("torch_first", [False, True])
def test_batch_goes_on_after_too_large_a_system(torch_first):
    w = W.gaussian(50, 200, seed=1, dtype="f64")
    v = torch.zeros(1024, device="cuda", dtype=torch.float64)
    with P.Batch("f64") as b:
        for _ in range(2):
            sid = C.c_int64(-1)
            st = P.lib().modap_batch_add(b._h, 1 << 30, 1024, C.c_void_p(v.data_ptr()), 1024, C.c_void_p(v.data_ptr()),
                                         None, 1, C.byref(sid))
            assert P.STATUS_NAMES[st] == "E_NOMEM"
            if torch_first:
                assert float((v + 1.0).sum()) == 1024.0
            k = b.add(w.A, w.b, x0=w.z + 0.3)
            assert b.solve(P.params(lam=0.02, eps=1e-6)).running == 0
            x, _, q = b.query(k)
            assert q.state == 1 and np.isfinite(x).all()


def test_server_goes_on_after_too_large_a_request():
    w = W.gaussian(50, 200, seed=1, dtype="f64")
    v = torch.zeros(64, device="cuda", dtype=torch.float64)
    A, b = torch.from_numpy(w.A).cuda(), torch.from_numpy(w.b).cuda()
    with P.Server("f64", budget_bytes=1e14, prm=P.params(lam=0.02, eps=1e-6), iters_per_round=8) as s:
        for _ in range(2):
            t = C.c_int64(-1)
            st = P.lib().modap_server_submit(s._h, 1 << 20, 1 << 20, C.c_void_p(v.data_ptr()), C.c_void_p(v.data_ptr()),
                                             None, 0, None, 0, 1, 0.0, C.byref(t))
            assert P.STATUS_NAMES[st] == "E_NOMEM"
            assert float((v + 1.0).sum()) == 64.0
            k = s.submit(A, b)
            for r in range(500):
                if s.round(float(r)) == 0:
                    break
            assert s.info(k)["status"] == 1 and np.isfinite(s.result(k)).all()
