"""The one-read sweep of long rows when a workgroup gives up waiting for another's dot product
(forced from the host with a bound of zero clock ticks; every kernel still exits normally): the
call ends at once with E_DEVICE instead of going on with void data, and so does every other until
a system is set again."""
import time

import numpy as np
import pytest

import paper_2003_09956_amd as P
import workloads as W

pytestmark = pytest.mark.gpu


def test_relay_timeout_ends_the_call(monkeypatch):
    w = W.gaussian(9000, 2000, seed=3, dtype="f64")
    x0 = w.z + np.random.default_rng(2).normal(size=w.n)
    prm = P.params(lam=1e-6, eps=1e-12, max_iters=300000)   # steps too short to get anywhere: 20 s of sweeps
    with P.Solver(0) as s:
        s.set_system(w.A, w.b, x0=x0, dtype="f64")
        assert s.get_tile()["kind"] == 1
        monkeypatch.setenv("MODAP_RESIDENT_TIMEOUT_TICKS", "0")
        t0 = time.monotonic()
        with pytest.raises(P.ModapError, match="E_DEVICE"):
            s.solve(prm)
        took = time.monotonic() - t0
        print(f"solve ended after {took:.3f} s", flush=True)
        assert took < 3.0
        monkeypatch.delenv("MODAP_RESIDENT_TIMEOUT_TICKS")
        for call in (lambda: s.iterate(3, prm), lambda: s.eval_sweep(x0), lambda: s.solve(prm), s.query):
            t0 = time.monotonic()
            with pytest.raises(P.ModapError, match="E_DEVICE"):
                call()
            assert time.monotonic() - t0 < 3.0
        s.set_system(w.A, w.b, x0=x0, dtype="f64")
        assert s.iterate(5, prm).iters == 5
        assert s.solve(P.params(lam=0.05, eps=1e3, eps_relative=False))[0].certified == 1
