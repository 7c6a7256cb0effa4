"""The one-read sweep of rows too long for a workgroup: the workgroups of a row band pass their
partial dot products on while the rows wait in LDS.  Against the oracle at the edges of its
tiles (two to sixteen of them, even and ragged), bands and pipeline, against the two-phase
form over many steps, and both sides of the rule that chooses it."""
import numpy as np
import pytest

import oracle
import paper_2003_09956_amd as P
import workloads as W
from parity import check_sweep

pytestmark = pytest.mark.gpu
SPLIT = {"f64": (256, 256, 8), "f32": (256, 256, 8), "bf16": (256, 256, 4)}

# n at one element past the one-pass shapes, at whole tiles and one past them; m with one to a
# few rows a band (below, at and past the rows in registers and in LDS), even and ragged
CASES = [("f64", 8193, 2100), ("f64", 8192 + 4096, 1400), ("f64", 12289, 1369), ("f64", 9001, 2555),
         ("f64", 20000, 900), ("f64", 32768, 517), ("f64", 65537, 300), ("f32", 16385, 2100), ("f32", 24576, 1401),
         ("f32", 24577, 1400), ("f32", 50001, 701), ("bf16", 24576, 2800), ("bf16", 29000, 2400), ("bf16", 40000, 1801)]


@pytest.mark.parametrize("dtype,n,m", CASES)
def test_relay_sweep_matches_oracle(dtype, n, m):
    sys_ = W.gaussian(n, m, seed=n + m, dtype=dtype)
    rng = np.random.default_rng(n)
    v = rng.normal(scale=0.05, size=n)
    with P.Solver(0) as s:
        s.set_system(sys_.A, sys_.b, dtype=dtype)
        assert s.get_tile()["kind"] == 1
        for far in (0.002, 1.0):      # few rows violated, about half of them
            x = sys_.z + rng.normal(scale=far, size=n)
            print(dtype, n, m, far, flush=True)
            g = s.eval_sweep(x)
            again = s.eval_sweep(x, want_r=False)
            assert np.array_equal(g.y, again.y) and g.h == again.h
            o = oracle.sweep(sys_.A, dtype, sys_.b, x)
            check_sweep(sys_.A, dtype, o, g.y, g.h, g.max_viol, g.r, label=f"relay {dtype} {n}x{m} {far}")
        s.update_coeffs(translate=v)
        g = s.eval_sweep(x)
    o = oracle.sweep(sys_.A, dtype, oracle.translate(sys_.A, dtype, sys_.b, v), x)
    check_sweep(sys_.A, dtype, o, g.y, g.h, g.max_viol, g.r, label=f"relay moved {dtype} {n}x{m}")


@pytest.mark.parametrize("dtype,n,m", [("f64", 9000, 2000), ("f32", 18000, 2000), ("bf16", 24000, 3000)])
def test_relay_iterations_follow_the_two_phases(dtype, n, m):
    """Sixty steps under drift, in calls of one and of many, end where the two-phase form ends, to
    the rounding of the sums (1e-11 in FP64; FP32 dots of rows of length one: 1e-5)."""
    sys_ = W.gaussian(n, m, seed=5, dtype=dtype)
    V = W.drift(n, 60, sigma=1e-3, seed=6)
    x0 = sys_.z + np.random.default_rng(1).normal(scale=1.0, size=n)
    prm = P.params(lam=0.05, eps=1e-9, track=True)
    got = {}
    for form in ("relay", "two phases"):
        with P.Solver(0) as s:
            s.set_system(sys_.A, sys_.b, x0=x0, dtype=dtype)
            if form != "relay":
                blk, lpr, ch = SPLIT[dtype]
                s.set_tile(blk, lpr, ch, 0, 1, kind=1)
            s.set_drift(V)
            for k in (1, 1, 38, 20):
                st = s.iterate(k, prm)
            x, b, _ = s.query(want_b=True)
            got[form] = (x, b, st.iters, st.sweeps)
    (xr, br, ir, sr), (xt, bt, it, stt) = got["relay"], got["two phases"]
    assert (ir, sr) == (it, stt) == (60, 60)
    tol = 1e-11 if dtype == "f64" else 1e-5
    assert np.linalg.norm(xr - xt) <= tol * np.linalg.norm(xt)
    assert np.array_equal(br, bt)     # the exact data: the same translations, in FP64


def test_relay_rule_by_size():
    """Below 128 MiB the two phases, from there on the one read: the same sweep."""
    n = 8448      # 67584 bytes a row
    for m in (1985, 1986):
        sys_ = W.gaussian(n, m, seed=m, dtype="f64")
        x = sys_.z + 0.01
        with P.Solver(0) as s:
            s.set_system(sys_.A, sys_.b, dtype="f64")
            g = s.eval_sweep(x)
        o = oracle.sweep(sys_.A, "f64", sys_.b, x)
        check_sweep(sys_.A, "f64", o, g.y, g.h, g.max_viol, g.r, label=f"relay rule {m}")
