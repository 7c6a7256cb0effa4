"""The one-read sweep of long rows translates b in place while the workgroups of its other column
tiles use it: iterations under drift with nine and sixteen tiles (workgroups of one band on the
same XCD), bands of 63 to 194 rows, against the two-phase form.  The working b itself is seen
through the next sweep's r and through what a certificate finds it off by."""
import numpy as np
import pytest
import torch

import paper_2003_09956_amd as P

pytestmark = pytest.mark.gpu
SPLIT = {"f64": (256, 256, 8), "f32": (256, 256, 8), "bf16": (256, 256, 4)}
TORCH = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
UNIT = {"f64": 2.0 ** -53, "f32": 2.0 ** -24, "bf16": 2.0 ** -24}    # of the dot products
STEPS, SIGMA = 40, 1e-2

# 28 bands of nine tiles, 16 of sixteen
CASES = [("f64", 33000, 28 * 130 + 3), ("f64", 62001, 16 * 65), ("f32", 66000, 28 * 64), ("f32", 128001, 16 * 63),
         ("bf16", 66001, 28 * 63 - 5), ("bf16", 130000, 16 * 193 + 1)]


@pytest.mark.parametrize("dtype,n,m", CASES)
def test_working_b_under_drift(dtype, n, m):
    g = torch.Generator(device="cuda").manual_seed(n + m)
    A = torch.randn((m, n), generator=g, device="cuda", dtype=torch.float32)
    A = (A / torch.linalg.vector_norm(A, dim=1, keepdim=True)).to(TORCH[dtype]).contiguous()
    z = torch.rand(n, generator=g, device="cuda", dtype=torch.float64)
    b = torch.cat([c.to(torch.float64) @ z for c in A.split(256)])
    b += torch.rand(m, generator=g, device="cuda", dtype=torch.float64)
    x0 = z + torch.randn(n, generator=g, device="cuda", dtype=torch.float64)
    V = SIGMA * torch.randn((STEPS, n), generator=g, device="cuda", dtype=torch.float64)
    prm = P.params(lam=0.05, eps=1e-9, track=True)
    loose = P.params(lam=0.05, eps=1e3, eps_relative=False, max_iters=5)
    got = {}
    for form in ("relay", "two phases"):
        print(dtype, n, m, form, flush=True)
        with P.Solver(0) as s:
            s.set_system(A, b, x0=x0, dtype=dtype)
            assert s.get_tile()["kind"] == 1
            if form != "relay":
                s.set_tile(*SPLIT[dtype], 0, 1, kind=1)
            s.set_drift(V)
            xs = []
            for k in (1, 2, STEPS - 3):
                st = s.iterate(k, prm)
                xs.append(s.query()[0])
            e = s.eval_sweep(xs[-1])
            q, code = s.solve(loose)      # stops at its first check; the certificate rebases b
            assert code == 0 and q.certified == 1
            got[form] = (xs, e.r, (st.iters, st.sweeps), q.b_drift)
        torch.cuda.empty_cache()
    (xr, rr, cr, dr), (xt, rt, ct, dt) = got["relay"], got["two phases"]
    assert cr == ct == (STEPS, STEPS)
    tol = 1e-11 if dtype == "f64" else 1e-5
    for u, v in zip(xr, xt):
        assert np.linalg.norm(u - v) <= tol * np.linalg.norm(v)
    # The working b took STEPS translations of <a_i, v>, at most ||v|| each and rounded in chains of
    # less than 64 terms, and an FP64 addition each; one missed or repeated is about SIGMA.
    slack = STEPS * (64 * UNIT[dtype] * SIGMA * np.sqrt(n) * 1.1 + 2.0 ** -52 * float(b.abs().max() + 1.0))
    print(f"b off by {dr:.2e} and {dt:.2e}, allowed {slack:.2e}", flush=True)
    assert slack < SIGMA / 10 and dr <= slack and dt <= slack
    # and r at points that differ by tol ||x|| at most, rows of length one
    assert np.abs(rr - rt).max() <= 2 * slack + 3 * tol * np.linalg.norm(xt[-1])
