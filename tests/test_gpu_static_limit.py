"""The largest systems that the sweep without allocation takes: their norms fill the scratch, and the
partials of one workgroup per CU are what is left room for."""
import pytest
import torch

import paper_2003_09956_amd as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,n,m", [("f64", 2, 4150000), ("f64", 2, 4180000), ("f64", 64, 4165000),
                                       ("f32", 60, 4175000), ("bf16", 250, 4120000)])
def test_largest_systems_are_taken(dtype, n, m):
    vec, store = {"f64": (2, torch.float64), "f32": (4, torch.float32), "bf16": (8, torch.bfloat16)}[dtype]
    lda = -(-n // vec) * vec
    g = torch.Generator(device="cuda").manual_seed(n)
    A = torch.zeros((m, lda), device="cuda", dtype=store)
    A[:, :n] = torch.randn((m, n), generator=g, device="cuda", dtype=torch.float32).to(store)
    b = torch.rand(m, generator=g, device="cuda", dtype=torch.float64)
    x = torch.randn(n, generator=g, device="cuda", dtype=torch.float32).to(torch.float64)
    y = torch.empty(n, device="cuda", dtype=torch.float64)
    r = torch.empty(m, device="cuda", dtype=torch.float64)
    print(dtype, n, m, flush=True)
    P.eval_sweep_static(A, b, x, y, dtype=dtype, r=r, lda=lda)
    want_y = torch.zeros(n, device="cuda", dtype=torch.float64)
    scale = torch.zeros(n, device="cuda", dtype=torch.float64)
    tol = 1e-12 if dtype == "f64" else 1e-5
    for c in range(0, m, 1 << 18):
        a = A[c:c + (1 << 18), :n].to(torch.float64)
        t = a.abs() @ x.abs() + b[c:c + (1 << 18)]
        rr = a @ x - b[c:c + (1 << 18)]
        assert bool(((r[c:c + (1 << 18)] - rr).abs() <= tol * t).all())
        nu = a.square().sum(1)
        want_y += torch.where(rr > 0, rr / nu, 0.0) @ a
        scale += torch.where(rr > -tol * t, t / nu, 0.0) @ a.abs()
    assert bool(((y - want_y).abs() <= tol * scale).all())


def test_one_row_past_the_scratch_is_refused():
    m = (32 << 20) // 8
    A = torch.ones((m, 2), device="cuda", dtype=torch.float64)
    v = torch.ones(m, device="cuda", dtype=torch.float64)
    y = torch.zeros(2, device="cuda", dtype=torch.float64)
    with pytest.raises(P.ModapError, match="E_INVAL"):
        P.eval_sweep_static(A, v, torch.ones(2, device="cuda", dtype=torch.float64), y, dtype="f64")
    assert bool((y == 0).all())
