"""How far the sums of a sweep are rounded: the dot products of every shape against what chains of
two 16-byte vectors a lane, added in pairs, come to (a wavefront that takes a whole row alone
must not round more than a workgroup that shares it)."""
import numpy as np
import pytest
import torch

import paper_2003_09956_amd as P

pytestmark = pytest.mark.gpu
TORCH = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
VEC = {"f64": 2, "f32": 4, "bf16": 8}


def system(dtype, n, m):
    g = torch.Generator(device="cuda").manual_seed(n)
    A = torch.randn((m, n), generator=g, device="cuda", dtype=torch.float32)
    A = (A / torch.linalg.vector_norm(A, dim=1, keepdim=True)).to(TORCH[dtype]).contiguous()
    x = torch.randn(n, generator=g, device="cuda", dtype=torch.float32).to(torch.float64)
    return A, x, torch.zeros(m, device="cuda", dtype=torch.float64)


def rms(e):
    return float(np.sqrt(np.mean(np.square(np.asarray(e, dtype=np.float64)))))


@pytest.mark.parametrize("dtype,n", [("bf16", 1500), ("bf16", 3000), ("bf16", 4096), ("bf16", 6000), ("bf16", 16384),
                                     ("f32", 1000), ("f32", 1500), ("f32", 2000), ("f32", 8192), ("f32", 16384),
                                     ("f64", 1000), ("f64", 1500)])
def test_dot_products_round_in_short_chains(dtype, n):
    m = 1500
    A, x, b = system(dtype, n, m)
    with P.Solver(0) as s:
        s.set_system(A, b, dtype=dtype)
        r = s.eval_sweep(x.cpu().numpy()).r
    acc, wide = (np.float64, np.longdouble) if dtype == "f64" else (np.float32, np.float64)
    a, xs = A.to(torch.float64).cpu().numpy().astype(wide), x.cpu().numpy().astype(wide)
    prod = a * xs
    exact = prod.sum(axis=1)
    # the model: fused multiply-adds along a chain, then sums of neighbours
    L = 2 * VEC[dtype]
    k = -(-n // L)
    p = np.zeros((m, k * L), dtype=wide)
    p[:, :n] = prod
    p = p.reshape(m, k, L)
    c = np.zeros((m, k), dtype=acc)
    for i in range(L):
        c = (c.astype(wide) + p[:, :, i]).astype(acc)
    while c.shape[1] > 1:
        if c.shape[1] % 2:
            c = np.concatenate([c, np.zeros((m, 1), dtype=acc)], axis=1)
        c = c[:, 0::2] + c[:, 1::2]
    got, model = rms(r - exact), rms(c[:, 0].astype(wide) - exact)
    print(f"{dtype} {n}: {got:.3e}, model {model:.3e}", flush=True)
    # 1500 rows: 2% of statistical error; the lanes and wavefronts of a row are added in pairs and fours
    assert got <= 1.15 * model


@pytest.mark.parametrize("dtype,n,m", [("f32", 20000, 2097), ("f32", 40000, 6000), ("bf16", 40000, 2097),
                                       ("bf16", 24000, 16384), ("f64", 9000, 8000)])
def test_the_one_read_sweep_rounds_no_more_than_the_two_phases(dtype, n, m):
    """Half as many bands of rows as the two phases have: r and y against 64 bits (FP64 storage: y of
    64 columns against 80 bits), in both forms."""
    split = {"f64": (256, 256, 8), "f32": (256, 256, 8), "bf16": (256, 256, 4)}[dtype]
    A, x, b = system(dtype, n, m)
    if dtype == "f64":
        cols = slice(0, 64)
        a = A.cpu().numpy()
        xs = x.cpu().numpy().astype(np.longdouble)
        exact = np.concatenate([(c.astype(np.longdouble) * xs).sum(axis=1) for c in np.array_split(a, 50)])
        nu = np.concatenate([np.square(c.astype(np.longdouble)).sum(axis=1) for c in np.array_split(a, 50)])
        y = np.where(exact > 0, exact / nu, 0) @ a[:, cols].astype(np.longdouble)
        limit = 1.5      # 64 columns: 9% of statistical error a side
    else:
        cols = slice(0, n)
        ex = torch.cat([c.to(torch.float64) @ x for c in A.split(512)])
        nu = torch.cat([c.to(torch.float64).square().sum(1) for c in A.split(512)])
        w = torch.where(ex > 0, ex / nu, 0.0)
        y = sum(p @ c.to(torch.float64) for p, c in zip(w.split(512), A.split(512))).cpu().numpy()
        exact = ex.cpu().numpy()
        limit = 1.05
    err = {}
    for form in ("one read", "two phases"):
        with P.Solver(0) as s:
            s.set_system(A, b, dtype=dtype)
            assert s.get_tile()["kind"] == 1
            if form != "one read":
                s.set_tile(*split, 0, 1, kind=1)
            e = s.eval_sweep(x.cpu().numpy())
        err[form] = rms(e.r - exact), rms(e.y[cols] - y)
    print(dtype, n, m, err, flush=True)
    (r1, y1), (r2, y2) = err["one read"], err["two phases"]
    assert r1 <= 1.05 * r2 and y1 <= limit * y2
