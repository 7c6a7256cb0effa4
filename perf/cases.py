"""The work this library does for its users, as cases that can be timed.

A case is a dict of plain values; ``prepare`` builds what a program has in hand
before the call (inputs on the GPU, a loaded context or batch), ``run`` makes
one pass through the public entry points, ``exact`` gives the same results in
plain 64-bit torch, and ``work`` counts the bytes and operations a pass cannot
do without.  Systems are the two families the library is measured on: dense
Gaussian rows of unit length around a hidden feasible point (``gaussian``),
and the box-plus-sum polytope (``box``).

FP64 systems return r, y, the counts and the points as the library gives them.
FP32- and BF16-stored systems return the points the iteration reaches, handed on
in FP32, the precision of the dot products behind them.  Step lengths and
tolerances of the solves are such that a rounding error stays one: with a step
far longer than the violations left, the method's path is chaotic.
"""
import math

import numpy as np
import torch

import paper_2003_09956_amd as P

TORCH = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
BYTES = {"f64": 8, "f32": 4, "bf16": 2}
VEC = {"f64": 2, "f32": 4, "bf16": 8}          # elements of 16 bytes
DEV = "cuda:0"


def listed():
    return [
        # one check of a point on a small system: the shortest call a program makes
        {"name": "check_small_f64", "kind": "check", "dtype": "f64", "n": 50, "m": 200},
        # the entry point that allocates nothing (tight loops, graph capture), ragged rows
        {"name": "check_static_f64", "kind": "static", "dtype": "f64", "n": 777, "m": 3000},
        # the stationary box-plus-sum solve, 256 of its iterations, from a far start
        {"name": "box_f64_256", "kind": "box", "dtype": "f64", "n": 256, "m": 513, "iters": 256},
        # following a moving system, one call of queued iterations each: a middling ragged
        # system, and the three sizes the library is benchmarked on
        {"name": "follow_f32_1000", "kind": "follow", "dtype": "f32", "n": 1000, "m": 4000, "iters": 16},
        {"name": "follow_f32_8192", "kind": "follow", "dtype": "f32", "n": 8192, "m": 16384, "iters": 16},
        {"name": "follow_f64_4096", "kind": "follow", "dtype": "f64", "n": 4096, "m": 32768, "iters": 8},
        {"name": "follow_bf16_16384", "kind": "follow", "dtype": "bf16", "n": 16384, "m": 65536, "iters": 8},
        # the translation experiment: rows too long for one pass, half of them violated, the
        # polytope moved between chunks of four iterations
        {"name": "catchup_f64_32000", "kind": "catchup", "dtype": "f64", "n": 32000, "chunks": 2},
        # a controller's tick: 1% of the rows replaced, the system moved, solved again to a
        # certified stop, the point and the right-hand side read back
        {"name": "tick_bf16_4096", "kind": "tick", "dtype": "bf16", "n": 4096, "m": 16384},
        # a batch of equal small systems iterated together
        {"name": "batch_f32_256", "kind": "batch", "dtype": "f32", "count": 256, "n_lo": 256, "n_hi": 256,
         "m_mult": 8, "iters": 16},
        # a fleet of uneven systems, each moved and then all solved again to certified stops
        {"name": "fleet_f32_64", "kind": "fleet", "dtype": "f32", "count": 64, "n_lo": 64, "n_hi": 2048,
         "m_mult": 4},
        # requests served together: submitted, admitted, moved while live, solved, read, released
        {"name": "serve_bf16_8", "kind": "serve", "dtype": "bf16", "count": 8, "n_lo": 128, "n_hi": 8192,
         "m_mult": 4},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["check", "static", "box", "follow", "follow", "catchup", "tick", "batch", "fleet", "serve"])
    if kind in ("check", "static"):
        n = _log_int(rng, 16, 1500)
        return {"kind": kind, "dtype": "f64", "n": n, "m": rng.randint(2 * n, 6 * n)}
    if kind == "box":
        n = _log_int(rng, 20, 400)
        return {"kind": kind, "dtype": "f64", "n": n, "m": 2 * n + 1, "iters": rng.randint(64, 512)}
    if kind == "follow":
        dtype = rng.choice(["f64", "f32", "bf16"])
        n = _log_int(rng, 200, {"f64": 6000, "f32": 12000, "bf16": 16384}[dtype])
        return {"kind": kind, "dtype": dtype, "n": n, "m": rng.randint(2 * n, 4 * n), "iters": rng.randint(4, 16)}
    if kind == "catchup":
        return {"kind": kind, "dtype": "f64", "n": _log_int(rng, 4500, 24000), "chunks": 2}
    if kind == "tick":
        dtype = rng.choice(["f64", "f32", "bf16"])
        n = _log_int(rng, 200, {"f64": 4000, "f32": 8000, "bf16": 12000}[dtype])
        return {"kind": kind, "dtype": dtype, "n": n, "m": rng.randint(2 * n, 4 * n)}
    if kind == "batch":
        lo = _log_int(rng, 32, 512)
        return {"kind": kind, "dtype": rng.choice(["f64", "f32", "bf16"]), "count": _log_int(rng, 8, 256), "n_lo": lo,
                "n_hi": rng.randint(lo, 2 * lo), "m_mult": rng.randint(2, 6), "iters": rng.randint(4, 16)}
    lo = _log_int(rng, 48, 200)
    if kind == "fleet":
        return {"kind": kind, "dtype": rng.choice(["f64", "f32", "bf16"]), "count": _log_int(rng, 4, 64), "n_lo": lo,
                "n_hi": rng.randint(2 * lo, 1024), "m_mult": rng.randint(2, 5)}
    return {"kind": kind, "dtype": rng.choice(["f32", "bf16"]), "count": _log_int(rng, 2, 12), "n_lo": lo,
            "n_hi": rng.randint(2 * lo, 4000), "m_mult": rng.randint(2, 4)}


# ------------------------------------------------------------------ inputs
def _gen(seed, part):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + 7919 * part + 17) % (1 << 62))
    return g


def _gaussian(n, m, dtype, g, away=0.1):
    """Unit Gaussian rows in the storage type, a hidden point z with slack U(0,1) per row, and a
    start `away` per coordinate from it."""
    A = torch.randn((m, n), generator=g, device=DEV, dtype=torch.float64 if n * m < 1 << 26 else torch.float32)
    A /= torch.linalg.vector_norm(A, dim=1, keepdim=True)
    A = A.to(TORCH[dtype]).contiguous()
    z = torch.rand(n, generator=g, device=DEV, dtype=torch.float64) * 2.0 - 1.0
    b = _wide(A) @ z + torch.rand(m, generator=g, device=DEV, dtype=torch.float64)
    x0 = z + away * torch.randn(n, generator=g, device=DEV, dtype=torch.float64)
    return A, b, x0


def _vector(n, norm, g):
    v = torch.randn(n, generator=g, device=DEV, dtype=torch.float64)
    return v * (norm / torch.linalg.vector_norm(v))


def _wide(A):
    return A.to(torch.float64)


def _sizes(case):
    """Row lengths spread (over their logarithm) between n_lo and n_hi, and the row counts."""
    k, lo, hi = case["count"], case["n_lo"], case["n_hi"]
    ns = [int(round(lo * (hi / lo) ** ((i * 0.6180339887498949) % 1.0))) for i in range(k)]
    return [(n, case["m_mult"] * n + (i % 7 if hi > lo else 0)) for i, n in enumerate(ns)]


def _sway(n, iters, sigma, g):
    """A drift that comes back: `iters` translations whose second half undoes the first."""
    half = sigma * torch.randn((iters // 2, n), generator=g, device=DEV, dtype=torch.float64)
    return torch.cat([half, -half] + ([torch.zeros((1, n), device=DEV, dtype=torch.float64)] if iters % 2 else []))


def _tick_inputs(case, seed):
    n, m = case["n"], case["m"]
    g = _gen(seed, 1)
    A, b, x0 = _gaussian(n, m, case["dtype"], g, 0.02)
    k = max(1, m // 100)
    rows = torch.randperm(m, generator=g, device=DEV)[:k].contiguous()
    new = torch.randn((k, n), generator=g, device=DEV, dtype=torch.float64)
    new = (new / torch.linalg.vector_norm(new, dim=1, keepdim=True)).to(TORCH[case["dtype"]]).contiguous()
    # the start (and with it the hidden point) satisfies the replaced rows
    new_b = _wide(new) @ x0 + 0.5 + torch.rand(k, generator=g, device=DEV, dtype=torch.float64)
    return A, b, x0, rows, new, new_b, _vector(n, 0.05, g)


def _box(n, seed, offset):
    """b and x0 of the box-plus-sum system translated by `offset` along (1, ..., 1)."""
    b = torch.empty(2 * n + 1, device=DEV, dtype=torch.float64)
    b[:n] = 200.0 + offset
    b[n:2 * n] = -offset
    b[2 * n] = 200.0 * (n - 1) + n * offset
    return b, torch.rand(n, generator=_gen(seed, 2), device=DEV, dtype=torch.float64)


def _box_rows(n):
    A = torch.zeros((2 * n + 1, n), device=DEV, dtype=torch.float64)
    i = torch.arange(n, device=DEV)
    A[i, i] = 1.0
    A[n + i, i] = -1.0
    A[2 * n] = 1.0
    return A


def _params(case):
    kind = case["kind"]
    if kind == "box":
        return P.params(lam=1.0, eps=1e-6)
    if kind == "follow":
        return P.params(lam=0.02, eps=1e-6, track=True)
    if kind == "batch":
        return P.params(lam=0.005, eps=1e-3, track=True)
    if kind == "catchup":
        return P.params(lam=10.0, eps=1e-6, eps_relative=False)
    return P.params(lam=0.005, eps=1e-3, max_iters=300)


def _systems(case, seed):
    return [_gaussian(n, m, case["dtype"], _gen(seed, 100 + i), 0.02) + (_vector(n, 0.05, _gen(seed, 5000 + i)),)
            for i, (n, m) in enumerate(_sizes(case))]


def prepare(case, seed):
    kind, dtype = case["kind"], case["dtype"]
    st = {"case": case, "prm": _params(case), "pass": 0}
    if kind == "static":
        n, m, v = case["n"], case["m"], VEC[dtype]
        A, b, x = _gaussian(n, m, dtype, _gen(seed, 1))
        padded = torch.zeros((m, (n + v - 1) // v * v), device=DEV, dtype=TORCH[dtype])
        padded[:, :n] = A
        f = {"device": DEV, "dtype": torch.float64}
        st.update(A=padded, b=b, x=x, y=torch.empty(n, **f), r=torch.empty(m, **f),
                  h=torch.empty(1, device=DEV, dtype=torch.int64), d=torch.empty(1, **f))
    elif kind in ("check", "follow", "tick"):
        if kind == "tick":
            A, b, x0, st["rows"], st["new"], st["new_b"], st["v"] = _tick_inputs(case, seed)
        else:
            g = _gen(seed, 1)
            A, b, x0 = _gaussian(case["n"], case["m"], dtype, g)
            if kind == "follow":
                st["V"] = _sway(case["n"], case["iters"], 1e-3, g)
        st["x0"], st["s"] = x0, P.Solver(0)
        st["s"].set_system(A, b, x0, dtype=dtype)
    elif kind in ("box", "catchup"):
        n = case["n"]
        b, u = _box(n, seed, 0.0 if kind == "box" else 2.0)
        # far outside the box, or (the translation experiment) near its lower corner
        st["x0"] = 400.0 + 100.0 * u if kind == "box" else 0.01 * u
        st["v"] = torch.full((n,), 0.004, device=DEV, dtype=torch.float64)
        st["s"] = P.Solver(0)
        st["s"].set_system(_box_rows(n), b, st["x0"], dtype=dtype)
    elif kind in ("batch", "fleet"):
        st["b"], st["ids"], st["v"] = P.Batch(dtype), [], []
        for A, b, x0, v in _systems(case, seed):
            st["ids"].append(st["b"].add(A, b, x0))
            st["v"].append(v)
    else:
        st["requests"] = _systems(case, seed)
        st["server"] = P.Server(dtype, budget_bytes=64e9, prm=st["prm"], iters_per_round=16)
    torch.cuda.synchronize()
    return st


# ------------------------------------------------------------------ a pass
def _point(x, case):
    return x if case["dtype"] == "f64" else x.astype(np.float32)


def run(st):
    case, prm = st["case"], st["prm"]
    kind = case["kind"]
    sign = 1.0 if st["pass"] % 2 == 0 else -1.0      # what a pass moved, the next one moves back
    st["pass"] += 1
    if kind == "check":
        q = st["s"].eval_sweep(st["x0"])
        return {"y": q.y, "r": q.r, "h": q.h, "max_viol": q.max_viol}
    if kind == "static":
        P.eval_sweep_static(st["A"], st["b"], st["x"], st["y"], dtype=case["dtype"], r=st["r"], h=st["h"],
                            max_viol=st["d"])
        return {"y": st["y"], "r": st["r"], "h": st["h"], "max_viol": st["d"]}
    if kind == "box":
        s = st["s"]
        s.set_x(st["x0"])
        q = s.iterate(case["iters"], prm)
        x, _, _ = s.query()
        return {"x": x, "steps": q.iters, "h": q.h, "max_viol": q.max_viol, "y_norm": q.y_norm}
    if kind == "follow":
        s = st["s"]
        s.set_x(st["x0"])
        s.set_drift(st["V"])
        q = s.iterate(case["iters"], prm)
        x, _, _ = s.query()
        return {"x": _point(x, case), "steps": q.iters, "sweeps": q.sweeps}
    if kind == "catchup":
        s = st["s"]
        s.set_x(st["x0"])
        for _ in range(case["chunks"]):
            s.update_coeffs(translate=st["v"] * sign)
            q = s.iterate(4, prm)
        x, _, _ = s.query()
        return {"x": x, "steps": q.iters, "h": q.h, "max_viol": q.max_viol}
    if kind == "tick":
        s = st["s"]
        s.set_x(st["x0"])
        s.update_coeffs(st["rows"], st["new"], st["new_b"], st["v"] * sign)
        q, _ = s.solve(prm)
        x, b, _ = s.query(want_b=True)
        return {"x": _point(x, case), "b": b, "steps": q.iters, "certified": q.certified}
    if kind == "batch":
        st["b"].iterate(case["iters"], prm)
        return {"x": _point(np.concatenate([st["b"].query(i)[0] for i in st["ids"]]), case)}
    if kind == "fleet":
        bt = st["b"]
        for i, v in zip(st["ids"], st["v"]):
            bt.update(i, translate=v)
        q = bt.solve(prm)
        got = [bt.query(i) for i in st["ids"]]
        return {"x": _point(np.concatenate([x for x, _, _ in got]), case), "running": q.running,
                "steps": np.array([k.iters for _, _, k in got]), "certified": np.array([k.certified for _, _, k in got])}
    sv = st["server"]
    tickets = [sv.submit(A, b, x0) for A, b, x0, _ in st["requests"]]
    left = sv.round()
    for t, (_, _, _, v) in zip(tickets, st["requests"]):
        if sv.info(t)["state_name"] == "live":
            sv.update(t, translate=v)
    while left:
        left = sv.round()
    x = np.concatenate([sv.result(t) for t in tickets])
    steps = np.array([sv.info(t)["iters"] for t in tickets])
    for t in tickets:
        sv.release(t)
    return {"x": _point(x, case), "steps": steps}


# ------------------------------------------------------------------ 64 bits
def _sweep(A, nu, b, x):
    r = A @ x - b
    w = r.clamp(min=0.0) / nu
    return r, w @ A, int((r > 0).sum()), float((r / nu.sqrt()).max().clamp(min=0.0))


def _iterate(A, b, x, k, lam, eps, track=False, V=None, eps_relative=True, limit=1 << 60):
    """k checks (and steps) of the method; returns x, b, steps, whether it stopped, and the last check."""
    nu = (A * A).sum(dim=1)
    steps, last, done = 0, None, False
    for j in range(k):
        _, y, h, d = _sweep(A, nu, b, x)
        yn = float(torch.linalg.vector_norm(y))
        last = (h, d, yn)
        if d <= (eps * float(b.abs().max()) if eps_relative else eps):
            if not track:
                done = True
                break
        elif steps >= limit:
            break
        else:
            x = x - (lam / yn) * y
            steps += 1
        if V is not None and j < V.shape[0]:
            b = b + A @ V[j]
    return x, b, steps, done, last


def _iterate_box(b, x, k, lam, n):
    """_iterate for the rows [I; -I; 1^T] without forming them."""
    nu = torch.ones(2 * n + 1, device=DEV, dtype=torch.float64)
    nu[2 * n] = n
    steps, last = 0, None
    for _ in range(k):
        r = torch.cat([x - b[:n], -x - b[n:2 * n], (x.sum() - b[2 * n]).reshape(1)])
        w = r.clamp(min=0.0) / nu
        y = w[:n] - w[n:2 * n] + w[2 * n]
        yn = float(torch.linalg.vector_norm(y))
        last = (int((r > 0).sum()), float((r / nu.sqrt()).max().clamp(min=0.0)), yn)
        if last[1] <= 0.0:
            break
        x = x - (lam / yn) * y
        steps += 1
    return x, steps, last


def exact(case, seed):
    kind, n = case["kind"], case.get("n")
    if kind in ("check", "static"):
        A, b, x = _gaussian(n, case["m"], case["dtype"], _gen(seed, 1))
        A = _wide(A)
        r, y, h, d = _sweep(A, (A * A).sum(dim=1), b, x)
        if kind == "static":
            return {"y": y, "r": r, "h": torch.tensor([h], device=DEV),
                    "max_viol": torch.tensor([d], device=DEV, dtype=torch.float64)}
        return {"y": y, "r": r, "h": h, "max_viol": d}
    if kind in ("box", "catchup"):
        b, u = _box(n, seed, 0.0 if kind == "box" else 2.0)
        if kind == "box":
            x, steps, (h, d, yn) = _iterate_box(b, 400.0 + 100.0 * u, case["iters"], 1.0, n)
            return {"x": x, "steps": steps, "h": h, "max_viol": d, "y_norm": yn}
        x, steps = 0.01 * u, 0
        for _ in range(case["chunks"]):
            b = b + 0.004 * torch.cat([torch.ones(n, device=DEV, dtype=torch.float64),
                                       -torch.ones(n, device=DEV, dtype=torch.float64),
                                       torch.full((1,), float(n), device=DEV, dtype=torch.float64)])
            x, k, (h, d, _) = _iterate_box(b, x, 4, 10.0, n)
            steps += k
        return {"x": x, "steps": steps, "h": h, "max_viol": d}
    if kind == "follow":
        g = _gen(seed, 1)
        A, b, x0 = _gaussian(n, case["m"], case["dtype"], g)
        V = _sway(n, case["iters"], 1e-3, g)
        x, _, steps, _, _ = _iterate(_wide(A), b, x0, case["iters"], 0.02, 1e-6, True, V)
        return {"x": x, "steps": steps, "sweeps": case["iters"]}
    if kind == "tick":
        A, b, x0, rows, new, new_b, v = _tick_inputs(case, seed)
        A = _wide(A)
        A[rows] = _wide(new)
        b[rows] = new_b
        x, b, steps, done, _ = _iterate(A, b + A @ v, x0, 301, 0.005, 1e-3, limit=300)
        return {"x": x, "b": b, "steps": steps, "certified": int(done)}
    xs, steps = [], []
    for A, b, x0, v in _systems(case, seed):
        A = _wide(A)
        if kind == "batch":
            x, k = _iterate(A, b, x0, case["iters"], 0.005, 1e-3, True)[0], 0
        elif kind == "fleet":
            x, _, k, _, _ = _iterate(A, b + A @ v, x0, 301, 0.005, 1e-3, limit=300)
        else:
            x, _, k, done, _ = _iterate(A, b, x0, 16, 0.005, 1e-3)
            if not done:
                x, _, k2, _, _ = _iterate(A, b + A @ v, x, 285, 0.005, 1e-3)
                k += k2
        xs.append(x)
        steps.append(k)
    out = {"x": torch.cat(xs).cpu().numpy()}
    if kind != "batch":
        out["steps"] = np.array(steps)
    if kind == "fleet":
        out["running"] = 0
        out["certified"] = np.ones(len(xs), dtype=np.int64)
    return out


# ------------------------------------------------------------------ what a pass needs
def _pass_cost(n, m, es, sweeps):
    """Sweeps of one system: A, b and the norms read, b written, two products per element (the dot
    product and the translation's) and the violated rows' share left out as small."""
    return sweeps * (m * n * es + 24.0 * m), sweeps * 4.0 * m * n


def work(case):
    kind, es = case["kind"], BYTES[case["dtype"]]
    if kind in ("check", "static"):
        n, m = case["n"], case["m"]
        return {"bytes": m * n * es + 24.0 * m + 16.0 * n, "flops": 4.0 * m * n}
    if kind == "box":     # held on the chip: the rows are read once, the operations are every iteration's
        n, m = case["n"], case["m"]
        return {"bytes": m * n * es + 16.0 * m + 16.0 * n, "flops": case["iters"] * 4.0 * m * n}
    if kind == "follow":
        b, f = _pass_cost(case["n"], case["m"], es, case["iters"])
    elif kind == "catchup":   # every row is read once an iteration, half of them are violated
        b, f = _pass_cost(case["n"], 2 * case["n"] + 1, es, 4 * case["chunks"])
    elif kind == "tick":      # some ten checks, the certificate and the right-hand side: a pass over A each
        b, f = _pass_cost(case["n"], case["m"], es, 12)
    else:
        sweeps = {"batch": case.get("iters", 0), "fleet": 6, "serve": 24}[kind]
        b = f = 0.0
        for n, m in _sizes(case):
            db, df = _pass_cost(n, m, es, sweeps)
            b, f = b + db, f + df
    return {"bytes": b, "flops": f}
