"""The built-in shape on both sides of the line below which a row's vectors are spread over more
wavefronts, at whole and ragged row lengths, with a translation pending and without."""
import numpy as np
import pytest

import oracle
import paper_2003_09956_amd as P
import workloads as W
from parity import check_sweep

pytestmark = pytest.mark.gpu

# storage, longest row of the entry, shortest, rows below which it is spread, lanes then and from there on
LINES = [("f64", 768, 513, 1000, 128), ("f64", 1024, 769, 1000, 256), ("f64", 1536, 1025, 2000, 256),
         ("f32", 1536, 1025, 1500, 128), ("f32", 2048, 1537, 1500, 256),
         ("bf16", 3072, 2049, 3500, 128), ("bf16", 4096, 3073, 3500, 256), ("bf16", 6144, 4097, 5000, 256)]


@pytest.mark.parametrize("dtype,longest,shortest,few,lanes", LINES)
def test_rows_are_spread_on_short_systems(dtype, longest, shortest, few, lanes):
    for n, m in ((longest, few - 1), (longest, few), (longest - 1, 3), (shortest, 7), (shortest, few - 1)):
        w = W.gaussian(n, m, seed=n + m, dtype=dtype)
        rng = np.random.default_rng(n)
        v = rng.normal(scale=0.05, size=n)
        x = w.z + rng.normal(scale=1.0 / np.sqrt(n) + 0.05, size=n)
        print(dtype, n, m, flush=True)
        with P.Solver(0) as s:
            s.set_system(w.A, w.b, dtype=dtype)
            t = s.get_tile()
            assert t["lanes_per_row"] == (lanes if m < few else 64)
            assert t["lanes_per_row"] * t["chunks"] * {"f64": 2, "f32": 4, "bf16": 8}[dtype] == longest
            still = s.eval_sweep(x)
            s.update_coeffs(translate=v)
            moved = s.eval_sweep(x)
        for g, b in ((still, w.b), (moved, oracle.translate(w.A, dtype, w.b, v))):
            o = oracle.sweep(w.A, dtype, b, x)
            check_sweep(w.A, dtype, o, g.y, g.h, g.max_viol, g.r, label=f"few rows {dtype} {n}x{m}")
