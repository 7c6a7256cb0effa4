"""The built-in shape of the one-pass sweep at the edges of its rule: the longest row of each
entry, one element less, and one more (the next entry), with a translation pending; and
both sides of the rule's two lines on the number of rows."""
import numpy as np
import pytest

import oracle
import paper_2003_09956_amd as P
import workloads as W
from parity import check_sweep

pytestmark = pytest.mark.gpu

EDGES = {"f64": [32, 64, 128, 256, 384, 512, 768, 1024, 1536, 2048, 3072, 4096, 6144, 8192],
         "f32": [64, 128, 256, 512, 768, 1024, 1536, 2048, 4096, 6144, 8192, 12288, 16384],
         "bf16": [128, 256, 512, 1024, 1536, 2048, 3072, 4096, 6144, 8192, 12288, 16384]}


def sweep_against_oracle(dtype, n, m):
    sys_ = W.gaussian(n, m, seed=n + m, dtype=dtype)
    rng = np.random.default_rng(n)
    v = rng.normal(scale=0.05, size=n)
    x = sys_.z + rng.normal(scale=1.0 / np.sqrt(n) + 0.05, size=n)
    with P.Solver(0) as s:
        s.set_system(sys_.A, sys_.b, dtype=dtype)
        tile = s.get_tile()
        s.update_coeffs(translate=v)
        g = s.eval_sweep(x)
    o = oracle.sweep(sys_.A, dtype, oracle.translate(sys_.A, dtype, sys_.b, v), x)
    check_sweep(sys_.A, dtype, o, g.y, g.h, g.max_viol, g.r, label=f"rule {dtype} {n}x{m}")
    return tile


@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
def test_rule_at_row_length_edges(dtype):
    vec = {"f64": 2, "f32": 4, "bf16": 8}[dtype]
    for edge in EDGES[dtype]:
        for n in (edge - 1, edge, edge + 1):
            print(dtype, n, flush=True)
            t = sweep_against_oracle(dtype, n, 530 if n < 3000 else 270)
            if n <= edge:
                assert t["kind"] == 0 and t["lanes_per_row"] * t["chunks"] * vec == edge, (n, t)
    assert t["kind"] == 1     # one element past the last entry: the split-row form


def test_rule_at_row_count_edges():
    assert sweep_against_oracle("f64", 100, 8191)["lanes_per_row"] == 64
    assert sweep_against_oracle("f64", 100, 8192)["lanes_per_row"] == 16
    one, two = (sweep_against_oracle("bf16", 20, m)["grid"] for m in (65535, 65536))
    assert two == 2 * one
