"""The FP64 certificates of a batch's stops, taken together: systems at the edges of
the row groups, bands and vectors, among systems whose stop the certificate overrules."""
import numpy as np
import pytest

import oracle
import paper_2003_09956_amd as P
import workloads as W
from test_gpu_certify import rounding_trap

pytestmark = pytest.mark.gpu

# (m, n): one row; a row group of 16 and one more; a band of 256 and one more;
# rows of one element, one vector, one wavefront's vectors and one more
SHAPES = [(1, 1), (15, 3), (16, 8), (17, 9), (255, 127), (256, 128), (257, 129), (300, 511), (513, 512), (40, 1000)]


@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
def test_stops_of_many_systems_certified_together(dtype):
    prm = P.params(lam=0.01, eps=1e-8, max_iters=2000)
    with P.Batch(dtype) as q:
        systems = []
        for k, (m, n) in enumerate(SHAPES):
            sys_ = W.gaussian(n, m, seed=k, dtype=dtype)
            v = 1e-3 * np.random.default_rng(k).standard_normal(n)
            i = q.add(sys_.A, sys_.b + 1.0, sys_.z)     # a unit of room: feasible before and after the move
            q.update(i, translate=v)
            systems.append((i, sys_, v, False))
            if k % 4 == 0:
                A, b, x = rounding_trap(dtype)
                systems.append((q.add(A, b, x), (A, b), None, True))
        out = q.solve(prm)
        assert out.running == 0
        for i, sys_, v, trap in systems:
            x, b, st = q.query(i, want_b=True)
            assert st.state == 1 and st.certified == 1, (i, st.as_dict())
            A, b0 = sys_ if trap else (sys_.A, sys_.b + 1.0)
            exact = b0 if trap else oracle.translate(A, dtype, b0, v)
            scale = np.abs(b0) + (0 if trap else np.abs(W.stored_to_f64(A, dtype)) @ np.abs(v))
            assert np.all(np.abs(b - exact) <= 1e-13 * scale)
            o = oracle.sweep(A, dtype, exact, x)
            assert o.dmax <= 1e-8 * o.binf * (1 + 1e-12) and o.dmax <= st.max_viol * (1 + 1e-12)
            assert st.iters >= 1 if trap else st.iters == 0
