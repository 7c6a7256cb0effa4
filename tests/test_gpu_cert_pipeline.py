"""The certificate's pass over A reads ahead, across the chunks of a row and across row groups:
enough systems that a workgroup takes several groups, rows of one chunk, a whole number of them
and one element more."""
import numpy as np
import pytest

import oracle
import paper_2003_09956_amd as P
import workloads as W

pytestmark = pytest.mark.gpu
# elements of a chunk: 64 vectors of 16 bytes
CHUNK = {"f64": 128, "f32": 256, "bf16": 512}


@pytest.mark.parametrize("dtype", list(CHUNK))
def test_groups_and_chunks_ahead(dtype):
    c = CHUNK[dtype]
    prm = P.params(lam=0.01, eps=1e-8, max_iters=2000)
    kinds = [W.gaussian(n, m, seed=n, dtype=dtype) for n, m in ((c, 3001), (c + 1, 3000), (2 * c, 2999), (3 * c - 1, 2993))]
    with P.Batch(dtype) as q:
        ids = []
        for k in range(16):
            w = kinds[k % 4]
            v = 1e-3 * np.random.default_rng(k).standard_normal(w.A.shape[1])
            i = q.add(w.A, w.b + 1.0, w.z)
            q.update(i, translate=v)
            ids.append((i, w, v))
        assert q.solve(prm).running == 0
        for i, w, v in ids:
            x, b, st = q.query(i, want_b=True)
            assert st.state == 1 and st.certified == 1 and st.iters == 0
            exact = oracle.translate(w.A, dtype, w.b + 1.0, v)
            scale = np.abs(w.b + 1.0) + np.abs(W.stored_to_f64(w.A, dtype)) @ np.abs(v)
            assert np.all(np.abs(b - exact) <= 1e-13 * scale)
            o = oracle.sweep(w.A, dtype, exact, x)
            assert o.dmax <= st.max_viol * (1 + 1e-12) and st.max_viol <= o.dmax + 1e-9
