"""Row norms in 16-byte loads and the evaluation that tells its totals itself: rows of one element
to past the four vectors in flight, in every type, against FP64 norms (through the distance of a
single violated row), and device results at the edge of the rule against host ones."""
import numpy as np
import pytest
import torch

import paper_2003_09956_amd as P
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f64", "f32", "bf16"])
def test_norms_of_every_length(dtype):
    vec = {"f64": 2, "f32": 4, "bf16": 8}[dtype]
    for n in (1, vec - 1 or 1, vec, vec + 1, 64 * vec - 1, 64 * vec, 64 * vec + 1, 256 * vec, 256 * vec + 1, 257 * vec - 1):
        print(dtype, n, flush=True)
        w = W.gaussian(n, 9, seed=n, dtype=dtype)
        A = W.stored_to_f64(w.A, dtype)
        with P.Solver(0) as s:
            for i in (0, 3, 8):    # only row i is violated, by exactly one in A x - b at x = 0
                b = np.ones(9)
                b[i] = -1.0
                s.set_system(w.A, b, dtype=dtype)
                g = s.eval_sweep(np.zeros(n))
                want = 1.0 / np.linalg.norm(A[i])
                assert g.h == 1 and abs(g.max_viol - want) <= 4e-15 * want * max(1, n) ** 0.5


@pytest.mark.parametrize("n", [2047, 2048, 2049, 2112])
def test_device_evaluations_match_host_ones(n):
    w = W.gaussian(n, 700, seed=n, dtype="f64")
    with P.Solver(0) as s:
        s.set_system(w.A, w.b, dtype="f64")
        for far in (1.0, 0.0, 1.0):
            x = w.z + far
            a, d = s.eval_sweep(x), s.eval_sweep(torch.from_numpy(x).cuda())
            assert a.h == d.h and a.max_viol == d.max_viol
            assert np.array_equal(a.y, d.y.cpu().numpy()) and np.array_equal(a.r, d.r.cpu().numpy())
