"""The batched sweep's cells and groups: a batch whose items are single cells, several, or whole
groups gives every system the same bits (the grid sets which, through the batch's size per
workgroup), and they follow the oracle.  Systems of several cells a group, in every row form,
with ragged last cells down to one row; a drift schedule has the rows' b written, too."""
import numpy as np
import pytest

import oracle
import paper_2003_09956_amd as P
import workloads as W
from parity import TOL, weighted_abs_rows

pytestmark = pytest.mark.gpu
SHAPES = {"f32": [(96, 12007), (255, 6081), (500, 4201), (1000, 2561), (1999, 3001), (64, 130)],
          "bf16": [(256, 20011), (512, 12289), (1000, 5003), (2000, 6007), (4000, 2999), (500, 1)],
          "f64": [(60, 18001), (128, 9025), (250, 6007), (500, 4993), (1000, 3001), (33, 7)]}


@pytest.mark.parametrize("dtype", list(SHAPES))
def test_cells_and_groups_agree(dtype):
    systems = [W.gaussian(n, m, seed=n + m, dtype=dtype) for n, m in SHAPES[dtype]]
    drifts = [W.drift(s.A.shape[1], 9, sigma=1e-3, seed=s.A.shape[0]) for s in systems]
    lam = 0.05
    prm = P.params(lam=lam, eps=1e-9)
    trk = P.params(lam=lam, eps=1e-9, track=True)
    ref = None
    for grid in (0, 48, 12, 1):   # items of one cell, of some, of groups
        print(dtype, grid, flush=True)
        with P.Batch(dtype) as B:
            kib = B.get_tile()["item_kib"]
            B.set_tile(item_kib=kib, grid=grid)
            ids = [B.add(s.A, s.b, x0=s.z + 0.3) for s in systems]
            B.iterate(1, prm)
            got = [B.query(i)[0] for i in ids]
            if grid == 0:
                for s, x1 in zip(systems, got):
                    x = s.z + 0.3
                    o = oracle.sweep(s.A, dtype, s.b, x)
                    xo, status = oracle.step(o.y, o.h, 0, lam, x)
                    if status:
                        assert np.array_equal(x1, x)   # no violated row: no step
                        continue
                    near = o.r > -TOL[dtype] * o.t
                    s_y = np.linalg.norm(weighted_abs_rows(s.A, dtype, np.where(near, o.t / o.nu, 0)))
                    bound = TOL[dtype] * (np.linalg.norm(x) + lam * s_y / np.linalg.norm(o.y))
                    assert np.linalg.norm(x1 - xo) <= bound, s.A.shape
            for i, V in zip(ids, drifts):
                B.set_drift(i, V)
            B.iterate(9, trk)
            B.iterate(2, prm)
            q = [B.query(i, want_b=True) for i in ids]
            got += [r[0] for r in q] + [r[1] for r in q] + [np.array([r[2].iters, r[2].h, r[2].max_viol]) for r in q]
        if ref is None:
            ref = got
        for k, (a, b) in enumerate(zip(ref, got)):
            assert np.array_equal(a, b), (grid, k)
