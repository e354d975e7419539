"""The field step's marching launches against the CPU oracle at their edges:
strips of 64 columns (one, one column into the next, two strips in a
workgroup), segments of rows down to a few, every split of the passes into
launches of one to four, wider guards and padded rows.

Bar as in the field solver's tests: |GPU - oracle| <= 1e-12 x the largest
magnitude of the component, at every element (the same formulas in FP64 on
both sides, a few ulp per pass, O(1) factors).
"""
import dataclasses

import numpy as np
import pytest
import torch

from oracle import oracle as orc
from paper_2503_04558_amd import grpic
from paper_2503_04558_amd import workload as wl

pytestmark = pytest.mark.gpu

TOL = 1e-12


@pytest.mark.parametrize("nr,nth,a,guard,pad,ncorr,damp", [
    (5, 63, 0.9, 2, 0, 7, 2),            # one strip, rows fewer than the launch's halo
    (6, 64, 0.99, 2, 0, 3, 0),           # one column into the second strip; 2 + 2 passes
    (30, 119, 0.0, 3, 5, 4, 9),          # 3 + 2 passes, last column of the second strip
    (31, 120, 0.99, 2, 1, 2, 0),         # 2 + 1 passes, first column of the third
    (48, 200, 0.99, 3, 3, 0, 6),         # no corrector: one pass from a copy
    (49, 201, 0.9, 2, 0, 1, 7),          # 1 + 1 passes
    (200, 700, 0.99, 2, 2, 7, 40),       # two strips in a workgroup, odd number of strips
    (301, 640, 0.9, 2, 0, 8, 33),        # three launches of 3, even number of strips
    (90, 1100, 0.99, 3, 0, 13, 0),       # four launches
])
def test_march_edges_match_oracle(nr, nth, a, guard, pad, ncorr, damp):
    print(f"[gpu] field march {nr}x{nth} a={a} guard={guard} pad={pad} ncorr={ncorr} damp={damp}", flush=True)
    g = wl.make_grid(nr, nth, a, guard=guard)
    g = dataclasses.replace(g, pitch=g.pitch + pad)
    rng = np.random.default_rng(nr * 1000 + nth)
    shape = (nr + 1 + 2 * guard, g.pitch)
    X = [rng.normal(size=shape) * 0.1 for _ in range(6)]
    J = [rng.normal(size=shape) * 0.01 for _ in range(3)]
    dt = wl.crossing_dt(g)
    solver = grpic.FieldSolver(grpic.make_metric(g.a, g.M), g)
    st, Jd = [torch.as_tensor(x).cuda() for x in X], [torch.as_tensor(f).cuda() for f in J]
    want = X
    for step in range(2):
        cur = Jd if step == 0 else None
        solver.step(st, cur, dt, 0.53, ncorr, damp, 0.2)
        want = orc.field_step(g, want, J if step == 0 else None, dt, 0.53, ncorr, damp_cells=damp, damp_max=0.2)
    torch.cuda.synchronize()
    for k in range(6):
        half = k in (0, 4, 5)
        scale = np.abs(want[k][guard:guard + nr + (0 if half else 1), guard:guard + nth + 1]).max()
        got = st[k].cpu().numpy()
        assert np.isfinite(got).all(), k
        assert np.abs(got - want[k]).max() <= TOL * scale, (k, np.abs(got - want[k]).max() / scale)
