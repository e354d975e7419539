"""The columns beyond the axes after a field step: every one is written, also
where the columns it mirrors lie in a strip of 64 that is neither the first nor
the last.

test_mirrors_match_oracle compares every element with the oracle at the field
solver's bar (1e-12 x the component's largest magnitude, the same FP64 formulas
on both sides).  test_every_mirror_is_written checks, for every column count of
a range that runs through each strip width, that a mirrored column is its
source times +1 or -1 exactly (it is stored from the same value).
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


def _state(g, seed):
    rng = np.random.default_rng(seed)
    return [rng.normal(size=g.shape) * 0.1 for _ in range(6)]


@pytest.mark.parametrize("nr,nth,guard,pad,ncorr", [
    (9, 126, 2, 0, 0), (9, 126, 2, 1, 1), (7, 188, 2, 0, 1), (9, 126, 2, 0, 2),   # last launch of one pass
    (8, 127, 3, 0, 2), (8, 126, 3, 2, 1),
    (8, 124, 3, 0, 3), (11, 184, 3, 0, 4),                                        # of two
    (8, 122, 4, 0, 5),                                                            # of three
    (8, 120, 5, 3, 7),                                                            # of four
    (6, 300, 65, 0, 7), (6, 300, 70, 1, 1),                                       # wider than a strip
    (4000, 9, 2, 0, 0), (3500, 16, 2, 1, 1), (1700, 130, 2, 0, 2), (3100, 30, 3, 0, 4),   # tall: short segments
    (12, 200, 2, 63, 1), (12, 200, 2, 64, 1), (9, 60, 3, 200, 0), (2, 8, 2, 130, 7), (14, 130, 4, 90, 3),   # wide padding
    (15, 40, 6, 0, 2), (15, 40, 7, 3, 2), (20, 64, 12, 0, 7), (2, 200, 100, 1, 0),   # guard rows in the waves, apart
    (40, 300, 2, 18, 1), (40, 300, 2, 19, 0),                                     # copied in one run, row by row
])
def test_mirrors_match_oracle(nr, nth, guard, pad, ncorr):
    print(f"[gpu] field mirrors {nr}x{nth} guard={guard} pad={pad} ncorr={ncorr}", flush=True)
    g = wl.make_grid(nr, nth, 0.9, guard=guard)
    g = dataclasses.replace(g, pitch=g.pitch + pad)
    X, J = _state(g, nth), _state(g, nth + 1)[:3]
    dt = wl.crossing_dt(g)
    solver = grpic.FieldSolver(grpic.make_metric(g.a, g.M), g)
    st = [torch.as_tensor(x).cuda() for x in X]
    Jd = [torch.as_tensor(0.1 * j).cuda() for j in J]
    solver.step(st, Jd, dt, 0.53, ncorr, 2, 0.2)
    torch.cuda.synchronize()
    want = orc.field_step(g, X, [0.1 * j for j in J], dt, 0.53, ncorr, damp_cells=2, damp_max=0.2)
    for k in range(6):
        scale = np.abs(want[k][guard:guard + nr, guard:guard + nth]).max()
        assert np.abs(st[k].cpu().numpy() - want[k]).max() <= TOL * scale, k


@pytest.mark.parametrize("guard", [2, 3, 5])
@pytest.mark.parametrize("ncorr", [1, 3, 5, 7])     # last launches of one to four passes
def test_every_mirror_is_written(guard, ncorr):
    print(f"[gpu] field mirrors, all nth, guard={guard} ncorr={ncorr}", flush=True)
    m = torch.arange(1, guard + 1, device="cuda")
    missing = []
    for nth in range(2 * guard, 256):
        g = wl.make_grid(4, nth, 0.9, guard=guard)
        st = list(torch.randn((6,) + g.shape, dtype=torch.float64, device="cuda"))
        grpic.FieldSolver(grpic.make_metric(g.a, g.M), g).step(st, None, wl.crossing_dt(g), 0.53, ncorr)
        ok = torch.ones((), dtype=torch.bool, device="cuda")
        for k, x in enumerate(st):
            sign = -1.0 if k in (1, 4) else 1.0
            half = 1 if k in (1, 3, 5) else 0
            ok &= (x[:, guard - m] == sign * x[:, guard + m - half]).all()
            ok &= (x[:, guard + nth + m - half] == sign * x[:, guard + nth - m]).all()
        if not bool(ok):
            missing.append(nth)
    assert not missing, missing


def test_cubic_push_after_a_step_reads_fresh_columns():
    """Guard 3, nth = 126, one corrector: the cubic gather of a particle in
    the last half cell reads column nth + 1 of D^th, B^r, B^ph.  The caller's
    arrays hold values there that a step must replace; the push through the
    stepped fields agrees with the oracle's (bars of the parity tests: 1e-11
    relative to 1 + |value| for one step)."""
    print("[gpu] cubic push after a field step, guard 3, nth 126", flush=True)
    g = wl.make_grid(40, 126, 0.9, guard=3)
    X = [np.array(f, copy=True) for f in wl.wald_fields(g, B0=2.0)]
    for x in X:
        x[:, :g.guard] = 1e3
        x[:, g.guard + g.nth + 1:] = 1e3
    dt = wl.crossing_dt(g)
    st = [torch.as_tensor(x).cuda() for x in X]
    grpic.FieldSolver(grpic.make_metric(g.a, g.M), g).step(st, None, dt, 0.53, 1)
    want = orc.field_step(g, X, None, dt, 0.53, 1)
    rng = np.random.default_rng(3)
    n = 500
    i = rng.integers(3, g.nr - 3, n)
    xth = rng.uniform(0.5, 0.99, n)
    uh = rng.normal(size=(3, n))
    ur, uth, uph = wl.frame_to_covariant(g.a, g.M, g.r(i + 0.5), g.theta(g.nth - 1 + xth), uh)
    host = dict(cell=(i * g.nth + g.nth - 1).astype(np.int32), xr=np.full(n, 0.5), xth=xth, ur=ur, uth=uth, uph=uph,
                w=np.ones(n), sp=np.zeros(n, np.uint8))
    parts = grpic.to_device(host)
    J = [torch.zeros(g.shape, dtype=torch.float64, device="cuda") for _ in range(3)]
    sp = wl.species_table()
    grpic.grpic_push_deposit(grpic.make_metric(g.a, g.M), g, sp, parts, st, J, dt, 1, order=3)
    out = grpic.to_host(parts)
    ref = orc.run(g, sp, host, want, dt, 1, order=3)[0]
    live = ref["cell"] >= 0
    assert live.any() and np.array_equal(out["cell"], ref["cell"])
    for k in ("xr", "xth", "ur", "uth", "uph"):
        err = np.abs(out[k][live] - ref[k][live]) / (1.0 + np.abs(ref[k][live]))
        assert err.max() <= 1e-11, (k, err.max())


@pytest.mark.parametrize("ncorr,launches", [(0, 1), (1, 1), (2, 2)])
def test_short_steps_take_one_launch(ncorr, launches):
    """A step of one or two passes reads a copy of the state (the third six
    planes of the workspace) and needs neither the corrector's constant part
    nor an iterate in memory: the first twelve planes keep what they held.
    (Two launches of a pass each move half as much again; on 100000 x 250 they
    were slower than a pass at a time through tiles had been.)"""
    g = wl.make_grid(40, 100, 0.9)
    solver = grpic.FieldSolver(grpic.make_metric(g.a, g.M), g)
    ws = solver.ws.view(torch.float64).view((18,) + g.shape)
    ws.fill_(7.0)
    st = list(torch.randn((6,) + g.shape, dtype=torch.float64, device="cuda"))
    solver.step(st, None, wl.crossing_dt(g), 0.53, ncorr)
    assert bool((ws[:12] == 7.0).all()) == (launches == 1)
