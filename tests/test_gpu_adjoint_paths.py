"""The reverse sweep's kernel variants against the oracle's dual numbers:
grids too coarse for the Taylor offsets and fine enough for them, three
correctors and another count, checkpoints every step (no state recomputed)
and every few, particles at both axes, numbers of particles around a wave,
and a lambda that is dense, on the last row, or in the last column only.

Bar, particle by particle, as in the adjoint's tests: |g_gpu - g_orc| <=
1e-9 |g_orc|_vec + 1e-13 max_p |g_orc|_vec + 64 s_p, s_p the change of the
oracle's derivative when the momenta move by 4 ulps.
"""
import numpy as np
import pytest

from oracle import oracle as orc
from paper_2503_04558_amd import workload as wl

from test_gpu_adjoint import EPS, backward, forward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nr,nth,a,n,every,nsteps,ncorr,where", [
    (64, 64, 0.99, 63, 1, 4, 3, "dense"),
    (64, 40, 0.0, 65, 3, 6, 5, "row"),
    (160, 130, 0.9, 64, 1, 5, 3, "dense"),
    (200, 100, 0.99, 129, 2, 4, 3, "column"),
    (130, 257, 0.9, 1, 4, 8, 1, "dense"),
])
def test_momentum_gradient_paths(nr, nth, a, n, every, nsteps, ncorr, where):
    print(f"[gpu] adjoint paths {nr}x{nth} a={a} n={n} every={every} steps={nsteps} ncorr={ncorr} {where}", flush=True)
    g = wl.make_grid(nr, nth, a)
    dt = wl.crossing_dt(g)
    fields = wl.wald_fields(g, B0=2.0)
    parts = {k: v[:n].copy() for k, v in wl.pairs(g, (n + 1) // 2, kind="mj", seed=n, params=dict(T=0.5)).items()}
    ci = parts["cell"] // nth
    edge = np.arange(n) % 4
    cj = np.where(edge == 0, 0, np.where(edge == 1, nth - 1, parts["cell"] % nth))
    if where == "row":
        ci = np.full(n, nr - 2)
    if where == "column":
        cj = np.full(n, nth - 1)
    parts["cell"] = (ci * nth + cj).astype(np.int32)
    rng = np.random.default_rng(nr)
    lam = [rng.normal(size=g.shape) * dt for _ in range(3)]
    if where == "row":
        for x in lam:
            x[: g.guard + nr - 1] = 0.0
    if where == "column":
        for x in lam:
            x[:, : g.guard + nth - 1] = 0.0
    sp = wl.species_table()
    start, F, _, ck, _ = forward(g, sp, parts, fields, dt, nsteps=nsteps, ckpt_every=every, ncorr=ncorr)
    gu, gF = backward(g, sp, start, F, lam, dt, ck, nsteps=nsteps, ckpt_every=every, ncorr=ncorr)

    def oracle(p0):
        out = np.zeros((n, 3))
        for p in range(n):
            one = {k: v[p:p + 1] for k, v in p0.items()}
            for k in range(3):
                t = [np.zeros(1) for _ in range(3)]
                t[k][0] = 1.0
                _, out[p, k], _ = orc.loss_dual(g, sp, one, fields, lam, dt, nsteps, ncorr=ncorr, tu=t)
        return out

    ref = oracle(parts)
    sens = np.abs(oracle({k: v * (1.0 + 4 * EPS) if k in ("ur", "uth", "uph") else v for k, v in parts.items()})
                  - ref).max(axis=1)
    scale = np.abs(ref).max(axis=1)
    assert scale.max() > 0
    err = np.abs(gu - ref).max(axis=1)
    bar = 1e-9 * scale + 1e-13 * scale.max() + 64 * sens
    assert np.all(err <= bar), (np.flatnonzero(err > bar)[:5], (err / np.maximum(bar, 1e-300)).max())
    tF = [rng.normal(size=g.shape) * np.abs(f).max() for f in fields]
    _, dL, _ = orc.loss_dual(g, sp, parts, fields, lam, dt, nsteps, ncorr=ncorr, tF=tF)
    got = sum(float((x * t).sum()) for x, t in zip(gF, tF))
    terms = sum(float(np.abs(x * t).sum()) for x, t in zip(gF, tF))
    assert abs(got - dL) <= 1e-9 * max(abs(dL), 1e-3 * terms), (got, dL)
