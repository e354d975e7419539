"""The push where its evaluation of sin and cos changes: columns on both sides
of the pole limit (sin theta = 0.1) at either axis, and the equator, on a grid
without Taylor offsets, one with the long and one with the short series, every
kick, against the oracle at the parity bar (tests/parity.py)."""
import math

import numpy as np
import pytest

from paper_2503_04558_amd import workload as wl

from parity import assert_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nr,nth,kick,tiled", [
    (40, 64, "boris", False), (200, 300, "boris", True), (200, 300, "vay", False), (1700, 1300, "boris", True),
])
def test_parity_around_the_pole_limit(nr, nth, kick, tiled):
    print(f"[gpu] parity around the pole limit {nr}x{nth} {kick} tiled={tiled}", flush=True)
    g = wl.make_grid(nr, nth, 0.99)
    parts = wl.pairs(g, 2000, kind="mj", seed=nr, params=dict(T=0.5))
    n = len(parts["cell"])
    j0 = int(math.asin(0.1) / g.dth)
    cols = np.clip(np.array([j0 - 1, j0, j0 + 1, nth - 2 - j0, nth - 1 - j0, nth - j0, nth // 2]), 0, nth - 1)
    parts["cell"] = (parts["cell"] // nth * nth + cols[np.arange(n) % len(cols)]).astype(np.int32)
    assert_parity(g, wl.species_table(), parts, wl.wald_fields(g), wl.crossing_dt(g), 3, 1e-12, tiled=tiled, kick=kick)
