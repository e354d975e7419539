"""The untiled push where its workgroup size changes (one wave up to 65,536
particles, four above) and at the ragged ends of either size, both kicks, CIC
and cubic shape, against the oracle at the parity bar (tests/parity.py)."""
import pytest

from paper_2503_04558_amd import grpic
from paper_2503_04558_amd import workload as wl

from parity import assert_parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,kick,order", [
    (1, "boris", 1), (64, "boris", 3), (65, "vay", 1), (65535, "boris", 1), (65536, "boris", 3), (65536, "vay", 1),
    (65537, "boris", 1), (65537, "boris", 3), (65793, "vay", 1),
])
def test_parity_around_the_block_size_change(n, kick, order):
    print(f"[gpu] untiled push of {n} particles, {kick}, order {order}", flush=True)
    g = wl.make_grid(128, 128, 0.9, guard=3)
    parts = {k: v[:n] for k, v in wl.pairs(g, 33000, kind="mj", seed=17, params=dict(T=0.5)).items()}
    assert len(parts["cell"]) == n
    assert_parity(g, wl.species_table(), parts, wl.wald_fields(g), 0.5 * wl.crossing_dt(g), 2, 1e-12, kick=kick,
                  order=order)
