"""The sort on grids on both sides of the scan's change (8192 tiles of 4096
cells): cell offsets, live count and order against torch's sort of the same
cells (whole numbers: equal), and the tiling through a push's live count."""
import pytest
import torch

from paper_2503_04558_amd import grpic
from paper_2503_04558_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nr,nth", [
    (8192, 4096 - 1),                    # below it
    (8192, 4096),                        # one tile above (the sentinel's)
    (9000, 4681),                        # 10,286 tiles: three passes of the totals, the last one short
])
def test_sort_offsets_on_large_grids(nr, nth):
    print(f"[gpu] sort on {nr}x{nth}", flush=True)
    g = wl.make_grid(nr, nth, 0.9)
    n = 60_001
    gen = torch.Generator(device="cuda").manual_seed(nth)
    cell = torch.randint(0, g.ncell, (n,), device="cuda", generator=gen)
    cell[:5] = torch.tensor([0, g.ncell - 1, g.ncell - 1, g.ncell // 2, 4095], device="cuda")
    cell[100:200] = -1
    p = grpic.empty_particles(n)
    for k in grpic.REAL_KEYS:
        p[k].fill_(0.5)
    p["sp"].zero_()
    p["cell"].copy_(cell)
    so = grpic.Sorter(g, n)
    off = torch.empty(g.ncell + 1, dtype=torch.int64, device="cuda")
    out = so.sort(p, cell_offsets=off)
    live = torch.sort(cell[cell >= 0])[0]
    assert int(so.n_alive.item()) == live.numel() == n - 100
    assert torch.equal(out["cell"][: live.numel()].long(), live)
    assert bool((out["cell"][live.numel():] == -1).all())
    probe = torch.unique(torch.cat([live, live + 1, torch.arange(0, g.ncell, 4096, device="cuda")]))
    assert torch.equal(off[probe], torch.searchsorted(live, probe))
    assert int(off[0]) == 0 and int(off[-1]) == live.numel()
    assert bool((off[1:] >= off[:-1]).all())
