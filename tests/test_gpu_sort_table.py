"""The sort's per-chunk cell table at its edges, against numpy's counting of
the same cells (whole numbers: equal): a full chunk of distinct cells that all
fall on one place of their 16-cell blocks, distinct neighbouring cells, one
crowded cell, chunks of removed particles, and grids of one and of several
scan blocks."""
import numpy as np
import pytest
import torch

from paper_2503_04558_amd import grpic
from paper_2503_04558_amd import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nr,nth,kind,n", [
    (64, 1024, "stride16", 2048), (64, 1024, "stride16", 4097), (64, 1024, "neighbours", 2047),
    (48, 48, "one", 5000), (64, 64, "removed", 6145), (63, 65, "random", 2049), (300, 200, "random", 100_000),
    (8, 8, "random", 1),
])
def test_sort_places_every_particle(nr, nth, kind, n):
    print(f"[gpu] sort table {nr}x{nth} {kind} n={n}", flush=True)
    g = wl.make_grid(nr, nth, 0.9)
    rng = np.random.default_rng(n)
    if kind == "stride16":
        cell = 16 * (rng.permutation(n) % (g.ncell // 16)) + 5
    elif kind == "neighbours":
        cell = 3000 + rng.permutation(n)
    elif kind == "one":
        cell = np.full(n, 77)
    else:
        cell = rng.integers(0, g.ncell, n)
    if kind == "removed":
        cell[: 2048] = -1
        cell[rng.random(n) < 0.3] = -1
    cell = cell.astype(np.int32)
    real = {k: rng.random(n) for k in ("xr", "xth", "ur", "uth", "uph", "w")}
    parts = grpic.to_device(dict(cell=cell, sp=(np.arange(n) % 3).astype(np.uint8), tag=np.arange(n, dtype=np.uint64),
                                 **real))
    so = grpic.Sorter(g, n, with_tag=True)
    off = torch.empty(g.ncell + 1, dtype=torch.int64, device="cuda")
    out = grpic.to_host(so.sort(parts, cell_offsets=off))
    torch.cuda.synchronize()
    live = cell[cell >= 0]
    want = np.concatenate([[0], np.cumsum(np.bincount(live, minlength=g.ncell))])
    assert int(so.n_alive.item()) == live.size
    assert np.array_equal(off.cpu().numpy(), want)
    assert np.array_equal(out["cell"][: live.size], np.sort(live))
    assert (out["cell"][live.size:] == -1).all()
    tag = out["tag"][: live.size].astype(np.int64)
    assert np.array_equal(np.sort(tag), np.flatnonzero(cell >= 0))
    assert np.array_equal(out["cell"][: live.size], cell[tag])
    assert np.array_equal(out["sp"][: live.size], tag % 3)
    for k, v in real.items():
        assert np.array_equal(out[k][: live.size], v[tag]), k
