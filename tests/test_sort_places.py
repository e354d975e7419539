"""The places that the sort's chunk table gives a chunk's cells, counted on the
host: every place is reached from any cell, and a full chunk of distinct cells
(the table half full) is inserted in few probes whatever cells of their
16-cell lines it uses.  Uniform probing takes 1.4 probes a cell at this load;
the bar is 6 on average and 64 at most."""
import ctypes

import numpy as np
import pytest

from hostlib import host_library

SOURCE = r"""
#include "grpic_launch.hpp"
#include <vector>
using namespace grpic;
extern "C" int places_reached(int c) {
    std::vector<char> seen(kHashSlots, 0);
    CellPlace at(c);
    int n = 0;
    for (int k = 0; k < kHashSlots; ++k, at.next()) {
        const int s = at.slot();
        if (s < 0 || s >= kHashSlots) return -1;
        n += !seen[s];
        seen[s] = 1;
    }
    return n;
}
// probes of inserting n distinct cells into an empty table: total, and the largest of one cell
extern "C" void probes(const int* cell, int n, long long* total, int* largest) {
    std::vector<char> taken(kHashSlots, 0);
    *total = 0;
    *largest = 0;
    for (int i = 0; i < n; ++i) {
        CellPlace at(cell[i]);
        int k = 1;
        for (; taken[at.slot()] && k <= kHashSlots; ++k) at.next();
        taken[at.slot()] = 1;
        *total += k;
        if (k > *largest) *largest = k;
    }
}
"""
N = 2048


@pytest.fixture(scope="module")
def table(tmp_path_factory):
    return host_library(tmp_path_factory.mktemp("places"), "places", SOURCE)


def test_every_place_is_reached(table):
    for c in (0, 5, 15, 16, 12345, 2**31 - 2):
        assert table.places_reached(c) == 2 * N


@pytest.mark.parametrize("nth", [16, 48, 1000, 1024, 2000, 2048, 4096, 65536])
@pytest.mark.parametrize("columns", ["one", "two neighbours", "four", "all"])
def test_few_probes(table, nth, columns):
    rng = np.random.default_rng(nth)
    rows = rng.permutation(8192)
    if columns == "one":
        cells = rows[:N] * nth + 5
    elif columns == "two neighbours":
        cells = (rows[: N // 2, None] * nth + np.array([6, 7])).ravel()
    elif columns == "four":
        cells = (rows[: N // 4, None] * nth + np.array([0, 3, 4, 8])).ravel()
    else:
        cells = rng.choice(8192 * min(nth, 2048), N, replace=False)
    cells = np.ascontiguousarray(rng.permutation(cells), dtype=np.int32)
    assert len(np.unique(cells)) == N
    total, largest = ctypes.c_longlong(), ctypes.c_int()
    table.probes(cells.ctypes.data_as(ctypes.c_void_p), N, ctypes.byref(total), ctypes.byref(largest))
    assert total.value <= 6 * N and largest.value <= 64, (total.value / N, largest.value)
