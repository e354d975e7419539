"""The field step's strips of 64 columns, listed on the host for every column
count up to 2100: each column is stored once, also where workgroups of two
strips leave a surplus one past the last, and a strip that stores a column
within a guard of an axis stores the column beyond the axis that mirrors it.
And the launch shapes: every row lies in one segment, no workgroup is empty, and
where a march's rows are what it waits for (narrow grids, small ones) fewer than
four passes cut them for two workgroups on each of the 256 compute units."""
import pytest

from hostlib import host_library

SOURCE = r"""
#include "grpic_fields.hpp"
using grpic::FieldStrips;
// the smallest nth in [2 guard, hi] at which a column of 0 .. nth is not stored by exactly one of the
// strips in workgroups of two, 0 if none does
extern "C" int not_stored_once(int K, int guard, int hi) {
    for (int nth = 2 * guard; nth <= hi; ++nth) {
        const FieldStrips c(K, nth);
        for (int j = 0; j <= nth; ++j) {
            int times = 0;
            for (int s = 0; s < (c.count + 1) / 2 * 2; ++s) {
                const int lane = j - c.first_column(s);
                if (lane >= 0 && lane < 64 && c.stores(s, lane)) ++times;
            }
            if (times != 1) return nth;
        }
    }
    return 0;
}
// the smallest nth at which a strip that stores a column within guard of an axis does not mirror
extern "C" int unmirrored(int K, int guard, int hi) {
    for (int nth = 2 * guard; nth <= hi; ++nth) {
        const FieldStrips c(K, nth);
        for (int s = 0; s < c.count; ++s)
            for (int lane = 0; lane < 64; ++lane) {
                const int j = c.first_column(s) + lane;
                if (c.stores(s, lane) && (j <= guard || j >= nth - guard) && !c.mirrors(s, guard)) return nth;
            }
    }
    return 0;
}
// 0 if the launch shape of K passes on nr x nth (guard 2, no padding) holds
extern "C" int bad_shape(int K, int nr, int nth, int short_segments) {
    const grpic::FieldMarch L(K, nr, nth, grpic::field_plane(nr, nth + 5, 2));
    const int segs = (nr + L.seg_rows) / L.seg_rows, units = L.two ? (L.strips + 1) / 2 : L.strips;
    if (L.strips != FieldStrips(K, nth).count || L.seg_rows < 1) return 1;
    if (segs * L.seg_rows < nr + 1 || (segs - 1) * L.seg_rows >= nr + 1) return 2;   // all rows, no empty segment
    if (L.workgroups != units * segs) return 3;
    if (short_segments) {                         // the rows that 512 one-strip workgroups leave, or 6
        const int cut = 512 / L.strips, rows = (nr + cut) / cut;
        if (L.two || L.seg_rows > (rows > 6 ? rows : 6)) return 4;
    }
    return 0;
}
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    return host_library(tmp_path_factory.mktemp("strips"), "strips", SOURCE)


@pytest.mark.parametrize("K", [1, 2, 3, 4])
@pytest.mark.parametrize("guard", [2, 3, 4, 5, 6, 70])
def test_strips_store_and_mirror_every_column(rules, K, guard):
    assert rules.not_stored_once(K, guard, 2100) == 0
    assert rules.unmirrored(K, guard, 2100) == 0


@pytest.mark.parametrize("K", [1, 2, 3, 4])
def test_launch_shapes(rules, K):
    for nr in (1, 5, 6, 7, 64, 300, 1535, 2048, 20000, 400000):
        for nth in (4, 16, 57, 63, 64, 119, 126, 130, 250, 500, 720, 1000, 2048, 100000):
            if nr * nth < 5e8:
                assert rules.bad_shape(K, nr, nth, 0) == 0, (nr, nth)


@pytest.mark.parametrize("nr,nth", [(20000, 16), (4000, 48), (400000, 8), (20000, 130), (2000, 250), (2000, 500)])
@pytest.mark.parametrize("K", [1, 2, 3])
def test_narrow_and_small_grids_take_short_segments(rules, K, nr, nth):
    assert rules.bad_shape(K, nr, nth, 1) == 0
