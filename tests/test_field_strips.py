"""The field step's strips of 64 columns, listed on the host for every column
count up to 2100: each column is stored once, also where workgroups of two
strips leave a surplus one past the last, and a strip that stores a column
within a guard of an axis stores the column beyond the axis that mirrors it."""
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
"""


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    return host_library(tmp_path_factory.mktemp("strips"), "strips", SOURCE)


@pytest.mark.parametrize("K", [1, 2, 3, 4])
@pytest.mark.parametrize("guard", [2, 3, 4, 5, 6, 70])
def test_strips_store_and_mirror_every_column(rules, K, guard):
    assert rules.not_stored_once(K, guard, 2100) == 0
    assert rules.unmirrored(K, guard, 2100) == 0
