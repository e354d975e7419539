"""bench.py's count of the grid planes that a field step moves at least, by its
launches: state, areas and currents in and state out for one or two passes;
otherwise a first launch that also writes the constant part, and later ones of
up to four passes in all."""
import pytest

import bench


@pytest.mark.parametrize("ncorr,planes", [(0, 21), (1, 21), (2, 27 + 24), (3, 27 + 24), (7, 27 + 24), (8, 27 + 2 * 24),
                                          (11, 27 + 2 * 24), (12, 27 + 3 * 24), (64, 27 + 16 * 24)])
def test_field_planes(ncorr, planes):
    assert bench.field_planes(ncorr) == planes
