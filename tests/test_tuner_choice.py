"""The threshold that the tuner takes for five measured times (host code of the
library): the default unless another is more than 2% faster, and of several that
time the same launches the one nearest to the default."""
import ctypes

import pytest


def nearest_faster(times):
    from paper_1402_4247_amd import kgev
    return kgev.lib.kgev_internal_nearest_faster((ctypes.c_float * 5)(*times))


@pytest.mark.parametrize("times,place", [
    ((1.0, 1.0, 1.0, 1.0, 1.0), 2),
    ((0.99, 0.985, 1.0, 0.981, 0.99), 2),          # within 2%
    ((1.0, 1.0, 1.0, 0.9, 0.897), 3),              # the same launches: the nearer one
    ((0.897, 0.9, 1.0, 1.0, 1.0), 1),
    ((1.0, 1.0, 1.0, 1.0, 0.9), 4),                # the nearer one changes nothing
    ((1.0, 1.0, 1.0, 0.95, 0.9), 4),
    ((0.94, 1.2, 1.0, 0.95, 0.948), 0),            # the faster side
    ((0.96, 0.95, 1.0, 0.9, 1.3), 3),
])
def test_nearest_faster(times, place):
    assert nearest_faster(times) == place
