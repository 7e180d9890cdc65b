"""How a reduction is divided (host logic of the library, no GPU): the order at
which the blocked columns hand over, and the groups of workgroups that take
over there."""
import ctypes

import pytest


@pytest.fixture(scope="module")
def plan():
    from paper_1402_4247_amd import kgev
    f = kgev.lib.kgev_internal_hetrd_plan
    f.argtypes = [ctypes.c_int32, ctypes.c_int32, ctypes.c_int64, ctypes.c_int32, ctypes.c_void_p]

    def call(n, nb, nk, units):
        out = (ctypes.c_int32 * 4)()
        f(n, nb, nk, units, out)
        return tuple(out)

    return call


ORDERS = (2, 128, 129, 160, 161, 200, 256, 257, 300, 384, 400, 512, 600, 640, 700, 768, 900, 1024, 1100, 2000, 4096)


@pytest.mark.parametrize("units", [0, 1, 8, 16, 32, 38, 64, 128, 228, 256, 304])
def test_groups_fit_beside_three_others(plan, units):
    # the members of a group must run together, also while three other
    # launches hold the compute units of one partly placed group each
    for n in ORDERS:
        for nk in (1, 2, 7, 16, 64, 1000):
            for nb in (8, 32, 64):
                order, rt, kc, members = plan(n, nb, nk, units)
                assert 1 <= order <= n and (order <= 128 or members > 0)
                if members:
                    assert 4 * members <= units, (n, nk, nb, order, members)
                    assert order <= 128 * rt and 16 * members * kc >= order


def test_whole_gpu_uses_every_shape(plan):
    # 256 compute units: the largest groups have 64 members, and few problems
    # take the narrowest share
    assert plan(1024, 32, 1, 256) == (1024, 8, 1, 64)
    assert plan(2000, 32, 1, 256) == (1008, 8, 1, 63)
    seen = {plan(n, 32, nk, 256)[1:3] for n in range(161, 1025, 9) for nk in range(1, 65)}
    assert seen >= {(2, 1), (2, 2), (2, 4), (3, 1), (3, 2), (3, 3), (4, 1), (4, 2), (5, 1), (5, 2), (6, 1), (8, 1)}
