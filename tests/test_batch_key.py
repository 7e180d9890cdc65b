"""The options' part of a batch graph's key (host code of the library): equal
for equal options whatever the stack held before, different for different
ones."""
import ctypes

import pytest


@pytest.fixture(scope="module")
def kg():
    from paper_1402_4247_amd import kgev
    return kgev


def key(kg, opts, dirt):
    f = kg.lib.kgev_internal_opts_key
    f.argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.c_void_p, ctypes.c_int32]
    words = (ctypes.c_uint64 * 64)()
    count = f(ctypes.byref(opts) if opts is not None else None, dirt, words, 64)
    return list(words[:count])


FIELDS = [dict(precision=1), dict(want_vectors=False), dict(panel_nb=16), dict(refine_iters=5), dict(s_tol=1e-9),
          dict(streams=2), dict(s_method=1), dict(hemv_slots=9), dict(gemm_slots=9),
          # the defaults by value: the same panels, but down to order 128
          dict(panel_nb=32)]


def test_equal_options_give_equal_keys(kg):
    for kw in [dict()] + FIELDS:
        opts = kg.make_opts(use_graph=True, **kw)
        keys = [key(kg, opts, dirt) for dirt in (0, 1, 2, 0x55, 0xff)]
        assert all(k == keys[0] for k in keys), kw
    assert key(kg, None, 1) == key(kg, kg.make_opts(), 2)


def test_different_options_give_different_keys(kg):
    keys = [tuple(key(kg, kg.make_opts(use_graph=True, **kw), 0)) for kw in [dict()] + FIELDS]
    assert len(set(keys)) == len(keys)
