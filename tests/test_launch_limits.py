"""CPU check of the exact passes' launches: a launch has fewer than 2^32 threads, so
more workgroups of 256 than that are taken in parts, up to the largest clouds that
the entry points accept."""

import ctypes
import math

import pytest


class Geom(ctypes.Structure):
    _fields_ = [("blocks", ctypes.c_int64), ("chunk", ctypes.c_int64),
                ("nchunk", ctypes.c_int32)]


@pytest.fixture(scope="module")
def fns():
    import paper_2307_03043_amd as ch
    lib = ctypes.CDLL(ch.lib()._name)
    i64, i32 = ctypes.c_int64, ctypes.c_int32

    def fn(name, res, args):
        f = getattr(lib, name)
        f.restype, f.argtypes = res, args
        return f

    half = fn("_ZN7chamfer9half_geomEllil", Geom, [i64, i64, i32, i64])
    sad = fn("_ZN7chamfer8sad_geomEllilRi", Geom, [i64, i64, i32, i64, ctypes.POINTER(i32)])
    return {
        "half": (lambda nx, nb, d: half(nx, nb, d, 0),
                 fn("_ZN7chamfer19half_launch_queriesElli", i64, [i64, i64, i32])),
        "sad": (lambda nx, nb, d: sad(nx, nb, d, 0, ctypes.byref(i32())),
                fn("_ZN7chamfer18sad_launch_queriesElli", i64, [i64, i64, i32])),
    }


LARGEST = 2 ** 31 - 1


@pytest.mark.parametrize("form,d", [("half", 1), ("half", 3), ("half", 12), ("half", 128),
                                    ("half", 256), ("sad", 9), ("sad", 100), ("sad", 256)])
@pytest.mark.parametrize("n_x,n_b", [(1, LARGEST), (1000, LARGEST), (1_000_000, 1_000_000),
                                     (20_000_000, 20_000_000), (40_000_000, 30_000_000),
                                     (LARGEST, 1000), (LARGEST, LARGEST)])
def test_launches(fns, form, d, n_x, n_b):
    geom, queries = fns[form]
    part = queries(n_x, n_b, d)
    assert 1 <= part <= n_x
    assert n_x / part < 2 ** 20  # still launches of many workgroups
    sizes = {part, n_x % part or part}
    for n in sizes:
        n = queries(n, n_b, d)
        g = geom(n, n_b, d)
        assert g.blocks * 256 < 2 ** 32
        assert g.chunk * g.nchunk >= n_b and g.chunk <= 65536
        assert g.blocks % g.nchunk == 0 and g.blocks >= g.nchunk
    if n_x * n_b <= 10 ** 12:
        assert part == n_x  # ordinary calls: one launch
    assert math.ceil(n_x / part) * part >= n_x
