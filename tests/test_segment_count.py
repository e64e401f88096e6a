"""The number of segments a column is cut into (host logic of the launcher, called
in the built library; no GPU)."""
import ctypes
import os

import pytest

from paper_2512_08571_amd import fehx


@pytest.fixture(scope="module")
def count():
    if not os.path.exists(fehx.LIB_PATH):
        pytest.skip("library not built")
    i32, i64 = ctypes.c_int, ctypes.c_int64
    f = getattr(fehx.lib(), "_ZN4fehx13segment_countEPKiilliilPd")
    f.restype = i32
    f.argtypes = [ctypes.POINTER(i32), i32, i64, i64, i32, i32, i64, ctypes.POINTER(ctypes.c_double)]

    def call(cols, cells, tiles, units, per_unit, cap):
        off = [0]
        for c in cols:
            off.append(off[-1] + c)
        return f((i32 * len(off))(*off), len(cols), cells, tiles, units, per_unit, cap, None)
    return call


@pytest.mark.parametrize("per_unit", [0, 1, 2, 8])
@pytest.mark.parametrize("cols", [[4, 4, 4, 4], [9, 3, 3, 1], [1]])
@pytest.mark.parametrize("tiles", [1, 7, 100000])
def test_range_and_no_resident_block(count, cols, tiles, per_unit):
    """An occupancy query that answers none counts as one unit's worth of work."""
    for cells in (2, 3, 16, 70000):
        for cap in (0, 1, 5, 1 << 40):
            n = count(cols, cells, tiles, 256, per_unit, cap)
            assert 1 <= n <= max(1, min(cells, cap, 2048))
            assert n * cells < 1 << 32
            if per_unit == 0:
                assert n == count(cols, cells, tiles, 256, 1, cap)


def test_small_launches_are_cut_and_full_ones_whole(count):
    assert count([4] * 4, 16, 1, 1024, 2, 1 << 40) == 16
    assert count([64] * 4, 16, 32, 1024, 2, 1 << 40) == 1


def test_nodes_past_the_grid_stay_whole():
    """The planes at the cuts are formed by a grid with the nodes along a_1 as its y, at most 65535."""
    if not os.path.exists(fehx.LIB_PATH):
        pytest.skip("library not built")
    f = getattr(fehx.lib(), "_ZN4fehx19plane_segment_countEPKNS_4MeshEiibilPd")
    f.restype = ctypes.c_int
    f.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_int, ctypes.c_bool, ctypes.c_int, ctypes.c_int64, ctypes.c_void_p]
    for n1, whole in ((1024, False), (32768, True)):
        m = fehx.Mesh([[2, 0, 0], [0, n1, 0], [0, 0, 4]], (2, n1, 4), 2, 3, (0, 0, 0), device=-1)
        assert (f(m._h, 3, 1, True, 1, 1 << 30, None) == 1) == whole
        m.close()
