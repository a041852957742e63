"""Grids of the halo fills' captured launches (host arithmetic only).  A step graph is kept
for every tree with its key, so the grid of a list of items must not depend on anything but the
list's size class, which the key holds, and must give every item of the class its workgroup."""
import ctypes as C

import pytest

from paper_2012_04385_amd import build, mrfv

MISSING, RHO_E, ITEMS = 2, 4, 16


class _Grid(C.Structure):
    _fields_ = [("x", C.c_int), ("y", C.c_int), ("z", C.c_int)]


@pytest.fixture(scope="module")
def fill_grid():
    import os
    if not os.path.exists(mrfv.LIB_PATH):
        build.build()
    f = mrfv.lib()._ZN4mrfv9fill_gridEiiib
    f.restype, f.argtypes = _Grid, [C.c_int, C.c_int, C.c_int, C.c_bool]
    return lambda *a: (lambda g: (g.x, g.y, g.z))(f(*a))


@pytest.mark.parametrize("mode", [ITEMS, ITEMS | RHO_E])
def test_captured_items_depend_on_their_class(fill_grid, mode):
    ends = [64, 256, 819, 1 << 20]
    bound, lo = 4096, 1
    for end in ends:
        grids = {fill_grid(n, bound, mode, True) for n in {lo, lo + 1, (lo + min(end, 9000)) // 2, min(end, 9000)}}
        assert len(grids) == 1, (lo, end, grids)
        x, y, z = grids.pop()
        assert y == 1 and x >= min(end, bound)                    # an item each, up to the bound
        if end <= 819:                                              # split as an eager launch is
            assert z == fill_grid(end, end, mode, False)[2] > 1
            assert x * 5 <= 4096 + 5 * 8                            # and no surplus beyond the split's
        lo = end + 1
    assert fill_grid(10, 40, mode, True)[0] == 40                   # never beyond the bound (in XCDs)


@pytest.mark.parametrize("mode", [0, RHO_E, MISSING, MISSING | RHO_E])
def test_captured_block_lists_fill_the_card(fill_grid, mode):
    """Lists of blocks: whatever the count at capture, the workgroups a grown list gets."""
    for n in (1, 10, 64, 65, 200, 1000, 5000):
        x, y, z = fill_grid(n, 1024, mode, True)
        assert x * y * z >= 2048, (n, x, y, z)
