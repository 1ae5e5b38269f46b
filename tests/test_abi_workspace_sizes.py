"""The g-matrix call's workspace stays what programs that keep one have always had to
bring: 44 spinor blocks and small buffers, on grids from one point to the double dot's."""

import ctypes as C

import pytest

SIZES = {(1, 1, 8): 76544, (2, 3, 5): 170496, (10, 8, 8): 2869248, (24, 8, 8): 6851840,
         (40, 14, 12): 29958144, (75, 31, 29): 300317696, (256, 48, 48): 2583178240}


@pytest.mark.parametrize("shape", SIZES, ids=["x".join(map(str, s)) for s in SIZES])
def test_gmatrix_workspace(shape):
    from paper_2607_08447_amd import _lib as L
    g = L.hkp_grid(*shape, 0.4)
    assert L.lib.hkp_gmatrix_workspace_bytes(C.byref(g)) == SIZES[shape]
