"""Host-only checks of the choice among the rotated smoothing kernel's forms."""
import ctypes

import pytest

import paper_1609_03782_amd as ig

LDS = 160 * 1024


def _form(r, shape=(200, 200, 200), ncu=256):
    nz, ny, nx = shape
    return ig.lib().ig_debug_dense_form((ctypes.c_int32 * 3)(*r), nx, ny, nz, ncu)


def _tile(r, planes=8):
    """LDS of the plain tile of 64 x 4 voxels by `planes`, with the weights."""
    rx, ry, rz = r
    return 4 * ((2 * rx + 1) * (2 * ry + 1) * (2 * rz + 1) + (64 + 2 * rx) * (4 + 2 * ry) * (planes + 2 * rz)) + 256


@pytest.mark.parametrize("shape", [(200, 200, 200), (5, 3, 40), (300, 400, 500)])
def test_column_form_wherever_its_plain_tile_fits(shape):
    """Every kernel of z half-width 1 to 8 whose plain tile fits a compute unit runs in
    columns, also where padding and the sums' table would not fit."""
    lean = 0
    for rz in range(1, 9):
        for rx in range(0, 40):
            for ry in range(0, 40):
                r = (rx, ry, rz)
                if _tile(r) > LDS:
                    assert _form(r, shape) <= 0
                    continue
                assert _form(r, shape) in (1, 2, 3), r
                lean += _form(r, shape) == 3
    assert lean > 200
    for r in ((8, 8, 7), (9, 9, 6), (11, 11, 4), (12, 12, 3)):
        assert _form(r, shape) == 3
    assert _form((4, 4, 0)) == 0 and _form((2, 2, 9)) == 0


def test_two_rows_where_the_gpu_is_full():
    assert _form((4, 3, 4), (290, 350, 360)) == 2
    assert _form((4, 3, 4), (16, 16, 128)) == 1
