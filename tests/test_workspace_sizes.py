"""Workspace sizes that need no GPU to be asked for."""
import ctypes

import pytest

import paper_1906_07102_amd as lmg


def batch_bytes(N, nchan, nvis, prec):
    n = ctypes.c_size_t()
    assert lmg.load().lmg_batch_workspace_size(N, 7, nchan, nvis, prec, ctypes.byref(n)) == 0
    return n.value


@pytest.mark.parametrize("prec,work_items", [(lmg.F32, 1), (lmg.F32_KAHAN, 5), (lmg.F64, 5)])
def test_work_items_of_quadrants_only_where_there_are_any(prec, work_items):
    """A channel of an 8192^2 batch holds its 16,384 tiles' counts, offsets and items (16 bytes each), and four more items
    per tile in the modes that grid by quadrants: plain FP32 does not."""
    a, b = batch_bytes(8192, 8, 1 << 24, prec), batch_bytes(8192, 9, 1 << 24, prec)
    tiles = 16384
    least = tiles * (16 * work_items + 12)
    assert least <= b - a < least + tiles * 12
