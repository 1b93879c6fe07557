"""The order that the index keeps its centroids in (C++ functions of
libchimera.so, no GPU): the operand order against its definition, and back."""
import ctypes

import numpy as np
import pytest

from paper_2608_23553_amd import chimera


@pytest.mark.parametrize("ncent", [1, 31, 32, 33, 257])
def test_operand_order_and_back(ncent):
    L = chimera.lib()
    size = L._ZN7chimera18probe_operand_sizeEi
    size.restype = ctypes.c_int64
    cent = np.random.default_rng(ncent).integers(0, 65536, (ncent, 128)).astype(np.uint16)
    op = np.zeros(size(ncent), np.uint16)
    L._ZN7chimera13probe_operandEPKtiPt(cent.ctypes.data_as(ctypes.c_void_p), ncent, op.ctypes.data_as(ctypes.c_void_p))
    # element i of lane l in step s of tile t: dimension 64 (l / 32) + 8 s + i of centroid 32 t + l % 32
    tiles = -(-ncent // 32)
    rows = np.minimum(np.arange(32 * tiles), ncent - 1)
    want = cent[rows].reshape(tiles, 32, 2, 8, 8).transpose(0, 3, 2, 1, 4)
    assert np.array_equal(op, want.ravel())
    back = np.zeros_like(cent)
    L._ZN7chimera10probe_rowsEPKtiPt(op.ctypes.data_as(ctypes.c_void_p), ncent, back.ctypes.data_as(ctypes.c_void_p))
    assert np.array_equal(back, cent)
