"""Row tiling of the split-bf16 contractions (host only): every row block of every operator length is computed once."""
import ctypes

import numpy as np
import pytest

from paper_2005_00322_amd import load_library


@pytest.mark.parametrize("lines", [1, 64, 65, 1000, 5440, 5441, 5476, 8192, 16384, 40000, 1000000])
def test_every_row_block_is_taken_once(lines):
    lib = load_library()
    lib.pstd_test_split_blocks.argtypes = [ctypes.c_int32, ctypes.c_int64, ctypes.POINTER(ctypes.c_int32)]
    for rows in range(1, 8194):          # past the longest dense axis (4097 nodes)
        blocks = (rows + 31) // 32
        if rows % 32 not in (0, 1):      # the rule sees only the count of row blocks: its first and last row
            continue
        taken = np.full(blocks, -1, np.int32)
        assert lib.pstd_test_split_blocks(rows, lines, taken.ctypes.data_as(ctypes.POINTER(ctypes.c_int32))) == 0, rows
        assert (taken == 1).all(), (rows, np.flatnonzero(taken != 1))
