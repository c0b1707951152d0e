"""An operator's images (MFMA fragments, rows) are formed piece by piece: every entry and all padding, at any piece size, and
no piece larger than it may be."""
import ctypes

import numpy as np
import pytest


def _images(M, K, images):
    """The images' layout: index of entry (i, k) in each, and their size."""
    Mp, Kp = -(-M // 128) * 128, -(-K // 64) * 64
    i, k = np.arange(M)[:, None], np.arange(K)[None, :]
    frag = ((i >> 4) * (Kp >> 4) + (k >> 4)) * 256 + 4 * ((i & 15) + 16 * (k & 3)) + ((k & 15) >> 2)
    return [frag, i * Kp + k][:images], Mp * Kp


@pytest.mark.parametrize("dtype", [np.float32, np.float64])
@pytest.mark.parametrize("M,K,images,cap", [(2, 3, 2, 0), (15, 16, 2, 1), (16, 17, 2, 1024), (127, 128, 1, 5000), (129, 128, 2, 1),
                                            (300, 299, 1, 20480), (700, 701, 2, 0), (1500, 1499, 1, 0), (1364, 1365, 2, 0)])
def test_images_by_pieces(M, K, images, cap, dtype):
    from paper_2005_00322_amd import load_library

    lib = load_library()
    m = np.random.default_rng(M + K).standard_normal((M, K))
    index, cnt = _images(M, K, images)
    out = np.full(images * cnt, np.nan, dtype)
    largest = ctypes.c_int64()
    V = ctypes.c_void_p
    status = lib.pstd_test_operator_images(M, K, V(m.ctypes.data), ctypes.c_double(0.3), int(dtype is np.float64), images,
                                           ctypes.c_int64(cap), V(out.ctypes.data), ctypes.byref(largest))
    assert status == 0
    want = np.zeros_like(out)
    for n, at in enumerate(index):
        want[n * cnt + at] = (0.3 * m).astype(dtype)
    assert np.array_equal(out, want)
    assert largest.value <= max(cap or (4 << 20) // out.itemsize, 16 * -(-K // 64) * 64)
