"""The exchange of a long 1D line between workgroups (host only): whoever reads a field takes part in publishing the
other one, so no value is replaced before every workgroup has read it."""
import ctypes

from paper_2005_00322_amd import load_library


def test_every_workgroup_owns_words_of_both_fields():
    lib = load_library()
    w, rows, words = ctypes.c_int32(), ctypes.c_int32(), ctypes.c_int32()
    for n in range(129, 1366):
        assert lib.pstd_test_line_shape(n, ctypes.byref(w), ctypes.byref(rows), ctypes.byref(words)) == 0
        assert (w.value - 1) * rows.value < n <= w.value * rows.value         # rows of p
        assert (w.value - 1) * rows.value < words.value <= n, n               # words of u, within the buffer of n
