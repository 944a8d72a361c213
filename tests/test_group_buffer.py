"""The buffer of the last level's grouping (rs_group.hip) holds all its parts: the
sort's temporary storage, the last of them, ends inside it."""
import ctypes
import os

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2010_08423_amd", "librestless_sieve.so")


class View(ctypes.Structure):
    _fields_ = [(f, ctypes.c_uint64) for f in ("key_in", "key_out", "idx_in", "idx_out", "head", "gid", "gstart", "ghi", "glo",
                                               "gq", "gcount", "temp")]


@pytest.mark.parametrize("kq", [4, 8, 12, 16])
def test_parts_end_inside_the_buffer(kq):
    lib = ctypes.CDLL(LIB)
    size, temp, view = lib._ZN2rs11group_bytesEmmj, lib._ZN2rs16group_temp_bytesEmm, lib._ZN2rs10group_viewEPhmj
    size.restype = temp.restype = ctypes.c_uint64
    size.argtypes = [ctypes.c_uint64, ctypes.c_uint64, ctypes.c_uint32]
    temp.argtypes = [ctypes.c_uint64, ctypes.c_uint64]
    view.restype, view.argtypes = View, [ctypes.c_uint64, ctypes.c_uint64, ctypes.c_uint32]
    for m in (1, 63, 64, 65, 654, 667, 1023, 4097, 10**6 + 1, 10**7):
        v = view(1 << 20, m, kq)
        at = [getattr(v, f) for f, _ in View._fields_]
        e = m + 64
        parts = [8 * e, 8 * e] + [4 * e] * 4 + [4 * (e + 1), 4 * e, 4 * e, 8 * e * kq, 4, temp(m, m // 10)]
        for a, b, after in zip(at, parts, at[1:] + [(1 << 20) + size(m, m // 10, kq)]):
            assert a % 256 == 0 and a + b <= after, (m, kq)
