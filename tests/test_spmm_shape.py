"""Host rules of the SpMM's layout, read from the built library (no GPU): lanes per neighbour group and feature tiles by the operand's width
and alignment."""
import ctypes as C
import os

import pytest


class Shape(C.Structure):
    _fields_ = [("vec", C.c_int), ("lpg", C.c_int), ("n_tiles", C.c_int), ("f_carry", C.c_int)]


@pytest.fixture(scope="module")
def shape():
    from paper_2306_15155_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2306_15155_amd import build
        build.build()
    fn = C.CDLL(binding.LIB_PATH)["_ZN6sensei10spmm_shapeEPKfli"]   # spmm_shape(const float *B, int64_t ldb, int f); B is not read
    fn.restype, fn.argtypes = Shape, [C.c_void_p, C.c_int64, C.c_int]

    def call(f, ld=None, addr=0x1000):
        s = fn(addr, f if ld is None else ld, f)
        assert s.n_tiles * s.lpg * s.vec == s.f_carry and s.f_carry >= f and (s.n_tiles - 1) * s.lpg * s.vec < f
        return s
    return call


# a group no wider than twice what the row fills: a group of 32 lanes on a one-column operand has one lane at work and two neighbours per step
@pytest.mark.parametrize("f,ld,vec,lpg", [(1, 1, 1, 8), (3, 3, 1, 8), (7, 7, 1, 8), (8, 9, 1, 8), (9, 9, 1, 16), (16, 17, 1, 16), (17, 17, 1, 32),
                                          (2, 2, 2, 8), (10, 10, 2, 8), (16, 18, 2, 8), (18, 18, 2, 16), (32, 34, 2, 16), (4, 4, 4, 8), (32, 32, 4, 8)])
def test_narrow_rows_take_narrow_groups(shape, f, ld, vec, lpg):
    s = shape(f, ld)
    assert (s.vec, s.lpg, s.n_tiles) == (vec, lpg, 1)


# every tile walks the pattern again: at most 32 of them until a group is a whole wavefront
@pytest.mark.parametrize("f,vec,lpg,tiles", [(1024, 4, 8, 32), (1028, 4, 16, 17), (2048, 4, 16, 32), (4096, 4, 32, 32), (8192, 4, 64, 32), (16384, 4, 64, 64),
                                             (4098, 2, 64, 33), (4097, 1, 64, 65)])
def test_wide_rows_take_wide_groups(shape, f, vec, lpg, tiles):
    s = shape(f)
    assert (s.vec, s.lpg, s.n_tiles) == (vec, lpg, tiles)
