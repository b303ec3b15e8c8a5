"""Scratch that the queries ask for, on sizes alone: buffers that callers sized by these figures stay large enough."""
import ctypes

import pytest

from paper_2306_15155_amd import binding
from paper_2306_15155_amd.binding import CsrStruct


def _csr(n_rows, n_cols, nnz):
    A = CsrStruct()
    A.n_rows, A.n_cols, A.nnz, A.row_ptr, A.col_idx = n_rows, n_cols, nnz, 256, 256   # the queries read no entry
    return A


# single heads and several (the query does not know how many), widths that are no multiple of a slice, wide inputs on small patterns
@pytest.mark.parametrize("n_rows,n_cols,nnz,f_in,f_out,comp,most", [
    (2_400_000, 2_400_000, 9_600_000, 128, 250, 0, 2_573_026_560), (100_000, 100_000, 2_100_000, 128, 100, 0, 67_552_256),
    (100_000, 100_000, 2_100_000, 128, 100, 3, 67_552_256), (233_000, 233_000, 115_000_000, 602, 41, 0, 813_578_240),
    (1_000, 5_000, 20_000, 1433, 120, 0, 3_185_408), (1_000, 5_000, 20_000, 1433, 120, 3, 3_185_408),
    (100_000, 100_000, 2_100_000, 128, 128, 0, 74_083_840), (0, 0, 0, 16, 33, 0, 3_072)])
def test_gat_layer(n_rows, n_cols, nnz, f_in, f_out, comp, most):
    need = ctypes.c_size_t()
    assert binding.lib().sensei_gat_workspace(ctypes.byref(_csr(n_rows, n_cols, nnz)), f_in, f_out, comp, ctypes.byref(need)) == 0
    assert need.value <= most


# many narrow heads on long rows, where the walks' own chunks would take more than there was room for; 4 heads of a slice on ordinary rows
@pytest.mark.parametrize("n_rows,n_cols,nnz,f_in,f_out,heads,most", [
    (40_571, 40_571, 14_892_209, 8, 34, 17, 292_005_632), (20_000, 60_000, 9_000_000, 36, 384, 16, 364_032_256),
    (50_000, 50_000, 30_000_000, 64, 512, 16, 734_928_640), (100_000, 100_000, 2_100_000, 128, 128, 4, 271_493_376)])
def test_gat_backward_heads(n_rows, n_cols, nnz, f_in, f_out, heads, most):
    need = ctypes.c_size_t()
    A, At = _csr(n_rows, n_cols, nnz), _csr(n_cols, n_rows, nnz)
    assert binding.lib().sensei_gat_backward_heads_workspace(ctypes.byref(A), ctypes.byref(At), f_in, f_out, heads, ctypes.byref(need)) == 0
    assert need.value <= most


# the slabs of a weight gradient of 144, 96 and 324 blocks: at least as many as fill three quarters of the rounds that they take, no more than there was room for
@pytest.mark.parametrize("n,f_in,f_out,least,most", [(50_000, 1433, 1433, 643_000_000, 692_632_832), (20_000, 1433, 1000, 231_000_000, 265_786_624),
                                                     (20_000, 2300, 2300, 529_000_000, 529_250_816), (233_000, 602, 256, 0, 512_369_408)])
def test_gcn_backward(n, f_in, f_out, least, most):
    need = ctypes.c_size_t()
    assert binding.lib().sensei_gcn_backward_workspace(ctypes.byref(_csr(n, n, 4 * n)), f_in, f_out, 0, ctypes.byref(need)) == 0
    assert least <= need.value <= most


# The weight gradients of a layer are formed one after the other in the same slabs.  The one of fewer columns (keys of 64, values of 114), or over fewer rows (sampled
# blocks), may take the larger ones.
@pytest.mark.parametrize("n_rows,n_cols,nnz,f_in,d_k,f_out,least,most", [
    (207_936, 207_936, 770_000, 576, 64, 114, 570_136_576, 620_953_600), (3_000, 100_000, 60_000, 700, 128, 130, 311_209_984, 324_112_384),
    (6_000, 6_000, 40_000, 300, 128, 129, 51_480_320, 54_470_912)])
def test_dotgat_backward(n_rows, n_cols, nnz, f_in, d_k, f_out, least, most):
    need = ctypes.c_size_t()
    assert binding.lib().sensei_dotgat_backward_workspace(ctypes.byref(_csr(n_rows, n_cols, nnz)), f_in, d_k, f_out, ctypes.byref(need)) == 0
    assert least <= need.value <= most


@pytest.mark.parametrize("n_rows,n_cols,nnz,f_in,f_out,least,most", [(4_000, 100_000, 60_000, 700, 400, 586_574_336, 586_574_336),
                                                                     (3_000, 6_000, 40_000, 700, 300, 111_214_336, 112_894_208)])
def test_gatv2_backward(n_rows, n_cols, nnz, f_in, f_out, least, most):
    need = ctypes.c_size_t()
    assert binding.lib().sensei_gatv2_backward_workspace(ctypes.byref(_csr(n_rows, n_cols, nnz)), f_in, f_out, ctypes.byref(need)) == 0
    assert least <= need.value <= most
