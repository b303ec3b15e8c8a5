"""The cost model prices a call on the path it takes: with a dense-tile split attached, an aggregation whose padded width reaches the split's
narrowest gets cheaper and a narrower one does not.  The operand is slice-major there, so 33 columns count as 64."""
import pytest

import synth
from paper_2306_15155_amd import KIND_GAT, KIND_GCN, SELECT_MODEL, Context, Tiles, binding, csr_struct

from gpu_util import DeviceCSR

pytestmark = pytest.mark.gpu

DYNF_UPD, REUSE = 3, 0


@pytest.fixture(scope="module")
def split():
    ctx = Context(0)
    g = synth.rmat(52, 6000, 400_000)
    A = DeviceCSR(g)
    T = Tiles(ctx, A.s, 0.05, 256)   # narrowest: 64 columns, 32 for the attention aggregation
    assert T.nnz_dense > 0.3 * g.row_ptr[-1]
    yield ctx, A, csr_struct(g.n_rows, g.n_cols, A.row_ptr, A.col_idx, tiles=T)
    T.close()
    ctx.close()


@pytest.mark.parametrize("f,split_taken", [(16, False), (32, False), (33, True), (41, True), (63, True), (64, True), (96, True), (256, True), (257, False)])
def test_gcn(split, f, split_taken):
    ctx, A, At = split
    plain, tiled = (ctx.select(KIND_GCN, a, 300, f, SELECT_MODEL)[1][DYNF_UPD] for a in (A.s, At))
    assert (tiled < 0.95 * plain) == split_taken, (plain, tiled)


@pytest.mark.parametrize("f", [20, 32, 41, 256])
def test_gat(split, f):
    ctx, A, At = split
    assert binding.gat_attention_path(At, 300, f, REUSE) == binding.GAT_PATH_TILES
    plain, tiled = (ctx.select(KIND_GAT, a, 300, f, SELECT_MODEL)[1][REUSE] for a in (A.s, At))
    # a split leaves no one-walk form: where there was one, its second pass over the pattern is priced too
    assert tiled < plain or binding.gat_attention_path(A.s, 300, f, REUSE) == binding.GAT_PATH_ONE_WALK
