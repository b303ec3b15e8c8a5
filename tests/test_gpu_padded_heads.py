"""Forward attention of heads whose columns do not begin at a multiple of four: side by side, or padded to slices of their own in Theta, as many at a time as it has room
for.  Batches with one left over, heads of one slice and of two, rows long enough for the one-walk form and not, with a dense-tile split, against
the oracle at the parity tolerance per element (fp32 sums of at most a few thousand terms of order one)."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2306_15155_amd import ACT_NONE, ACT_RELU, Context, Tiles, binding, csr_struct

from gpu_util import DEV, DeviceCSR, assert_close, dev, hub_and_empty_graph, rect_block

pytestmark = pytest.mark.gpu

PATTERNS = {"long": lambda: synth.rmat(5, 2_000, 60_000), "short": lambda: synth.rmat(6, 4_000, 16_000), "hub": lambda: hub_and_empty_graph(3, 900, 5_000, 700, 40),
            "rect": lambda: rect_block(4, 260, 900, 20), "large": lambda: synth.rmat(9, 8_000, 110_000)}


@pytest.fixture(scope="module")
def ctx():
    c = Context(0)
    yield c
    c.close()


def _inputs(g, heads, d):
    X, W = synth.uniform(7, 1, (g.n_cols, 36), -0.5, 0.5), synth.glorot(7, 2, 36, heads * d)
    return X, W, synth.normal(7, 3, (heads * d,), 0.0, 0.3), synth.normal(7, 4, (heads * d,), 0.0, 0.3)


# 2 x 14: Theta holds one padded head; 4 x 23: three and one; 17 x 3: two and a last one; 3 x 37: two slices a head, two heads and one; 20 x 31: more than one launch takes
@pytest.mark.parametrize("name", PATTERNS)
@pytest.mark.parametrize("heads,d", [(2, 1), (2, 14), (4, 23), (17, 3), (3, 37), (20, 31)])
def test_heads(ctx, name, heads, d):
    g = PATTERNS[name]()
    A, (X, W, a_l, a_r) = DeviceCSR(g), _inputs(g, heads, d)
    for act, comp in ((ACT_RELU, 0), (ACT_NONE, 3)):
        want = oracle.gat_layer_heads(g.n_rows, g.n_cols, g.row_ptr, g.col_idx, X, W, a_l, a_r, heads, 0.2, act)
        assert_close(ctx.gat_layer_heads(A.s, dev(X), dev(W), dev(a_l), dev(a_r), heads, comp, 0.2, act), want, what=f"comp {comp}")


def test_with_tiles(ctx):
    g = synth.rmat(8, 3_000, 300_000)
    heads, d = 2, 37
    row_ptr, col_idx = dev(g.row_ptr), dev(g.col_idx)
    tiles = Tiles(ctx, csr_struct(g.n_rows, g.n_cols, row_ptr, col_idx), 0.05, 128)
    At = csr_struct(g.n_rows, g.n_cols, row_ptr, col_idx, tiles=tiles)
    assert tiles.n_tiles > 0 and binding.gat_attention_path(At, 36, heads * d, 0, heads) == binding.GAT_PATH_TILES
    X, W, a_l, a_r = _inputs(g, heads, d)
    want = oracle.gat_layer_heads(g.n_rows, g.n_cols, g.row_ptr, g.col_idx, X, W, a_l, a_r, heads, 0.2, ACT_RELU)
    for comp in (0, 3):
        assert_close(ctx.gat_layer_heads(At, dev(X), dev(W), dev(a_l), dev(a_r), heads, comp, 0.2, ACT_RELU), want, what=f"comp {comp}")


# scratch of exactly the size that the query asks for, full of NaN before: W with its padding and the vectors of several heads lie in pieces of it that
# other forms use
@pytest.mark.parametrize("name", ["long", "short", "rect", "large"])
@pytest.mark.parametrize("heads,d,f_in", [(2, 1, 36), (8, 15, 36), (4, 23, 36), (20, 31, 36), (3, 37, 36), (32, 3, 36), (5, 7, 900)])
def test_scratch(ctx, name, heads, d, f_in):
    g = PATTERNS[name]()
    A = DeviceCSR(g)
    X, W = dev(synth.uniform(7, 1, (g.n_cols, f_in), -0.5, 0.5)), dev(synth.glorot(7, 2, f_in, heads * d))
    a_l, a_r = dev(synth.normal(7, 3, (heads * d,), 0.0, 0.3)), dev(synth.normal(7, 4, (heads * d,), 0.0, 0.3))
    want = oracle.gat_layer_heads(g.n_rows, g.n_cols, g.row_ptr, g.col_idx, X.cpu().numpy(), W.cpu().numpy(), a_l.cpu().numpy(), a_r.cpu().numpy(), heads, 0.2,
                                  ACT_NONE)
    for comp in (0, 3):
        need = ctx.gat_workspace(A.s, f_in, heads * d, comp)
        room = torch.full((need + 1024,), 0xFF, dtype=torch.uint8, device=DEV)
        at = -room.data_ptr() % 256
        Y = torch.empty(g.n_rows, heads * d, device=DEV)
        binding._check(binding.lib().sensei_gat_layer_heads(ctx._h, ctypes.byref(A.s), binding.mat_struct(X), binding.mat_struct(W), a_l.data_ptr(), a_r.data_ptr(), heads, 0.2,
                                                            Y.data_ptr(), heads * d, ACT_NONE, comp, room.data_ptr() + at, need, binding._stream()), "sensei_gat_layer_heads")
        assert_close(Y, want, what=f"comp {comp}")
        assert bool((room[:at] == 0xFF).all()) and bool((room[at + need:] == 0xFF).all())


# How many products there are says which form a call took.  Products over a wide X cost more than padding saves where rows are short or the heads narrow, and where
# there are few entries at all.
@pytest.mark.parametrize("n,per_row,f_in,heads,d,products", [
    (60_000, 4, 600, 8, 3, 1), (60_000, 4, 600, 8, 5, 1), (60_000, 4, 600, 17, 3, 1), (60_000, 4, 600, 8, 1, 1), (20_000, 10, 600, 2, 14, 1), (3_000, 40, 36, 2, 14, 1),
    (60_000, 4, 16, 4, 23, 2), (60_000, 20, 36, 17, 3, 9), (20_000, 60, 100, 8, 15, 2), (20_000, 60, 100, 2, 37, 2), (20_000, 60, 100, 3, 37, 2), (30_000, 18, 36, 4, 7, 4)])
def test_products_over_the_input(ctx, n, per_row, f_in, heads, d, products):
    g = rect_block(n, n, n, per_row)
    A, X, W = DeviceCSR(g), synth.uniform(7, 1, (n, f_in), -0.5, 0.5), synth.glorot(7, 2, f_in, heads * d)
    a_l, a_r = synth.normal(7, 3, (heads * d,), 0.0, 0.3), synth.normal(7, 4, (heads * d,), 0.0, 0.3)
    args = (A.s, dev(X), dev(W), dev(a_l), dev(a_r), heads)
    for comp in (0, 3):
        ctx.profile_enable(True)
        Y = ctx.gat_layer_heads(*args, comp, 0.2, ACT_NONE)
        torch.cuda.synchronize()
        count = len(ctx.profile_read(1))
        ctx.profile_enable(False)
        assert count == products, f"comp {comp}"
        rows = np.random.default_rng(d).integers(0, n, 200)
        want = np.empty((rows.size, heads * d))
        for k, i in enumerate(rows):
            want[k] = _row(g, X, W, a_l, a_r, heads, d, i)
        assert_close(Y[torch.from_numpy(rows).cuda()], want, what=f"comp {comp}")


def _row(g, X, W, a_l, a_r, heads, d, i):
    """One row of the layer in fp64."""
    j = np.concatenate([[i], g.col_idx[g.row_ptr[i]:g.row_ptr[i + 1]]])
    theta = (X[j].astype(np.float64) @ W.astype(np.float64)).reshape(j.size, heads, d)
    s_l, s_r = (theta[0] * a_l.reshape(heads, d)).sum(1), (theta[1:] * a_r.reshape(heads, d)).sum(2)
    e = s_l + s_r
    e = np.where(e > 0, e, 0.2 * e)
    p = np.exp(e - e.max(0))
    return ((p / p.sum(0))[:, :, None] * theta[1:]).sum(0).reshape(-1)
