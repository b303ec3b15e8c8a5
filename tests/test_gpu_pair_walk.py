"""The walks in which a group of four lanes keeps the vectors of the row it is in: rows that end with a group's part of a chunk, inside it, and with the chunk; rows of
one entry beside rows that take several parts; one slice and several, in one launch (small operands) and in launches of one slice.  Against the oracle
at the parity tolerance per element (fp32 sums of at most a few thousand terms of order one)."""
import numpy as np
import pytest

import oracle
import synth
from paper_2306_15155_amd import ACT_NONE, Context, binding

from gpu_util import DeviceCSR, assert_close, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = Context(0)
    yield c
    c.close()


def pattern(t, least, n_cols):
    """Rows whose ends meet the sixteenths of a chunk of t entries in every way, then rows of random lengths up to `least` entries."""
    part = t // 16
    head = [part] * 16 + [1] * (part - 1) + [part + 1] + [part - 1 or 1, 1] * 7 + [t, t + part, 1, 0, t - part, 3 * t + 1, 0] + [1] * t + [5 * part] * 5
    rng = np.random.default_rng(t)
    tail = rng.integers(0, 40, max(least - sum(head), 0) // 19 + 50)   # 19.5 on average
    lens = np.minimum(np.concatenate([head, tail]), n_cols).astype(np.int64)
    row_ptr = np.concatenate([[0], np.cumsum(lens)])
    row = np.repeat(np.arange(lens.size), lens)
    k = np.arange(row_ptr[-1]) - row_ptr[row]
    step = n_cols // np.maximum(lens[row], 1)
    col = k * step + (rng.random(k.size) * step).astype(np.int64)   # ascending and distinct: one column per `step`
    return synth.CSR(lens.size, max(n_cols, lens.size), row_ptr.astype(np.int32), col.astype(np.int32))


# (the walks of narrow heads have chunks of at most 256 entries)
@pytest.mark.parametrize("t,least", [(64, 3_000), (128, 140_000), (256, 270_000), (256, 530_000)])
@pytest.mark.parametrize("heads,d", [(2, 12), (1, 32)])
def test_narrow_heads(ctx, t, least, heads, d):
    g = pattern(t, least, 4_000)
    assert min(binding.chunk_nnz(g.nnz), 256) == t and g.nnz >= least
    X, W = synth.uniform(t, 1, (g.n_cols, 20), -0.5, 0.5), synth.glorot(t, 2, 20, heads * d)
    a_l, a_r = synth.normal(t, 3, (heads * d,), 0.0, 0.3), synth.normal(t, 4, (heads * d,), 0.0, 0.3)
    # every score well away from zero, where the derivative jumps: feature 0 is +-1 and only a_r sees it
    X[:, 0] = np.where(np.random.default_rng(t).random(g.n_cols) < 0.5, 1.0, -1.0)
    W[0, :], W[:, ::d] = 0.0, 0.0
    W[0, ::d], a_l[::d], a_r[::d] = 1.0, 0.0, 4.0
    dY = synth.normal(t, 5, (g.n_rows, heads * d))
    A, At = DeviceCSR(g), DeviceCSR(synth.transpose(g))
    want = oracle.gat_backward_heads(g.n_rows, g.n_cols, g.row_ptr, g.col_idx, X, W, a_l, a_r, heads, dY, slope=0.2)
    got = ctx.gat_backward_heads(A.s, At.s, ctx.transpose_positions(A.s, At.s), dev(X), dev(W), dev(a_l), dev(a_r), heads, dev(dY), neg_slope=0.2)
    for gpu, ref, what in zip(got, want, ("dX", "dW", "da_l", "da_r")):
        assert_close(gpu, ref, what=what)


# the dot products (keys of 40 columns, values of 33 to 96) and the scores behind them; 100,000 sources of 96 columns are past the size that one launch takes whole
@pytest.mark.parametrize("t,least,n_cols,f_out", [(64, 3_000, 4_000, 33), (128, 140_000, 4_000, 96), (256, 270_000, 100_000, 96), (512, 530_000, 4_000, 70),
                                                  (512, 530_000, 100_000, 96)])
def test_dots_and_scores(ctx, t, least, n_cols, f_out):
    g = pattern(t, least, n_cols)
    assert binding.chunk_nnz(g.nnz) == t
    f_in, d_k = 12, 40
    X = np.round(synth.uniform(t, 1, (g.n_cols, f_in), -1.0, 1.0) * 8) / 8   # on a grid: the projections are exact, the score's derivative jumps on both sides alike
    Wq, Wk, Wv = (np.round(synth.uniform(t, 2 + i, (f_in, w), -0.5, 0.5) * 16) / 16 for i, w in enumerate((d_k, d_k, f_out)))
    att = np.round(synth.normal(t, 6, (f_out,), 0.0, 0.2) * 64) / 64
    X, Wq, Wk, Wv, att = (a.astype(np.float32) for a in (X, Wq, Wk, Wv, att))
    dY = synth.normal(t, 7, (g.n_rows, f_out))
    A, At = DeviceCSR(g), DeviceCSR(synth.transpose(g))
    pos = ctx.transpose_positions(A.s, At.s)
    args = (g.n_rows, g.n_cols, g.row_ptr, g.col_idx, X)
    Y = ctx.dotgat_layer(A.s, dev(X), dev(Wq), dev(Wk), dev(Wv), 0.15, 0, ACT_NONE)
    assert_close(Y, oracle.dotgat_layer(*args, Wq, Wk, Wv, 0.15, ACT_NONE), what="key-query Y")
    want = oracle.dotgat_backward(*args, Wq, Wk, Wv, 0.15, dY)
    for gpu, ref, what in zip(ctx.dotgat_backward(A.s, At.s, pos, dev(X), dev(Wq), dev(Wk), dev(Wv), 0.15, dev(dY)), want, ("dX", "dW_q", "dW_k", "dW_v")):
        assert_close(gpu, ref, what="key-query " + what)
    Wl = np.roll(Wv, 1, axis=1)
    Y = ctx.gatv2_layer(A.s, dev(X), dev(Wl), dev(Wv), dev(att), 0, 0.25)
    assert_close(Y, oracle.gatv2_layer(*args, Wl, Wv, att, 0.25, ACT_NONE), what="GATv2 Y")
    want = oracle.gatv2_backward(*args, Wl, Wv, att, dY, slope=0.25)
    for gpu, ref, what in zip(ctx.gatv2_backward(A.s, At.s, pos, dev(X), dev(Wl), dev(Wv), dev(att), dev(dY), neg_slope=0.25), want, ("dX", "dW_l", "dW_r", "datt")):
        assert_close(gpu, ref, what="GATv2 " + what)


# Places behind the last entry of the pattern are walked with the last chunk: what is read there belongs to the chunk's first entry, and must reach no result
# also where it is no number.  Both the oracle and the call with zeros in its place say what the sources without a link to that destination get.
@pytest.mark.parametrize("bad", [np.inf, np.nan])
@pytest.mark.parametrize("n,per_row,heads,d", [(300, 9, 1, 32), (3_000, 50, 2, 20), (4_000, 75, 2, 32)])
def test_no_number_behind_the_last_entry(ctx, n, per_row, heads, d, bad):
    rng = np.random.default_rng(n)
    last = 40   # the last sources have three links each, so that the last chunk holds several
    dst = np.concatenate([np.repeat(np.arange(n), per_row), rng.integers(0, n, last * 3)])
    src = np.concatenate([rng.integers(0, n - last, n * per_row), np.repeat(np.arange(n - last, n), 3)])
    g = synth.build_csr(n, n, dst, src, False, False)
    gt = synth.transpose(g)
    t = min(binding.chunk_nnz(g.nnz), 256)
    assert g.nnz % t, "the last chunk is to be a short one"
    first = int(gt.col_idx[g.nnz // t * t])   # the destination of the last chunk's first entry
    linked = np.zeros(n, bool)
    linked[g.col_idx[g.row_ptr[first]:g.row_ptr[first + 1]]] = True
    linked[first] = True
    assert not linked[n - 1] and gt.row_ptr[n] > gt.row_ptr[n - 1]
    X, W = synth.uniform(n, 1, (n, 20), -0.5, 0.5), synth.glorot(n, 2, 20, heads * d)
    a_l, a_r = synth.normal(n, 3, (heads * d,), 0.0, 0.3), synth.normal(n, 4, (heads * d,), 0.0, 0.3)
    dY = synth.normal(n, 5, (n, heads * d))
    dY[first] = 0.0
    want = oracle.gat_backward_heads(n, n, g.row_ptr, g.col_idx, X, W, a_l, a_r, heads, dY, slope=0.2)[0]
    dY[first] = bad
    A, At = DeviceCSR(g), DeviceCSR(gt)
    dX = ctx.gat_backward_heads(A.s, At.s, ctx.transpose_positions(A.s, At.s), dev(X), dev(W), dev(a_l), dev(a_r), heads, dev(dY), neg_slope=0.2)[0].cpu().numpy()
    assert_close(dX[~linked], want[~linked], what="dX")
    assert not np.isfinite(dX[linked]).all()
