"""The per-entry kernels that walk the entries of a chunk instead of its rows: row lengths around the chunk length, rows that start and
end exactly on chunk boundaries, runs of empty and of one-entry rows, a row over more chunks than one lane joins, and a ragged last
chunk, for each of the four chunk lengths, against fp64 on the host."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2306_15155_amd import ACT_NONE, ACT_RELU, SPMM_PATTERN, SPMM_SCALED, SPMM_WEIGHTED, Context
from paper_2306_15155_amd.binding import GAT_PATH_ONE_WALK, chunk_nnz, gat_attention_path

from gpu_util import DeviceCSR, assert_close, dev

pytestmark = pytest.mark.gpu

N_COLS = 12_000


@pytest.fixture(scope="module")
def ctx():
    c = Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def pattern(t, least):
    """Row lengths that meet the chunk boundaries of length t in every way, then random short rows up to `least` entries and a ragged end."""
    rng = np.random.default_rng(t)
    head = [t, t, 1, 0, t - 1, 0, 0, 2 * t, t + 1, 9 * t + 3, 63, 64, 65] + [1] * 130 + [0] * 70 + [17 * t + 5 if 17 * t + 5 <= N_COLS else N_COLS, 0, 1]
    rest = max(least - sum(head), 0) + 7
    tail = rng.integers(0, 90, rest // 30 + 2)
    cut = int(np.searchsorted(np.cumsum(tail), rest))
    lens = np.concatenate([head, tail[:cut + 1], [0, 0, 5, 0]]).astype(np.int64)
    row_ptr = np.concatenate([[0], np.cumsum(lens)])
    row = np.repeat(np.arange(lens.size), lens)
    k = np.arange(row_ptr[-1]) - row_ptr[row]
    step = N_COLS // lens[row]
    col = k * step + (rng.random(k.size) * step).astype(np.int64)   # ascending and distinct: one column per `step`
    return synth.CSR(lens.size, max(N_COLS, lens.size), row_ptr.astype(np.int32), col.astype(np.int32))


@pytest.mark.parametrize("t,least", [(64, 3_000), (128, 140_000), (256, 270_000), (512, 530_000)])
def test_flat_walk_at_chunk_boundaries(ctx, t, least):
    g = pattern(t, least)
    assert chunk_nnz(g.nnz) == t
    n, A = g.n_rows, DeviceCSR(g)
    row = np.repeat(np.arange(n), np.diff(g.row_ptr))
    s_l, s_r = synth.normal(t, 1, (n,)), synth.normal(t, 2, (g.n_cols,))
    e = s_l[row].astype(np.float64) + s_r[g.col_idx]
    e = np.where(e > 0, e, 0.2 * e)
    got = ctx.sddmm_score(A.s, dev(s_l), dev(s_r))
    assert_close(got, e, tol=2.0 ** -22, what="logits")   # one fp32 addition and one product
    m = np.full(n, -np.inf)
    np.maximum.at(m, row, e)
    p = np.exp(e - m[row])
    z = np.zeros(n)
    np.add.at(z, row, p)
    # exponents up to 16 (rounded at 2^-24 relative: 1e-6) and about twenty additions per value in the sum (1.2e-6)
    assert_close(ctx.edge_softmax(A.s, got), p / z[row], tol=4e-6, what="softmax")
    # two 32-column slices of per-entry dot products, their row sums and the sums of dt over rows of the pattern and of its transpose
    # (slope 1: the derivative of the score does not jump)
    gt = synth.transpose(g)
    f_in, f_out = 24, 40
    X, W, dY = synth.uniform(t, 3, (g.n_cols, f_in)), synth.glorot(t, 4, f_in, f_out), synth.normal(t, 5, (n, f_out))
    a_l, a_r = synth.normal(t, 6, (f_out,), 0.0, 0.3), synth.normal(t, 7, (f_out,), 0.0, 0.3)
    At = DeviceCSR(gt)
    pos = ctx.transpose_positions(A.s, At.s)
    want = oracle.gat_backward(n, g.n_cols, g.row_ptr, g.col_idx, X, W, a_l, a_r, dY, slope=1.0)
    for gpu, ref, what in zip(ctx.gat_backward(A.s, At.s, pos, dev(X), dev(W), dev(a_l), dev(a_r), dev(dY), neg_slope=1.0), want, ("dX", "dW", "da_l", "da_r")):
        assert_close(gpu, ref, what=what)


@pytest.mark.parametrize("t,least", [(64, 3_000), (128, 140_000), (256, 270_000), (512, 530_000)])
def test_flat_spmm_at_chunk_boundaries(ctx, t, least):
    """Every mode of the SpMM on the same patterns, operands of one and two 32-column tiles (the second partly filled) and of an odd width."""
    g = pattern(t, least)
    n, row = g.n_rows, np.repeat(np.arange(g.n_rows), np.diff(g.row_ptr))
    val = synth.uniform(t, 8, (g.nnz,))
    r, c = synth.uniform(t, 9, (n,), 0.5, 1.5), synth.uniform(t, 10, (g.n_cols,), 0.5, 1.5)
    A, Av = DeviceCSR(g), DeviceCSR(g, val)
    for f in (32, 40, 41):
        B = synth.uniform(t, 11, (g.n_cols, f))
        for mode, a, w in ((SPMM_PATTERN, A, np.ones(g.nnz)), (SPMM_WEIGHTED, Av, val.astype(np.float64)),
                           (SPMM_SCALED, A, r[row].astype(np.float64) * c[g.col_idx])):
            ref = np.zeros((n, f))
            for lo in range(0, g.nnz, 1 << 18):
                np.add.at(ref, row[lo:lo + (1 << 18)], w[lo:lo + (1 << 18), None] * B[g.col_idx[lo:lo + (1 << 18)]].astype(np.float64))
            scaled = mode == SPMM_SCALED
            for act in (ACT_NONE, ACT_RELU):
                got = ctx.spmm(a.s, mode, dev(B), dev(r) if scaled else None, dev(c) if scaled else None, act)
                assert_close(got, np.maximum(ref, 0) if act else ref, what=f"mode {mode}, {f} columns, activation {act}")
    # attention aggregations: one walk or two passes by the mean row, and the sums with a vector per entry of the GATv2 backward
    X, W, Wl = synth.uniform(t, 12, (g.n_cols, 24)), synth.glorot(t, 13, 24, 32), synth.glorot(t, 14, 24, 32)
    a_l, a_r = synth.normal(t, 15, (32,), 0.0, 0.5), synth.normal(t, 16, (32,), 0.0, 0.5)
    for f in (32, 20):
        ref = oracle.gat_layer(n, g.n_cols, g.row_ptr, g.col_idx, X, W[:, :f].copy(), a_l[:f], a_r[:f], 0.2, 1)
        assert_close(ctx.gat_layer(A.s, dev(X), dev(W[:, :f].copy()), dev(a_l[:f]), dev(a_r[:f]), 0, 0.2, ACT_RELU), ref, what=f"attention, {f} columns")
    gt = synth.transpose(g)
    At, dY = DeviceCSR(gt), synth.normal(t, 17, (n, 32))
    want = oracle.gatv2_backward(n, g.n_cols, g.row_ptr, g.col_idx, X, Wl, W, a_l, dY, slope=1.0)
    got = ctx.gatv2_backward(A.s, At.s, ctx.transpose_positions(A.s, At.s), dev(X), dev(Wl), dev(W), dev(a_l), dev(dY), neg_slope=1.0)
    for gpu, ref, what in zip(got, want, ("dX", "dW_l", "dW_r", "datt")):
        assert_close(gpu, ref, what=what)


def head_inputs(g, t, f_in, heads, d):
    """X, W, a_l, a_r whose logits stay away from zero with both signs in every longer row: the derivative of LeakyReLU jumps there.  Column 0 of
    every head is +-1 by the source and only a_r sees it (2.5), the rest of the score stays below 2."""
    X, W = synth.uniform(t, 21, (g.n_cols, f_in)), synth.glorot(t, 22, f_in, heads * d)
    a_l, a_r = synth.normal(t, 23, (heads * d,), 0.0, 0.1), synth.normal(t, 24, (heads * d,), 0.0, 0.1)
    X[:, 0] = np.where(np.random.default_rng(t).random(g.n_cols) < 0.5, 1.0, -1.0)
    W[0, :], W[:, ::d] = 0.0, 0.0
    W[0, ::d], a_l[::d], a_r[::d] = 1.0, 0.0, 2.5
    theta = (X.astype(np.float64) @ W).reshape(g.n_cols, heads, d)
    s_l, s_r = ((theta * a.reshape(heads, d)).sum(-1) for a in (a_l, a_r))
    assert (np.abs(s_r).min(0) - np.abs(s_l).max(0)).min() > 0.1
    return X, W, a_l, a_r


# heads of at most one slice: the two walks of the backward at every chunk length, heads that fill their slice and heads that do not
@pytest.mark.parametrize("t,least", [(64, 3_000), (128, 140_000), (256, 270_000), (512, 530_000)])
@pytest.mark.parametrize("heads,d", [(1, 32), (3, 20), (4, 32)])
def test_narrow_heads_at_chunk_boundaries(ctx, t, least, heads, d):
    g = pattern(t, least)
    assert chunk_nnz(g.nnz) == t
    f_in = 24
    X, W, a_l, a_r = head_inputs(g, t, f_in, heads, d)
    dY = synth.normal(t, 25, (g.n_rows, heads * d))
    A, At = DeviceCSR(g), DeviceCSR(synth.transpose(g))
    want = oracle.gat_backward_heads(g.n_rows, g.n_cols, g.row_ptr, g.col_idx, X, W, a_l, a_r, heads, dY, slope=0.2)
    got = ctx.gat_backward_heads(A.s, At.s, ctx.transpose_positions(A.s, At.s), dev(X), dev(W), dev(a_l), dev(a_r), heads, dev(dY), neg_slope=0.2)
    for gpu, ref, what in zip(got, want, ("dX", "dW", "da_l", "da_r")):
        assert_close(gpu, ref, what=what)


# the forward walk of heads of one slice: more of them than slices are worked on at a time (8), and than one launch takes (16)
@pytest.mark.parametrize("t,least", [(256, 270_000), (512, 530_000)])
@pytest.mark.parametrize("heads", [2, 9, 17])
def test_heads_of_one_walk(ctx, t, least, heads):
    g = pattern(t, least)
    f_in, A = 24, DeviceCSR(g)
    assert chunk_nnz(g.nnz) == t and gat_attention_path(A.s, f_in, heads * 32, 0, heads) == GAT_PATH_ONE_WALK
    X, W, a_l, a_r = head_inputs(g, t, f_in, heads, 32)
    want = oracle.gat_layer_heads(g.n_rows, g.n_cols, g.row_ptr, g.col_idx, X, W, a_l, a_r, heads, 0.2, ACT_RELU)
    assert_close(ctx.gat_layer_heads(A.s, dev(X), dev(W), dev(a_l), dev(a_r), heads, 0, 0.2, ACT_RELU), want, what=f"{heads} heads")


# logits of -inf (masked entries) weigh 0 wherever they stand in their row; a row of nothing else is NaN, as 0 / 0 is; the lowest finite
# value is an ordinary logit
@pytest.mark.parametrize("mask", [-np.inf, np.finfo(np.float32).min])
@pytest.mark.parametrize("t,least", [(64, 3_000), (128, 140_000), (256, 270_000), (512, 530_000)])
def test_softmax_of_masked_logits(ctx, t, least, mask):
    g = pattern(t, least)
    n, A, row = g.n_rows, DeviceCSR(g), np.repeat(np.arange(g.n_rows), np.diff(g.row_ptr))
    pos = np.arange(g.nnz) - g.row_ptr[row]
    rng = np.random.default_rng(t + 1)
    for what, hit in (("one in 500", rng.random(g.nnz) < 0.002), ("a third", rng.random(g.nnz) < 0.33), ("the first of a row", pos == 0),
                      ("the first 600 of a row", pos < 600), ("all", np.ones(g.nnz, bool))):
        e = np.where(hit, np.float32(mask), synth.normal(t, 1, (g.nnz,)))
        m = np.full(n, -np.inf)
        np.maximum.at(m, row, e)
        with np.errstate(invalid="ignore"):
            p = np.exp(e.astype(np.float64) - m[row])
            z = np.zeros(n)
            np.add.at(z, row, p)
            want = p / z[row]
        got = ctx.edge_softmax(A.s, dev(e)).cpu().numpy()
        assert np.array_equal(np.isnan(got), np.isnan(want)), f"{what}: {np.isnan(got).sum()} NaN, {np.isnan(want).sum()} wanted"
        assert_close(np.nan_to_num(got), np.nan_to_num(want), tol=4e-6, what=what)   # as above


# value-less SpMM on both sides of the mean rows between which it goes by rows (2.5 and 5 entries): empty rows, a row over many chunks, row-major operands of
# every lane group and slice-major ones of several tiles (a layer that aggregates first), infinities where they belong
@pytest.mark.parametrize("n", [2_000, 60_000, 150_000])
@pytest.mark.parametrize("mean", [2.4, 2.6, 4.9, 5.1])
def test_spmm_on_short_rows(ctx, n, mean):
    rng = np.random.default_rng(n)
    lens = np.bincount(rng.integers(0, n, int(n * mean) - 1_500), minlength=n)
    lens[7] += 1_500
    row_ptr = np.concatenate([[0], np.cumsum(lens)])
    row = np.repeat(np.arange(n), lens)
    step = n // lens[row]
    col = (np.arange(row.size) - row_ptr[row]) * step + (rng.random(row.size) * step).astype(np.int64)
    g = synth.CSR(n, n, row_ptr.astype(np.int32), col.astype(np.int32))
    A = DeviceCSR(g)
    r, c = (ctx.norm_vectors(d) for d in ctx.degrees(A.s))
    for f in (4, 13, 16, 20, 32, 64, 100) if n < 100_000 else (8, 64):
        B = synth.uniform(n, f, (n, f))
        ref = np.zeros((n, f))
        np.add.at(ref, row, B[g.col_idx].astype(np.float64))
        assert_close(ctx.spmm(A.s, SPMM_PATTERN, dev(B)), ref, what=f"{f} columns")
        W = synth.glorot(n, 10, f, 16)
        assert_close(ctx.gcn_layer(A.s, r, c, dev(B), dev(W), 0, ACT_RELU), oracle.gcn_layer(n, n, g.row_ptr, g.col_idx, B, W, 1), what=f"layer, {f} columns")
    B[3] = np.inf
    hit = np.zeros(n, bool)
    hit[row[g.col_idx == 3]] = True
    got = ctx.spmm(A.s, SPMM_PATTERN, dev(B)).cpu().numpy()
    assert np.isposinf(got[hit]).all() and np.isfinite(got[~hit]).all()


# operands of 8- and 4-byte words: widths on both sides of every lane group (8, 16, 32 lanes) and of two tiles
@pytest.mark.parametrize("t,least", [(64, 3_000), (512, 530_000)])
def test_spmm_on_narrow_words(ctx, t, least):
    g = pattern(t, least)
    row = np.repeat(np.arange(g.n_rows), np.diff(g.row_ptr))
    A, r, c = DeviceCSR(g), synth.uniform(t, 9, (g.n_rows,), 0.5, 1.5), synth.uniform(t, 10, (g.n_cols,), 0.5, 1.5)
    for f, ld in ((1, 1), (1, 3), (2, 2), (3, 3), (7, 7), (8, 9), (9, 9), (10, 10), (16, 17), (16, 18), (18, 18), (31, 31), (33, 33), (62, 62)):
        B = synth.uniform(t, f, (g.n_cols, ld))
        ref = np.zeros((g.n_rows, f))
        w = r[row].astype(np.float64) * c[g.col_idx]
        for lo in range(0, g.nnz, 1 << 18):
            np.add.at(ref, row[lo:lo + (1 << 18)], w[lo:lo + (1 << 18), None] * B[g.col_idx[lo:lo + (1 << 18)], :f].astype(np.float64))
        assert_close(ctx.spmm(A.s, SPMM_SCALED, dev(B)[:, :f], dev(r), dev(c), ACT_NONE), ref, what=f"{f} of {ld} columns")


# wide row-major operands: groups of 16, 32 and 64 lanes, widths that fill their last tile and widths that do not (the pattern has too few
# entries per column for the slice-major copy)
@pytest.mark.parametrize("f", [1_028, 2_048, 2_052, 4_096, 4_100, 8_192, 8_196])
def test_spmm_on_wide_rows(ctx, f):
    g = pattern(64, 3_000)
    row = np.repeat(np.arange(g.n_rows), np.diff(g.row_ptr))
    val = synth.uniform(f, 8, (g.nnz,))
    gen = torch.Generator(device="cuda").manual_seed(f)
    B = torch.randn(g.n_cols, f, generator=gen, device="cuda")
    col, rows = torch.from_numpy(g.col_idx).long().cuda(), torch.from_numpy(row).cuda()
    for mode, A, w in ((SPMM_PATTERN, DeviceCSR(g), None), (SPMM_WEIGHTED, DeviceCSR(g, val), dev(val).double()[:, None])):
        ref = torch.zeros(g.n_rows, f, dtype=torch.float64, device="cuda")
        for lo in range(0, g.nnz, 4096):
            x = B[col[lo:lo + 4096]].double()
            ref.index_add_(0, rows[lo:lo + 4096], x if w is None else w[lo:lo + 4096] * x)
        assert_close(ctx.spmm(A.s, mode, B), ref.cpu().numpy(), what=f"mode {mode}, {f} columns")
