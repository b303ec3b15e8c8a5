"""The two-walk backward of narrow heads and of the GATv2 score where they can go wrong, against the oracle: rows that span many chunks beside
empty rows, fewer destinations than sources, widths inside a 32-column slice and across slices, more heads than one launch takes, a pattern
without entries.  Bound: the parity tolerance per element (fp32 sums of at most a few thousand terms of order one)."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2306_15155_amd import ACT_NONE, ACT_RELU, Context, binding

from gpu_util import DeviceCSR, assert_close, dev, hub_and_empty_graph, rect_block

pytestmark = pytest.mark.gpu

PATTERNS = {"hub": lambda: hub_and_empty_graph(3, 900, 5_000, 700, 40), "wide": lambda: rect_block(4, 260, 900, 9), "one": lambda: rect_block(5, 1, 6, 3)}


@pytest.fixture(scope="module")
def ctx():
    c = Context(0)
    yield c
    c.close()


def _patterns(ctx, name):
    g = PATTERNS[name]()
    rows = np.repeat(np.arange(g.n_rows), np.diff(g.row_ptr))
    gt = synth.build_csr(g.n_cols, g.n_rows, g.col_idx.astype(np.int32), rows.astype(np.int32), False, False)
    A, At = DeviceCSR(g), DeviceCSR(gt)
    return g, A, At, ctx.transpose_positions(A.s, At.s)


@pytest.mark.parametrize("name", PATTERNS)
@pytest.mark.parametrize("heads,d", [(1, 8), (3, 20), (2, 32), (17, 8), (4, 31)])
def test_narrow_heads(ctx, name, heads, d):
    g, A, At, pos = _patterns(ctx, name)
    f_in, f_out = 36, heads * d
    X, W = synth.uniform(7, 1, (g.n_cols, f_in), -0.5, 0.5), synth.glorot(7, 2, f_in, f_out)
    a_l, a_r = synth.normal(7, 3, (f_out,), 0.0, 0.3), synth.normal(7, 4, (f_out,), 0.0, 0.3)
    dY = synth.normal(7, 5, (g.n_rows, f_out), 0.0, 1.0)
    for act in (ACT_NONE, ACT_RELU):
        Y = oracle.gat_layer_heads(g.n_rows, g.n_cols, g.row_ptr, g.col_idx, X, W, a_l, a_r, heads, 0.2, act)
        for comp in (0, 1):
            assert_close(ctx.gat_layer_heads(A.s, dev(X), dev(W), dev(a_l), dev(a_r), heads, comp, 0.2, act), Y, what=f"Y {comp}")
        Y = Y.astype(np.float32)
        want = oracle.gat_backward_heads(g.n_rows, g.n_cols, g.row_ptr, g.col_idx, X, W, a_l, a_r, heads, dY, Y=Y, slope=0.2, act=act)
        got = ctx.gat_backward_heads(A.s, At.s, pos, dev(X), dev(W), dev(a_l), dev(a_r), heads, dev(dY), Y=dev(Y), neg_slope=0.2, activation=act)
        for what, a, b in zip(("dX", "dW", "da_l", "da_r"), got, want):
            assert_close(a, b, what=f"{what} act {act}")


# Coefficients far below their row's largest, whose exponential must be as exact there as near 0.  X is the identity, so dW is dTheta.  Row i has a source i
# of logit 100 and a source n + i of 100 - x, x up to 80 (positive and exact: neither the slope nor the subtraction rounds).  Source n + i gets alpha dP_i in the
# columns that no attention vector reads.  Column 0, which a_r reads, gets alpha (dalpha - rowdot) of source i, where dalpha is 0 and rowdot the product of the
# small coefficient and a power of two that makes it about one.  Bound: two units of 2^-23 for the exponential, one each for 1 / z and the products.
@pytest.mark.parametrize("d", [8, 32])
def test_small_coefficients_are_exact(ctx, d):
    n = 300
    x = np.round(np.linspace(0.0, 80.0, n) * 1024) / 1024
    g = synth.CSR(n, 2 * n, (2 * np.arange(n + 1)).astype(np.int32), np.stack([np.arange(n), n + np.arange(n)], 1).reshape(-1).astype(np.int32))
    A, At = DeviceCSR(g), DeviceCSR(synth.transpose(g))
    theta, dY = synth.uniform(9, 1, (2 * n, d), 0.5, 1.0), synth.uniform(9, 2, (n, d), 0.5, 1.0)
    theta[:, 0] = 100.0 - np.concatenate([np.zeros(n), x])
    theta[:, 1] = np.concatenate([np.zeros(n), np.exp2(np.round(x / np.log(2.0)))])
    dY[:, 0], dY[:, 1] = 0.0, 1.0
    theta[:, 2:] = 0.0
    a_l, a_r = np.zeros(d, np.float32), np.zeros(d, np.float32)
    a_r[0] = 1.0
    pos = ctx.transpose_positions(A.s, At.s)
    dW = ctx.gat_backward(A.s, At.s, pos, torch.eye(2 * n, device="cuda"), dev(theta), dev(a_l), dev(a_r), dev(dY), neg_slope=0.2)[1].double().cpu().numpy()
    small = 1.0 / (1.0 + np.exp(x))
    rel = np.abs(dW[n:, 2:] / (small[:, None] * dY[:, 2:].astype(np.float64)) - 1.0)
    assert rel.max() <= 5 * 2.0 ** -23, rel.max()
    rowdot = small * theta[n:, 1].astype(np.float64)
    rel = np.abs(dW[:n, 0] / (-(1.0 - small) * rowdot) - 1.0)
    assert rel.max() <= 8 * 2.0 ** -23, rel.max()


@pytest.mark.parametrize("name", PATTERNS)
@pytest.mark.parametrize("f_out", [1, 31, 64, 97])
def test_gatv2_score(ctx, name, f_out):
    g, A, At, pos = _patterns(ctx, name)
    f_in = 21
    X = synth.uniform(8, 1, (g.n_cols, f_in), -0.5, 0.5)
    W_l, W_r, att = synth.glorot(8, 2, f_in, f_out), synth.glorot(8, 3, f_in, f_out), synth.normal(8, 4, (f_out,), 0.0, 0.3)
    dY = synth.normal(8, 5, (g.n_rows, f_out), 0.0, 1.0)
    Y = oracle.gatv2_layer(g.n_rows, g.n_cols, g.row_ptr, g.col_idx, X, W_l, W_r, att, 0.2, ACT_RELU).astype(np.float32)
    for act in (ACT_NONE, ACT_RELU):
        want = oracle.gatv2_backward(g.n_rows, g.n_cols, g.row_ptr, g.col_idx, X, W_l, W_r, att, dY, Y=Y, slope=0.2, act=act)
        got = ctx.gatv2_backward(A.s, At.s, pos, dev(X), dev(W_l), dev(W_r), dev(att), dev(dY), Y=dev(Y), neg_slope=0.2, activation=act)
        for what, a, b in zip(("dX", "dW_l", "dW_r", "datt"), got, want):
            assert_close(a, b, what=f"{what} act {act}")


def test_no_entries(ctx):
    ptr, col = np.zeros(6, dtype=np.int32), np.zeros(0, dtype=np.int32)
    g = synth.CSR(n_rows=5, n_cols=5, row_ptr=ptr, col_idx=col)
    A = DeviceCSR(g)
    pos = ctx.transpose_positions(A.s, A.s)
    X, W, a, dY = torch.ones(5, 8, device="cuda"), torch.ones(8, 32, device="cuda"), torch.ones(32, device="cuda"), torch.ones(5, 32, device="cuda")
    for got in (ctx.gat_backward_heads(A.s, A.s, pos, X, W, a, a, 4, dY, neg_slope=0.2), ctx.gatv2_backward(A.s, A.s, pos, X, W, W, a, dY, neg_slope=0.2)):
        assert all(bool((t == 0).all()) for t in got)
    torch.cuda.synchronize()


# scratch of exactly the size that the query asks for, full of NaN before: pieces and carry sums share a place, and many heads on long rows (300 entries: chunks of
# 512 instead of the walks' 256) have no room for shorter chunks
@pytest.mark.parametrize("n,per_row,heads,d", [(2_000, 300, 17, 2), (2_000, 300, 16, 31), (2_000, 300, 2, 20), (3_000, 90, 1, 32), (500, 7, 3, 20)])
def test_scratch_of_narrow_heads(ctx, n, per_row, heads, d):
    rng = np.random.default_rng(n + per_row)
    col = np.sort(rng.permuted(np.tile(np.arange(n), (n, 1)), axis=1)[:, :per_row], axis=1)
    g = synth.CSR(n, n, (per_row * np.arange(n + 1)).astype(np.int32), col.reshape(-1).astype(np.int32))
    f_in, f_out = 12, heads * d
    X, W = synth.uniform(7, 1, (n, f_in), -0.5, 0.5), synth.glorot(7, 2, f_in, f_out)
    a_l, a_r = synth.normal(7, 3, (f_out,), 0.0, 0.3), synth.normal(7, 4, (f_out,), 0.0, 0.3)
    dY = synth.normal(7, 5, (n, f_out))
    want = oracle.gat_backward_heads(n, n, g.row_ptr, g.col_idx, X, W, a_l, a_r, heads, dY, slope=0.2)
    A, At = DeviceCSR(g), DeviceCSR(synth.transpose(g))
    pos = ctx.transpose_positions(A.s, At.s)
    need = ctypes.c_size_t()
    L = binding.lib()
    binding._check(L.sensei_gat_backward_heads_workspace(ctypes.byref(A.s), ctypes.byref(At.s), f_in, f_out, heads, ctypes.byref(need)), "workspace")
    need = need.value
    room = torch.full((need + 1024,), 0xFF, dtype=torch.uint8, device="cuda")
    at = -room.data_ptr() % 256
    ins = [dev(a) for a in (X, W, a_l, a_r, dY)]
    outs = [torch.empty(s, device="cuda") for s in ((n, f_in), (f_in, f_out), (f_out,), (f_out,))]
    p, m = [t.data_ptr() for t in ins + outs], binding.mat_struct
    binding._check(L.sensei_gat_backward_heads(ctx._h, ctypes.byref(A.s), ctypes.byref(At.s), pos.data_ptr(), m(ins[0]), m(ins[1]), p[2], p[3], heads, 0.2, None, f_out, m(ins[4]),
                                               ACT_NONE, p[5], f_in, p[6], f_out, p[7], p[8], room.data_ptr() + at, need, binding._stream()), "sensei_gat_backward_heads")
    for got, ref, what in zip(outs, want, ("dX", "dW", "da_l", "da_r")):
        assert_close(got, ref, what=what)
    assert bool((room[:at] == 0xFF).all()) and bool((room[at + need:] == 0xFF).all())


# Products with the slope are not rounded before they are added.  Row i has the sources i and m + i; Theta_l is 0, Theta_r (X is the identity) is (1, -1) and (-1, 1) in
# the two columns that `att` reads with ones, so that both logits are 1 - slope, both coefficients 1/2, dalpha u and -u, and dTheta_l[i, 0] the sum of u / 2 and
# -u / 2 times the slope: one rounding.  dW_l is dTheta_l.
@pytest.mark.parametrize("m,f_out", [(300, 8), (1_000, 40)])
def test_products_with_the_slope_are_not_rounded(ctx, m, f_out):
    g = synth.CSR(m, 2 * m, (2 * np.arange(m + 1)).astype(np.int32), np.stack([np.arange(m), m + np.arange(m)], 1).reshape(-1).astype(np.int32))
    A, At = DeviceCSR(g), DeviceCSR(synth.transpose(g))
    W_l, W_r = np.zeros((2 * m, f_out), np.float32), np.zeros((2 * m, f_out), np.float32)
    W_r[:m, :2], W_r[m:, :2] = (1.0, -1.0), (-1.0, 1.0)
    att, dY = np.zeros(f_out, np.float32), np.zeros((m, f_out), np.float32)
    att[:2] = 1.0
    dY[:, 0] = synth.uniform(11, 1, (m,), 0.5, 1.0)
    dW_l = ctx.gatv2_backward(A.s, At.s, ctx.transpose_positions(A.s, At.s), torch.eye(2 * m, device="cuda"), dev(W_l), dev(W_r), dev(att), dev(dY), neg_slope=0.7)[1]
    u, slope = dY[:, 0].astype(np.float64), np.float64(np.float32(0.7))
    assert np.array_equal(dW_l[:m, 0].cpu().numpy(), (u / 2 - u / 2 * slope).astype(np.float32))


# Scratch of exactly the size that the query asks for.  The weight gradients share their slabs: keys of 64 columns take more of them than values of 114, keys of 128 more than
# values of 129, and destinations below 4,096 more than the sources above.
@pytest.mark.parametrize("n_rows,n_cols,f_in,d_k,f_out", [(7_000, 7_000, 576, 64, 114), (6_000, 6_000, 300, 128, 129), (3_000, 6_000, 700, 128, 300), (500, 700, 20, 64, 33)])
def test_slabs_of_several_weight_gradients(ctx, n_rows, n_cols, f_in, d_k, f_out):
    g = rect_block(n_rows, n_rows, n_cols, 3)
    A, At = DeviceCSR(g), DeviceCSR(synth.transpose(g))
    pos = ctx.transpose_positions(A.s, At.s)
    X = np.round(synth.uniform(7, 1, (n_cols, f_in), -1.0, 1.0) * 8) / 8   # on grids: the projections are exact, the derivatives of the score jump alike
    Wq, Wk, Wv, Wl = (np.round(synth.uniform(7, 2 + i, (f_in, w), -0.5, 0.5) * 16) / 64 for i, w in enumerate((d_k, d_k, f_out, f_out)))
    att, dY = np.round(synth.normal(7, 6, (f_out,), 0.0, 0.2) * 64) / 64, synth.normal(7, 7, (n_rows, f_out))
    X, Wq, Wk, Wv, Wl, att = (a.astype(np.float32) for a in (X, Wq, Wk, Wv, Wl, att))
    L, m, need = binding.lib(), binding.mat_struct, ctypes.c_size_t()
    x, q, k, v, l, a, dy = (dev(t) for t in (X, Wq, Wk, Wv, Wl, att, dY))
    args = (n_rows, n_cols, g.row_ptr, g.col_idx, X)

    def checked(call, want, names):
        room = torch.full((need.value + (1 << 22),), 0xFF, dtype=torch.uint8, device="cuda")
        at = -room.data_ptr() % 256
        outs = [torch.empty(w.shape, device="cuda") for w in want]
        binding._check(call([t.data_ptr() for t in outs], room.data_ptr() + at), "backward")
        for got, ref, what in zip(outs, want, names):
            assert_close(got, ref, what=what)
        assert bool((room[at + need.value:] == 0xFF).all())

    binding._check(L.sensei_dotgat_backward_workspace(ctypes.byref(A.s), f_in, d_k, f_out, ctypes.byref(need)), "workspace")
    checked(lambda o, w: L.sensei_dotgat_backward(ctx._h, ctypes.byref(A.s), ctypes.byref(At.s), pos.data_ptr(), m(x), m(q), m(k), m(v), 0.01, None, f_out, m(dy), ACT_NONE,
                                                  o[0], f_in, o[1], d_k, o[2], d_k, o[3], f_out, w, need.value, binding._stream()),
            oracle.dotgat_backward(*args, Wq, Wk, Wv, 0.01, dY), ("dX", "dW_q", "dW_k", "dW_v"))
    binding._check(L.sensei_gatv2_backward_workspace(ctypes.byref(A.s), f_in, f_out, ctypes.byref(need)), "workspace")
    checked(lambda o, w: L.sensei_gatv2_backward(ctx._h, ctypes.byref(A.s), ctypes.byref(At.s), pos.data_ptr(), m(x), m(l), m(v), a.data_ptr(), 0.25, None, f_out, m(dy), ACT_NONE,
                                                 o[0], f_in, o[1], f_out, o[2], f_out, o[3], w, need.value, binding._stream()),
            oracle.gatv2_backward(*args, Wl, Wv, att, dY, slope=0.25), ("dX", "dW_l", "dW_r", "datt"))
