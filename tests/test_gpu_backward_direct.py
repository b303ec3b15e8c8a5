"""Weight gradients by way of the aggregated input, where its rows are gathered too seldom to earn a scaled copy: the walk over the input itself on
both sides of the line (four gathers a row, 16-byte rows), against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2306_15155_amd import ACT_NONE, ACT_RELU, GCN_BWD_UPD, Context, binding, csr_struct

from gpu_util import DeviceCSR, assert_close, dev, rect_block

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n_rows,n_cols,per_row,f_in,act", [(700, 9_000, 11, 100, ACT_RELU), (3_000, 3_001, 2, 36, ACT_NONE), (900, 2_000, 30, 64, ACT_RELU),
                                                            (700, 9_000, 11, 33, ACT_RELU), (1, 5, 2, 4, ACT_NONE)])
def test_weight_gradient_from_rarely_gathered_rows(ctx, n_rows, n_cols, per_row, f_in, act):
    g = rect_block(9, n_rows, n_cols, per_row)
    rows = np.repeat(np.arange(n_rows), np.diff(g.row_ptr))
    gt = synth.build_csr(n_cols, n_rows, g.col_idx.astype(np.int32), rows.astype(np.int32), False, False)
    A, At = DeviceCSR(g), DeviceCSR(gt)
    deg_r, deg_c = ctx.degrees(A.s)
    r, c = ctx.norm_vectors(deg_r), ctx.norm_vectors(deg_c)
    f_out = 24
    X, W, dY = synth.uniform(6, 1, (n_cols, f_in)), synth.glorot(6, 2, f_in, f_out), synth.normal(6, 3, (n_rows, f_out), 0.0, 1.0)
    Y = oracle.gcn_layer(g.n_rows, g.n_cols, g.row_ptr, g.col_idx, X, W, act).astype(np.float32)
    want_dx, want_dw = oracle.gcn_backward(g.n_rows, g.n_cols, g.row_ptr, g.col_idx, X, W, dY, Y=Y, act=act)
    dX, dW = ctx.gcn_backward(A.s, At.s, r, c, dev(X), dev(W), dev(dY), GCN_BWD_UPD, Y=dev(Y), activation=act)
    assert_close(dX, want_dx, what="dX")
    assert_close(dW, want_dw, what="dW")
