"""A layer that aggregates its input first and gathers it where it lies is the call's only sparse launch: its wavefronts find their rows themselves.
Row counts around the 64-fold narrowing, empty rows at either end and in the middle, rows that span chunks, one and several chunks."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2306_15155_amd import ACT_NONE, Context

from gpu_util import DeviceCSR, assert_close, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("n_rows", [1, 2, 63, 64, 65, 66, 129, 131, 4_225, 4_227, 9_000])
@pytest.mark.parametrize("kind", ["even", "hub", "gaps"])
def test_rows_found_by_the_walk(ctx, n_rows, kind):
    rng = np.random.default_rng(n_rows)
    n_cols = max(n_rows, 3_000)
    deg = rng.integers(0, 9, n_rows)
    if kind == "hub":
        deg[n_rows // 2] = 2_500
    if kind == "gaps":
        deg[: n_rows // 3] = 0
        deg[-(n_rows // 4) - 1 :] = 0
        deg[n_rows // 2] = 200
    u = np.repeat(np.arange(n_rows), deg).astype(np.int32)
    v = np.concatenate([rng.choice(n_cols, d, replace=False) for d in deg] + [np.empty(0, np.int64)]).astype(np.int32)
    g = synth.build_csr(n_rows, n_cols, u, v, False, False)
    A = DeviceCSR(g)
    dr, dc = ctx.degrees(A.s)
    r, c = ctx.norm_vectors(dr), ctx.norm_vectors(dc)
    f_in, f_out = 20, 12
    X, W = synth.uniform(2, 1, (n_cols, f_in)), synth.glorot(2, 2, f_in, f_out)
    Y = ctx.gcn_layer(A.s, r, c, dev(X), dev(W), 2, ACT_NONE)   # scalings inside the walk, aggregated first
    assert_close(Y, oracle.gcn_layer(g.n_rows, g.n_cols, g.row_ptr, g.col_idx, X, W, ACT_NONE), what=kind)
