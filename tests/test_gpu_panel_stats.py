"""The statistics pass of the attention layer over column panels, whose share of the score vector lies in LDS: rows that span chunks and panels,
rows without entries in a panel or at all, hubs, and the widths on both sides of what fits."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2306_15155_amd import ACT_NONE, Context, Panels, binding, csr_struct

from gpu_util import DeviceCSR, assert_close, dev, hub_and_empty_graph

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = Context(0)
    yield c
    c.close()


# 20,480 floats of a panel fit: 40,000 / 2 do, 45,000 / 2 do not (the pass over the pattern itself); chunks of 512 entries need 2^19 of them
@pytest.mark.parametrize("n,pairs,hub,panels", [(9_000, 600_000, 8_000, 3), (40_000, 560_000, 30_000, 2), (45_000, 560_000, 30_000, 2), (20_483, 700_000, 15_000, 8),
                                                (9_000, 100_000, 4_000, 2)])
def test_attention_over_panels(ctx, n, pairs, hub, panels):
    g = hub_and_empty_graph(23, n, pairs, hub, 700)
    A = DeviceCSR(g)
    P = Panels(ctx, A.s, panels)
    binding._check(binding.lib().sensei_panels_set_min_width(P._h, 32), "min_width")
    Ap = csr_struct(g.n_rows, g.n_cols, A.row_ptr, A.col_idx, None, P)
    f_in, f_out = 24, 64
    X, W = synth.uniform(4, 1, (n, f_in)), synth.glorot(4, 2, f_in, f_out)
    a_l, a_r = synth.normal(4, 3, (f_out,), 0.0, 1.0), synth.normal(4, 4, (f_out,), 0.0, 1.0)
    assert binding.gat_attention_path(Ap, f_in, f_out, 0) == binding.GAT_PATH_PANELS
    Y = ctx.gat_layer(Ap, dev(X), dev(W), dev(a_l), dev(a_r), 0, 0.2, ACT_NONE)
    assert_close(Y, oracle.gat_layer(g.n_rows, g.n_cols, g.row_ptr, g.col_idx, X, W, a_l, a_r, 0.2, ACT_NONE), what="gat over panels")
