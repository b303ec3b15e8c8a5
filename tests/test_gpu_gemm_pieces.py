"""The dense product on bf16 pieces where it can go wrong: k around the 16- and 32-wide steps and the chunk lengths, columns around blocks of 32,
the last tile of rows, operands whose rows are longer than the product and start at odd words, infinities; and the epilogue that adds a
slice-major matrix.  The bound on a product is that of fp32 accumulation: one rounding of the running sum per instruction (six a step of 16 k)
and the roundings inside one, all relative to the sum of the terms' magnitudes."""
import numpy as np
import pytest
import torch

import oracle
import synth
from paper_2306_15155_amd import ACT_NONE, ACT_RELU, Context, binding

from gpu_util import DeviceCSR, assert_close, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = Context(0)
    yield c
    c.close()


# resident and chunked W, every number of column blocks a wavefront takes, ragged last tiles
SHAPES = [(65_537, 16, 5), (65_540, 17, 33), (65_567, 31, 64), (30_001, 32, 100), (28_001, 33, 128), (16_031, 64, 65), (16_001, 65, 130), (17_000, 100, 47),
          (16_005, 127, 160), (20_001, 129, 256), (16_033, 255, 31), (40_001, 256, 96), (70_000, 257, 47), (6_001, 300, 600), (33_000, 602, 24),
          (36_001, 602, 41), (6_033, 601, 300), (7_001, 700, 224), (50_000, 340, 384)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("extra", [0, 3])   # floats by which the rows of both operands are longer (and start late)
def test_product_against_fp64(ctx, shape, extra):
    n, k, m = shape
    assert binding.gemm_kernel(n, k, m) == binding.GEMM_BF16_PIECES
    g = torch.Generator(device="cuda:0").manual_seed(n + k + m)
    A = torch.randn(n, k + extra, device="cuda:0", generator=g)[:, extra // 2 : extra // 2 + k]
    W = torch.randn(k, m + extra, device="cuda:0", generator=g)[:, extra - extra // 2 : extra - extra // 2 + m]
    for act in (ACT_NONE, ACT_RELU):
        Y = ctx.gemm(A, W, act).double()
        ref, terms = A.double() @ W.double(), A.double().abs() @ W.double().abs()
        if act == ACT_RELU:
            ref = ref.clamp(min=0)
        bound = 2.0 ** -24 * (6 * ((k + 15) // 16) + 16)
        worst = ((Y - ref).abs() / terms).max().item()
        assert worst <= bound, (worst, bound)


def test_infinities_and_the_largest_values(ctx):
    n, k, m = 20_000, 70, 40
    A, W = synth.uniform(5, 1, (n, k), 0.5, 1.0), synth.uniform(5, 2, (k, m), 0.5, 1.0)
    big = float(np.finfo(np.float32).max)
    A[7, 3], A[9, 5], A[11, 0] = np.inf, -np.inf, np.nan
    A[13, :], A[13, 2] = 0.0, -big
    Y = ctx.gemm(dev(A), dev(W), ACT_NONE).cpu().numpy()
    assert np.all(Y[7] == np.inf) and np.all(Y[9] == -np.inf) and np.all(np.isnan(Y[11]))
    ref = -big * W[2].astype(np.float64)
    assert np.all(np.abs(Y[13] - ref) <= 2.0 ** -22 * np.abs(ref))
    rest = np.setdiff1d(np.arange(n), [7, 9, 11, 13])
    assert np.all(np.isfinite(Y[rest]))


# resident and chunked W, one to four blocks of columns, more than 64 tiles of rows a wavefront
@pytest.mark.parametrize("shape", [(66_000, 70, 20), (66_000, 720, 17), (66_000, 100, 64), (66_000, 301, 50), (66_000, 90, 96), (66_001, 259, 88), (66_031, 66, 128),
                                   (66_000, 200, 256), (4_300_000, 16, 32)])
def test_overflow_and_infinities_are_those_of_fp32(ctx, shape):
    """Pieces of mixed signs must not turn a product that overflows, or one with an infinity, into NaN or the other infinity: one element per row,
    weights of both signs that are cut with rounding up and down, products from 2^100 to 2^200."""
    n, k, m = shape
    assert binding.gemm_kernel(n, k, m) == binding.GEMM_BF16_PIECES
    g = torch.Generator(device="cuda:0").manual_seed(n + k)
    W = torch.randn(k, m, device="cuda:0", generator=g) * 700.0
    W[:, 0], W[:, 1] = 602.5, -602.5          # second piece against the first
    W[:, 2:4] *= 1e30
    A = torch.randn(n, k, device="cuda:0", generator=g)
    plain = ctx.gemm(A, W, ACT_NONE)
    rows = torch.randperm(n, device="cuda:0", generator=g)[: 64 * 12].reshape(64, 12)
    rows[0, 0], rows[0, 1] = n - 1, 31
    rows = rows.flatten()
    rows = torch.unique(rows)
    special = torch.zeros(rows.numel(), k, device="cuda:0")
    at = torch.arange(rows.numel(), device="cuda:0")
    x = torch.randn(rows.numel(), device="cuda:0", generator=g) * 2.0 ** (100 + (at % 28).float())
    x[at % 7 == 0], x[at % 7 == 1], x[at % 7 == 2] = float("inf"), float("-inf"), float(np.finfo(np.float32).max)
    q = torch.randint(0, k, (rows.numel(),), device="cuda:0", generator=g)
    special[at, q] = x
    A[rows] = special
    finite = torch.isfinite(x)
    rest = torch.ones(n, dtype=torch.bool, device="cuda:0")
    rest[rows] = False
    for act in (ACT_NONE, ACT_RELU):
        Y = ctx.gemm(A, W, act)
        # a finite element: its product, infinite where fp32 has no value for it; an infinite one: 0 * w of the others does not matter, w = 0 would be NaN
        ref = (x[:, None].double() * W[q].double()).float()
        ref = ref.clamp(min=0) if act == ACT_RELU else ref
        got = Y[rows]
        assert torch.equal(Y[rest], plain[rest] if act == ACT_NONE else plain[rest].clamp(min=0))   # the rows beside keep their bits
        assert torch.equal(torch.isinf(got), torch.isinf(ref)) and not torch.isnan(got).any()
        assert torch.equal(got[torch.isinf(ref)], ref[torch.isinf(ref)])
        ok = torch.isfinite(ref) & (ref.abs() > 1e-30)
        assert ((got[ok].double() - ref[ok].double()).abs() <= 2.0 ** -22 * ref[ok].double().abs()).all()
        assert finite.any()
    # a row with a NaN is NaN, the rows around it are not
    A[rows] = 0.0
    A[17, k // 2] = float("nan")
    Y = ctx.gemm(A, W, ACT_NONE)
    assert torch.isnan(Y[17]).all() and torch.isfinite(Y[:17]).all() and torch.isfinite(Y[18:]).all()
    rest[17] = False
    assert torch.equal(Y[rest], plain[rest])   # the rows beside such a row keep their bits


# fewer than 256 blocks of 256 rows, eight piece products: one to four blocks of columns, resident and chunked W; more, six products
SMALL = [(40_000, 100, 32), (20_033, 720, 17), (40_000, 200, 64), (33_000, 301, 50), (40_001, 100, 96), (40_001, 259, 88), (40_000, 66, 128), (30_000, 602, 256)]
LARGE = [(66_000, 100, 32), (66_000, 301, 50), (66_001, 259, 88), (66_000, 602, 256)]


@pytest.mark.parametrize("shape,units", [(s, 1.11) for s in SMALL] + [(s, 3.2) for s in LARGE])
def test_a_single_term(ctx, shape, units):
    """One element a row, so that every sum is one product, in units of 2^-24 of it.  With eight piece products it is rounded once (1), and its small
    ones, at most 2^-7 of it, lose up to 2^-23 of that each time one of seven is added (0.11): as exact as the fp32 instruction, which products
    of these sizes would take otherwise.  With six, what is left out is up to 1.07, and the instruction's own sum of the largest with the others loses up
    to another 2^-23 (2).  A third of the operands is 1 +- 2^-8 -+ 2^-17, whose second and third pieces are as large as rounding leaves them."""
    n, k, m = shape
    assert binding.gemm_kernel(n, k, m) == binding.GEMM_BF16_PIECES
    g = torch.Generator(device="cuda:0").manual_seed(n + k + m)
    wide = torch.tensor([1.0 + 2.0 ** -8 - 2.0 ** -17, 1.0 - 2.0 ** -8 + 2.0 ** -17], device="cuda:0")

    def operand(*size):
        x, pick = torch.randn(*size, device="cuda:0", generator=g), torch.randint(0, 6, size, device="cuda:0", generator=g)
        return torch.where(pick < 2, wide[pick.clamp(max=1)] * x.sign(), x)
    W, x = operand(k, m), operand(n)
    A, q = torch.zeros(n, k, device="cuda:0"), torch.randint(0, k, (n,), device="cuda:0", generator=g)
    A[torch.arange(n, device="cuda:0"), q] = x
    ref = x.double()[:, None] * W.double()[q]
    worst = ((ctx.gemm(A, W, ACT_NONE).double() - ref).abs() / ref.abs()).max().item() * 2.0 ** 24
    assert worst <= units, worst


@pytest.mark.parametrize("f_in,f_out", [(64, 41), (101, 96)])
def test_epilogue_adds_a_sliced_matrix(ctx, f_in, f_out):
    """TAGCN, update first: every product but the first adds the running sum of the hops."""
    g = synth.rmat(17, 20_011, 60_000)
    A = DeviceCSR(g)
    dr, dc = ctx.degrees(A.s)
    r, c = ctx.norm_vectors(dr), ctx.norm_vectors(dc)
    X, W = synth.uniform(17, 1, (g.n_cols, f_in)), synth.glorot(17, 2, 3 * f_in, f_out)
    Y = ctx.tagcn_layer(A.s, r, c, dev(X), dev(W), 2, 1, ACT_RELU)
    assert_close(Y, oracle.tagcn_layer(g.n_rows, g.row_ptr, g.col_idx, X, W, 2, ACT_RELU), what="tagcn update first")
