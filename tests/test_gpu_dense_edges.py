"""Dense kernels at the edges of their tiles, against fp64: every element within (number of terms + 1) fp32 roundings of the sum of the
terms' magnitudes, which bounds any order of summation."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _bound_check(got, a, w):
    ref = a.double() @ w.double()
    mag = a.double().abs() @ w.double().abs()
    err = (got.double() - ref).abs()
    assert bool((err <= (a.size(1) + 1) * 2.0 ** -24 * mag + 1e-30).all()), float((err / (mag + 1e-30)).max())


# the kernel that splits k over the wavefronts: one row to the largest grid it takes, k around its 16-wide steps and 64-wide groups, odd
# widths, and rows whose alignment rules out 16-byte loads
@pytest.mark.parametrize("n,k,m", [(1, 1, 1), (31, 3, 31), (32, 4, 32), (33, 15, 33), (65, 16, 64), (64, 17, 47), (100, 63, 100), (130, 64, 65),
                                   (257, 65, 8), (40, 100, 256), (1024, 257, 47), (10_240, 64, 32), (10_240, 1030, 64), (7, 602, 3)])
@pytest.mark.parametrize("pad", [0, 1])
def test_small_gemm(n, k, m, pad):
    from paper_2306_15155_amd import ACT_RELU, Context
    ctx = Context(0)
    g = torch.Generator(device="cuda").manual_seed(n * 7919 + k * 31 + m)
    a = torch.randn(n, k + pad, generator=g, device="cuda")[:, :k]
    w = torch.randn(k, m + pad, generator=g, device="cuda")[:, :m]
    y = ctx.gemm(a, w)
    _bound_check(y, a, w)
    assert torch.equal(ctx.gemm(a, w, activation=ACT_RELU), y.clamp_min(0))
    if n > 2 and k > 2:   # infinities and NaN stay in their rows and columns
        a = a.clone()
        a[1, 1], a[2, 0] = float("inf"), float("nan")
        z = ctx.gemm(a, w)
        assert bool(z[1].isinf().all()) and bool(z[2].isnan().all())
        keep = [i for i in range(n) if i not in (1, 2)]
        assert torch.equal(z[keep], y[keep])
    ctx.close()


# both sides of the lines where that kernel ends: by k for each alignment and each number of blocks
@pytest.mark.parametrize("n,k,m", [(10_240, 128, 64), (10_240, 129, 64), (10_240, 256, 64), (10_240, 260, 64), (10_240, 384, 32), (10_240, 388, 32),
                                   (10_240, 2_052, 16), (8_192, 2_052, 32), (2_048, 512, 256), (2_049, 512, 256), (4_096, 1_030, 40), (4_097, 1_024, 40), (4_097, 1_030, 40)])
@pytest.mark.parametrize("pad", [0, 1])
def test_gemm_beside_the_small_kernel(n, k, m, pad):
    from paper_2306_15155_amd import Context
    ctx = Context(0)
    g = torch.Generator(device="cuda").manual_seed(n + k * 31 + m)
    a = torch.randn(n, k + pad, generator=g, device="cuda")[:, :k]
    w = torch.randn(k, m, generator=g, device="cuda")
    _bound_check(ctx.gemm(a, w), a, w)
    ctx.close()


# the weight gradient of a layer on the identity pattern is X^T dY: around the 64 columns that choose the narrow block, the 128 x 64 block's
# edges, odd leading dimensions and row counts that leave a ragged last slab.  Slabs of 32 rows are summed in fp32 (six products a term),
# everything after that in fp64.
# The last three: 90 and 144 blocks of 128 x 128, for which the slabs of one round leave a part of the chip idle, and more blocks than compute units.
@pytest.mark.parametrize("n,f_in,f_out", [(4096, 1, 1), (4097, 100, 47), (5003, 128, 64), (4999, 129, 63), (6000, 130, 65), (20_001, 33, 32), (4099, 1280, 1100),
                                          (4097, 1433, 1433), (4096, 2200, 2200)])
def test_weight_gradient_columns(n, f_in, f_out):
    from paper_2306_15155_amd import Context, csr_struct
    ctx = Context(0)
    g = torch.Generator(device="cuda").manual_seed(n + f_in)
    ptr, col = torch.arange(n + 1, dtype=torch.int32, device="cuda"), torch.arange(n, dtype=torch.int32, device="cuda")
    A, one = csr_struct(n, n, ptr, col), torch.ones(n, device="cuda")
    x, dy = torch.randn(n, f_in, generator=g, device="cuda"), torch.randn(n, f_out, generator=g, device="cuda")
    w = torch.randn(f_in, f_out, generator=g, device="cuda")
    _, dw = ctx.gcn_backward(A, A, one, one, x, w, dy, 0, want_dx=False)
    ref, mag = x.double().t() @ dy.double(), x.double().abs().t() @ dy.double().abs()
    assert bool(((dw.double() - ref).abs() <= (32 * 6 + 1) * 2.0 ** -24 * mag).all())
    ctx.close()


# the per-entry products of kept tiles, their places: a full pattern (whole tiles, and a last row and column of tiles that are partly empty)
# with zero attention vectors, where alpha = 1 / n, every logit sits on the LeakyReLU's lower branch, and da_r = Theta^T ds_r is what the
# products <dP_i, Theta_j> reach; Theta = W exactly (X is the identity).  96 columns are below the width from which tiles serve these products
# and take the per-entry kernel.  Bound: f + 8 roundings per product, n + 8 in each of the two sums over nodes it passes through: wide enough
# to pass products of fewer bits, which the test after this one measures.
@pytest.mark.parametrize("n,f", [(128, 96), (128, 128), (300, 160), (300, 256)])
def test_tile_products_of_the_attention_backward(n, f):
    from paper_2306_15155_amd import Context, Tiles, csr_struct
    ctx, slope = Context(0), 0.2
    g = torch.Generator(device="cuda").manual_seed(n * 31 + f)
    row_ptr = (torch.arange(n + 1, device="cuda") * n).to(torch.int32)
    col_idx = torch.arange(n, device="cuda", dtype=torch.int32).repeat(n)
    W, dY = torch.randn(n, f, generator=g, device="cuda"), torch.randn(n, f, generator=g, device="cuda")
    X, zero = torch.eye(n, device="cuda"), torch.zeros(f, device="cuda")
    A = csr_struct(n, n, row_ptr, col_idx)
    T = Tiles(ctx, A, 0.05, 256, min_width=32)
    assert T.n_tiles == ((n + 127) // 128) ** 2
    Ah = csr_struct(n, n, row_ptr, col_idx, tiles=T)
    got = ctx.gat_backward(Ah, Ah, ctx.transpose_positions(A, A), X, W, zero, zero, dY, neg_slope=slope)[3].double()
    D = dY.double() @ W.double().t()
    ref = W.double().t() @ ((D - D.mean(1, keepdim=True)) * (slope / n)).sum(0)
    M = dY.double().abs() @ W.double().abs().t()
    bound = W.double().abs().t() @ ((M + M.mean(1, keepdim=True)) * (slope / n)).sum(0) * (f + 2 * n + 24) * 2.0 ** -24
    assert bool(((got - ref).abs() <= bound).all()), float(((got - ref).abs() / bound).max())
    T.close()
    ctx.close()


# their accuracy: one row of dY with one element, so that every product of that row is a single term d Theta_jq and reaches dW unsummed.  X is
# the identity, all logits are 1 (columns 1 and 2 of Theta are 1 and the attention vectors select them), alpha = 2^-8 exactly, and column 1 of
# dW is dt of that row: 2^-8 (d Theta_jq - m), m the row's mean.  The difference of neighbours is free of m.  Each product may be one fp32
# rounding off, the subtraction of m another, and m itself is 0 but for one node's term; the rest is exact, so 3 units of 2^-24 hold any
# fp32 product.  Theta holds full 24-bit significands and, every fourth pair, 1 + 2^-7 - 2^-23, whose pieces of eight bits are as large as they get.
@pytest.mark.parametrize("f", [128, 160, 256])
def test_tile_products_keep_all_bits(f):
    from paper_2306_15155_amd import Context, Tiles, csr_struct
    ctx, n = Context(0), 256
    g = torch.Generator(device="cuda").manual_seed(f)
    row_ptr = (torch.arange(n + 1, device="cuda") * n).to(torch.int32)
    col_idx = torch.arange(n, device="cuda", dtype=torch.int32).repeat(n)
    A = csr_struct(n, n, row_ptr, col_idx)
    T = Tiles(ctx, A, 0.05, 256, min_width=32)
    assert T.n_tiles == 4
    Ah, pos = csr_struct(n, n, row_ptr, col_idx, tiles=T), ctx.transpose_positions(A, A)
    half = 1.0 + torch.rand(n // 2, f, generator=g, device="cuda")
    half[::4] = 1.0 + 2.0 ** -7 - 2.0 ** -23
    theta = torch.stack([half, -half], 1).reshape(n, f).contiguous()   # neighbours cancel in the mean
    theta[:, 1:3] = 1.0
    a_l, a_r = torch.zeros(f, device="cuda"), torch.zeros(f, device="cuda")
    a_l[2] = a_r[1] = 0.5
    X, worst = torch.eye(n, device="cuda"), 0.0
    for q, i in ((0, 0), (3, 127), (17, 128), (f // 2 + 5, 200), (f - 1, 255)):
        for d in (1.0 + 2.0 ** -7 - 2.0 ** -23, 1.7320508):
            dY = torch.zeros(n, f, device="cuda")
            dY[i, q] = d
            dW = ctx.gat_backward(Ah, Ah, pos, X, theta, a_l, a_r, dY, neg_slope=0.2)[1]
            ds_r = 2.0 * dW[:, 1].double()   # a_r[1] = 1 / 2
            term = theta[:, q].double() * float(dY[i, q])
            got, want = ds_r[0::2] - ds_r[1::2], (term[0::2] - term[1::2]) * 2.0 ** -8
            mag = (term[0::2].abs() + term[1::2].abs()) * 2.0 ** -8
            worst = max(worst, float(((got - want).abs() / mag).max()) * 2.0 ** 24)
    print(f"{f} columns: {worst:.2f} units of 2^-24")
    assert worst <= 3.0, worst
    T.close()
    ctx.close()


# The same over many operands, and held to what the kernel claims: a product is rounded once (one unit of 2^-24 of it at most) and its small piece
# products lose seven times 2^-23 of at most 2^-7 of it (0.11 units).  Neighbours cancel exactly, so m is 0 and nothing else rounds.  Every eighth
# pair has 1 +- 2^-8 -+ 2^-17, whose second and third pieces are as large as rounding leaves them.
@pytest.mark.parametrize("f", [128, 256])
def test_tile_products_are_rounded_once(f):
    from paper_2306_15155_amd import Context, Tiles, csr_struct
    ctx, n = Context(0), 256
    g = torch.Generator(device="cuda").manual_seed(f)
    row_ptr = (torch.arange(n + 1, device="cuda") * n).to(torch.int32)
    col_idx = torch.arange(n, device="cuda", dtype=torch.int32).repeat(n)
    A = csr_struct(n, n, row_ptr, col_idx)
    T = Tiles(ctx, A, 0.05, 256, min_width=32)
    assert T.n_tiles == 4
    Ah, pos = csr_struct(n, n, row_ptr, col_idx, tiles=T), ctx.transpose_positions(A, A)
    half = torch.rand(n // 2, f, generator=g, device="cuda") - 0.5
    half[::8], half[1::8] = 1.0 + 2.0 ** -8 - 2.0 ** -17, 1.0 - 2.0 ** -8 + 2.0 ** -17
    theta = torch.stack([half, -half], 1).reshape(n, f).contiguous()
    theta[:, 1:3] = 1.0
    a_l, a_r = torch.zeros(f, device="cuda"), torch.zeros(f, device="cuda")
    a_l[2] = a_r[1] = 0.5
    X, worst = torch.eye(n, device="cuda"), 0.0
    for i in range(0, 256, 7):
        q = int(torch.randint(3, f, (1,), generator=g, device="cuda"))
        d = float(torch.rand(1, generator=g, device="cuda")) - 0.5
        for d in (d, 1.0 + 2.0 ** -8 - 2.0 ** -17, -1.0 + 2.0 ** -8 - 2.0 ** -17):
            dY = torch.zeros(n, f, device="cuda")
            dY[i, q] = d
            dW = ctx.gat_backward(Ah, Ah, pos, X, theta, a_l, a_r, dY, neg_slope=0.2)[1]
            ds_r = 2.0 * dW[:, 1].double()
            term = theta[:, q].double() * float(dY[i, q]) * 2.0 ** -8
            got, want = ds_r[0::2] - ds_r[1::2], term[0::2] - term[1::2]
            worst = max(worst, float(((got - want).abs() / want.abs()).nan_to_num().max()) * 2.0 ** 24)
    print(f"{f} columns: {worst:.3f} units of 2^-24")
    assert worst <= 1.11, worst
    T.close()
    ctx.close()
