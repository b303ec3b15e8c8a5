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


# the weight gradient of a layer on the identity pattern is X^T dY: around the 64 columns that choose the narrow block, the 128 x 64 block's
# edges, odd leading dimensions and row counts that leave a ragged last slab.  Slabs of 32 rows are summed in fp32 (six products a term),
# everything after that in fp64.
@pytest.mark.parametrize("n,f_in,f_out", [(4096, 1, 1), (4097, 100, 47), (5003, 128, 64), (4999, 129, 63), (6000, 130, 65), (20_001, 33, 32)])
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
