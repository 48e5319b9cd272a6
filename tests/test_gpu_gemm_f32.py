"""fp32 products on bf16 parts (K of 256 and more) and on the fp32 instruction, through the fp32 embedding, against fp64."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vd():
    import paper_2501_14183_amd as m
    return m


def product(vd, x, We, dxs):
    """x [B, n, L] We [L, d] and its weight gradient x^T dxs, both fp32."""
    ctx = vd.Context(0)
    B, n, L = x.shape
    sel = torch.arange(n, dtype=torch.int32, device="cuda")
    xs, saved = vd.vardrop_embed_fwd(ctx, x.cuda(), sel, n, We.cuda(), None, False)
    dWe, _ = vd.vardrop_embed_bwd(ctx, dxs.cuda(), L, saved, want_bias=False)
    torch.cuda.synchronize()
    return xs.cpu().reshape(B * n, -1), dWe.cpu()


def assert_close(got, a, b, bound):
    """|error| <= bound * sum |a||b| for every element: what a rounding of every term costs, whatever the scales."""
    a, b = a.double(), b.double()
    slack = bound * (a.abs() @ b.abs())
    assert bool(((got.double() - a @ b).abs() <= slack).all()), float(((got.double() - a @ b).abs() / slack).max())


# 2^-22: the dropped products of parts are at most 2^-24 of a term, another 2^-24 is the rounding of the result; sums of up
# to 1024 terms of mixed sign stay below a rounding (2^-24) of every term beyond that.
BOUND = 2.0 ** -22


@pytest.mark.parametrize("B,n,L,d", [(1, 1, 256, 64), (1, 63, 256, 60), (5, 13, 260, 68), (2, 65, 284, 132), (3, 100, 1024, 192),
                                     (8, 70, 512, 64), (2, 40, 252, 64), (2, 33, 257, 65)])
@pytest.mark.parametrize("wide", [False, True])
def test_products(vd, B, n, L, d, wide):
    g = torch.Generator().manual_seed(B * 1000003 + n * 1009 + L * 31 + d + wide)
    x, We, dxs = (torch.randn(s, generator=g) for s in ((B, n, L), (L, d), (B, n, d)))
    if wide:          # every row and column of a scale of its own
        x = x * torch.exp2(torch.randint(-30, 31, (B, n, 1), generator=g).float())
        We = We * torch.exp2(torch.randint(-30, 31, (1, d), generator=g).float())
        dxs = dxs * torch.exp2(torch.randint(-30, 31, (1, 1, d), generator=g).float())
    xs, dWe = product(vd, x, We, dxs)
    X = x.reshape(B * n, L)
    # Weight gradients over few rows use the fp32 instruction, which rounds the running sum every 2 k, by half a unit
    # (2^-24 of it) at random sign, and that sum can be as large as all terms together (rows of scales of their own make one
    # term the whole of it): four standard deviations of K / 2 such roundings are 4 sqrt(K / 2) 2^-24 / sqrt(3) < 2 sqrt(K) 2^-24.
    assert_close(xs, X, We, BOUND)
    assert_close(dWe, X.T, dxs.reshape(B * n, d), BOUND + 2.0 * (B * n) ** 0.5 * 2.0 ** -24)


def significands(g, shape):
    """Numbers of magnitude [1, 2) and either sign; every fourth has the bits that a split handles worst, 1 + 2^-7 - 2^-23."""
    v = 1.0 + torch.rand(shape, generator=g, dtype=torch.float64)
    v = torch.where(torch.rand(shape, generator=g) < 0.25, torch.full(shape, 1 + 2.0 ** -7 - 2.0 ** -23, dtype=torch.float64), v).float()
    return v * (1.0 - 2.0 * torch.randint(0, 2, shape, generator=g).float())


# One term: 2^-24 for the rounding of the sum of its parts, twice 2^-25 for the products that are not formed (the fp32 instruction:
# 2^-24); the smaller parts' own sums are rounded at 2^-31.
ONE_TERM = 2.0 ** -23 + 2.0 ** -28


@pytest.mark.parametrize("scale", [(0, 0), (-100, 60), (-112, 70), (-118, 100), (-126, 100), (-135, 120), (100, -118), (-60, -62)])
def test_single_terms(vd, scale):
    """One number in every row and column of x, so that each result is one product: nothing covers what the split loses.
    x and the weights (and dxs) at the scales of `scale`, small ones with large ones among them: numbers too small for bf16 parts."""
    n = L = 512
    d = 68
    g = torch.Generator().manual_seed(1000 + scale[0])
    p = torch.randperm(n, generator=g)
    x = torch.zeros(1, n, L)
    x[0, torch.arange(n), p] = significands(g, (n,)) * 2.0 ** scale[0]
    We, dxs = (significands(g, s) * 2.0 ** scale[1] for s in ((L, d), (1, n, d)))
    xs, dWe = product(vd, x, We, dxs)
    assert_close(xs, x[0], We, ONE_TERM)
    assert_close(dWe, x[0].T, dxs[0], ONE_TERM)


@pytest.mark.parametrize("exponents", [(-100, 127), (-149, -100)])
def test_products_with_one_are_exact(vd, exponents):
    """Rows of x with a single 1: the result is the weight itself, so the parts of a number add up to it."""
    n = L = 256
    d = 64
    g = torch.Generator().manual_seed(-exponents[0])
    x = torch.eye(L)[torch.randperm(L, generator=g)][None]
    We, dxs = (torch.ldexp(significands(g, s).double(), torch.randint(*exponents, s, generator=g)).float() for s in ((L, d), (1, n, d)))
    assert bool(torch.isfinite(We).all())
    xs, dWe = product(vd, x, We, dxs)
    assert torch.equal(xs, x[0] @ We) and torch.equal(dWe, x[0].T @ dxs[0])


def test_large_numbers(vd):
    """Numbers next to the largest one, whose upper part rounds to infinity."""
    n = L = 256
    d = 64
    g = torch.Generator().manual_seed(9)
    top = torch.finfo(torch.float32).max
    x = torch.eye(L)[None] * 0.5
    We, dxs = (torch.where(torch.rand(s, generator=g) < 0.1, top, torch.randn(s, generator=g)) for s in ((L, d), (1, n, d)))
    xs, dWe = product(vd, x, We, dxs)
    assert torch.equal(xs, We * 0.5) and torch.equal(dWe, dxs[0] * 0.5)


@pytest.mark.parametrize("n,L", [(200, 64), (200, 512), (300, 64), (520, 512)])
def test_infinities_and_nan(vd, n, L):
    """They reach the results they belong to and no others, as with the fp32 instruction (weight gradients: K = n, by parts
    from 256 on)."""
    g = torch.Generator().manual_seed(L + n)
    d = 128
    x, We, dxs = torch.randn((1, n, L), generator=g), torch.randn((L, d), generator=g), torch.randn((1, n, d), generator=g)
    x[0, 3, 5], x[0, 70, L - 1], x[0, 131, 7] = float("inf"), float("-inf"), float("nan")
    xs, dWe = product(vd, x, We, dxs)
    X, Y = x[0].double(), dxs[0].double()
    rows, ks = torch.ones(n, dtype=torch.bool), torch.ones(L, dtype=torch.bool)
    rows[[3, 70, 131]], ks[[5, L - 1, 7]] = False, False
    # tiles beside a bad row or column: the fp32 instruction, a rounding every 2 k
    assert_close(xs[rows], X[rows], We, 4 * BOUND)
    assert_close(dWe[ks], X.T[ks], Y, 4 * BOUND)
    for row in (3, 70):
        assert torch.equal(xs[row].double(), X[row] @ We.double())
    for row, k in ((3, 5), (70, L - 1)):
        assert torch.equal(dWe[k].double(), X[row, k] * Y[row])
    assert bool(torch.isnan(xs[131]).all()) and bool(torch.isnan(dWe[7]).all())


@pytest.mark.parametrize("L", [64, 512])
def test_overflow(vd, L):
    g = torch.Generator().manual_seed(L)
    n, d = 200, 128
    x, We, dxs = torch.randn((1, n, L), generator=g), torch.randn((L, d), generator=g), torch.randn((1, n, d), generator=g)
    x[0, 150, :] = 3e38
    xs, _ = product(vd, x, We, dxs)
    want = x[0].double() @ We.double()
    clean = torch.ones(n, dtype=torch.bool)
    clean[150] = False
    assert_close(xs[clean], x[0][clean], We, 4 * BOUND)
    assert not bool(torch.isfinite(xs[150][want[150].abs() > 3.5e38]).any())


def test_very_wide_rows(vd):
    """32 rows of the weights span more than 2^32 bytes."""
    L, d = 256, 36_000_000
    if torch.cuda.mem_get_info()[0] < 100 << 30:
        pytest.skip("needs 100 GiB of free device memory")
    g = torch.Generator(device="cuda").manual_seed(1)
    x, We = torch.randn((1, 1, L), generator=g, device="cuda"), torch.randn((L, d), generator=g, device="cuda")
    xs, _ = vd.vardrop_embed_fwd(vd.Context(0), x, torch.zeros(1, dtype=torch.int32, device="cuda"), 1, We, None, False)
    want, scale = (torch.zeros(d, dtype=torch.float64, device="cuda") for _ in range(2))
    for k in range(L):
        want += x[0, 0, k].double() * We[k]
        scale += (x[0, 0, k].double() * We[k]).abs()
    # (the fp32 instruction: 128 roundings of 2^-24 of at most all terms together)
    assert bool(((xs[0, 0] - want).abs() <= 2.0 ** -17 * scale).all())
