"""fp32 products on bf16 parts (K of 256 and more) and on the fp32 instruction, through the fp32 embedding, against fp64."""
import numpy as np
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


# 2^-22: the three dropped products of parts are at most 3 * 2^-24 of a term; sums of up to 1024 terms of mixed sign stay
# far below a rounding (2^-24) of every term.
BOUND = 2.0 ** -22


@pytest.mark.parametrize("B,n,L,d", [(1, 1, 256, 64), (1, 63, 256, 60), (5, 13, 260, 68), (2, 65, 284, 132), (3, 100, 1024, 192),
                                     (8, 70, 512, 64), (2, 40, 252, 64), (2, 33, 257, 65)])
@pytest.mark.parametrize("wide", [False, True])
def test_products(vd, B, n, L, d, wide):
    g = torch.Generator().manual_seed(B * 1000003 + n * 1009 + L * 31 + d + wide)
    x, We, dxs = (torch.randn(s, generator=g) for s in ((B, n, L), (L, d), (B, n, d)))
    if wide:          # every row, column and k of a scale of its own: the parts of a number must carry all of its bits
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


@pytest.mark.parametrize("L", [64, 512])
def test_infinities_and_nan(vd, L):
    """They reach the results they belong to and no others, as with the fp32 instruction."""
    g = torch.Generator().manual_seed(L)
    n, d = 200, 128
    x, We, dxs = torch.randn((1, n, L), generator=g), torch.randn((L, d), generator=g), torch.randn((1, n, d), generator=g)
    x[0, 3, 5], x[0, 70, L - 1], x[0, 131, 7] = float("inf"), float("-inf"), float("nan")
    x[0, 150, :] = 3e38                                                       # overflows
    xs, dWe = product(vd, x, We, dxs)
    X = x[0]
    want = X.double() @ We.double()
    clean = torch.ones(n, dtype=torch.bool)
    clean[[3, 70, 131, 150]] = False
    assert_close(xs[clean], X[clean], We, 4 * BOUND)      # tiles beside a bad row: the fp32 instruction, a rounding every 2 k
    for row in (3, 70):
        assert torch.equal(xs[row].double(), want[row])
    assert bool(torch.isnan(xs[131]).all()) and not bool(torch.isfinite(xs[150][want[150].abs() > 3.5e38]).any())
    bad_k = ~torch.isfinite(X.double().T @ dxs[0].double()).all(1) | (X.abs().max(0).values > 1e38)
    assert not bool(torch.isfinite(dWe[[5, 7, L - 1]]).any())
    assert bool(bad_k[[5, 7, L - 1]].all())


def test_split_is_exact():
    """The three parts of a finite fp32 number (upper halves of the number and of what is left of it, twice) add up to it."""
    rng = np.random.default_rng(1)
    x = (rng.standard_normal(100000) * np.exp2(rng.integers(-90, 100, 100000))).astype(np.float32)
    upper = lambda v: (v.view(np.uint32) & np.uint32(0xffff0000)).view(np.float32)
    hi = upper(x)
    mid = upper(x - hi)
    lo = upper((x - hi) - mid)
    assert np.array_equal(hi.astype(np.float64) + mid + lo, x.astype(np.float64))
