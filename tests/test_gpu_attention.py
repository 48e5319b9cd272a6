"""GPU multi-head attention forward/backward against the fp64 oracle.

Tolerance (per tensor): max|gpu - oracle| / max|oracle| <= 2e-2 for bf16, 1e-5 for fp32, and on top of that the
element-wise bounds of util_gpu.elem_err (RMS of the difference, and every element against a relative term plus a
floor proportional to the tensor's RMS), so that small elements are constrained as well.
The oracle receives the same bf16- (or fp32-) representable inputs, converted to fp64.
"""
import numpy as np
import pytest
import torch

import workloads as wl
from util_gpu import TOL, elem_err, oracle_attention, rel_err, to_dev, torch_dtype

pytestmark = pytest.mark.gpu

GRADS = ("dxs", "dWq", "dWk", "dWv", "dWo")


@pytest.fixture(scope="module")
def vd():
    import paper_2501_14183_amd as m
    return m


@pytest.fixture(scope="module")
def ctx(vd):
    return vd.Context(0)


def run_gpu(vd, ctx, xs, W, H, dy, dtype, biases=None):
    td = torch_dtype(dtype)
    xs_t, dy_t = to_dev(xs, td), to_dev(dy, td)
    W_t = [to_dev(w, td) for w in W]
    b_t = [to_dev(b, td) for b in biases] if biases else [None] * 4
    y, saved = vd.vardrop_attn_fwd(ctx, xs_t, *W_t, H, *b_t)
    out = vd.vardrop_attn_bwd(ctx, dy_t, xs_t, *W_t, H, saved, bias_grads=biases is not None)
    torch.cuda.synchronize()
    names = GRADS + (("dbq", "dbk", "dbv", "dbo") if biases else ())
    res = dict(zip(names, out))
    res["y"] = y
    return res


def random_case(seed, B, n, d, dtype, bias):
    rng = np.random.default_rng(seed)
    xs = wl.quantise(rng.standard_normal((B, n, d)), dtype)
    W = [wl.quantise(rng.standard_normal((d, d)) / np.sqrt(d), dtype) for _ in range(4)]
    dy = wl.quantise(rng.standard_normal((B, n, d)), dtype)
    b = [wl.quantise(0.2 * rng.standard_normal(d), dtype) for _ in range(4)] if bias else None
    return xs, W, dy, b


def compare(got, want, dtype, names):
    errs = {k: rel_err(got[k], want[k]) for k in names}
    if "dbk" in names:
        # Softmax does not see a shift of all logits of a row, so the key-bias gradient is identically zero
        # (and with a single token the query-bias gradient too): measure both against a scale that does
        # not vanish, the larger of their own, the query-bias and 1% of the value-bias gradient.
        floor = max(np.abs(want["dbq"]).max(), 1e-2 * np.abs(want["dbv"]).max())
        for k in ("dbq", "dbk"):
            diff = np.abs(got[k].float().cpu().numpy() - want[k]).max()
            errs[k] = float(diff / max(np.abs(want[k]).max(), floor))
    bad = {k: v for k, v in errs.items() if not v <= TOL[dtype]}
    assert not bad, "relative errors above %g: %s (all: %s)" % (TOL[dtype], bad, errs)
    # element-wise (the two bias gradients that vanish identically or nearly so keep the scale chosen above)
    fine = {k: elem_err(got[k], want[k], dtype) for k in names if k not in ("dbq", "dbk")}
    bad = {k: v for k, v in fine.items() if v is not None and not (v[0] <= 1.0 and v[1] <= 1.0)}
    assert not bad, "element-wise bounds exceeded (rms ratio, element ratio; both must be <= 1): %s (all: %s)" % (bad, fine)
    return errs


@pytest.mark.parametrize("name", wl.ORDER)
def test_five_workloads(vd, ctx, name):
    """Tokens of the workload, gathered at the oracle's selection, through attention fwd + bwd."""
    from util_gpu import workload_inputs, workload_selection
    w, x, *_ = workload_inputs(name)
    gid, sel, G = workload_selection(name)
    tok = wl.make_tokens(w, x)
    xs = tok[:, sel, :]
    W = wl.make_weights(w)
    dy = wl.make_upstream(w, len(sel))
    want = oracle_attention(xs, W, w.H, dy)
    got = run_gpu(vd, ctx, xs, W, w.H, dy, w.dtype)
    errs = compare(got, want, w.dtype, ("y",) + GRADS)
    print("%s: n=%d %s" % (name, len(sel), {k: "%.2e" % v for k, v in errs.items()}))


@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 63, 64, 65, 127, 128, 129, 130, 257, 300])
def test_bf16_ragged_token_counts_with_biases(vd, ctx, n):
    xs, W, dy, b = random_case(n, 3, n, 128, "bf16", bias=True)
    want = oracle_attention(xs, W, 2, dy, tuple(b))
    got = run_gpu(vd, ctx, xs, W, 2, dy, "bf16", biases=b)
    compare(got, want, "bf16", ("y",) + GRADS + ("dbq", "dbk", "dbv", "dbo"))


@pytest.mark.parametrize("n", [129, 188, 192, 200, 256, 257, 321])
def test_bf16_ragged_token_counts_in_the_wide_launch_shape(vd, ctx, n):
    """Enough (batch, head) pairs that the long-selection kernels run with four wavefronts and 128 rows per
    workgroup (the shape the large workloads use), at token counts that end a block of 64 and of 128 early, the first
    count past the single-kernel path (129) and the token count the paper reports for Traffic (188, Table 3)."""
    xs, W, dy, b = random_case(1000 + n, 32, n, 512, "bf16", bias=False)
    want = oracle_attention(xs, W, 8, dy)
    got = run_gpu(vd, ctx, xs, W, 8, dy, "bf16")
    compare(got, want, "bf16", ("y",) + GRADS)


@pytest.mark.parametrize("B,n,d,H", [(4, 150, 192, 3), (8, 100, 320, 5), (6, 90, 64, 1), (2, 130, 64, 1), (3, 200, 320, 5)])
def test_bf16_model_widths_off_the_tile_grid(vd, ctx, B, n, d, H):
    """d is a multiple of 64 but not of the 128-wide GEMM tiles; B*n large enough for sliced weight gradients; more
    than 128 tokens with one head and with an odd head count (the dO product then forms the row sums of dO * O)."""
    xs, W, dy, b = random_case(7 * d + n, B, n, d, "bf16", bias=True)
    want = oracle_attention(xs, W, H, dy, tuple(b))
    got = run_gpu(vd, ctx, xs, W, H, dy, "bf16", biases=b)
    compare(got, want, "bf16", ("y",) + GRADS + ("dbq", "dbk", "dbv", "dbo"))


@pytest.mark.parametrize("B,n,d,H", [(1, 5, 16, 1), (2, 70, 64, 2), (3, 33, 128, 2), (2, 9, 128, 1), (4, 10, 64, 2)])
def test_fp32_head_sizes_and_biases(vd, ctx, B, n, d, H):
    xs, W, dy, b = random_case(d + n, B, n, d, "fp32", bias=True)
    want = oracle_attention(xs, W, H, dy, tuple(b))
    got = run_gpu(vd, ctx, xs, W, H, dy, "fp32", biases=b)
    compare(got, want, "fp32", ("y",) + GRADS + ("dbq", "dbk", "dbv", "dbo"))


@pytest.mark.parametrize("B,n,d,H,dtype", [(1, 127, 64, 1, "bf16"), (1, 128, 64, 1, "bf16"), (3, 43, 576, 9, "bf16"),
                                           (33, 129, 128, 2, "bf16"), (1, 129, 272, 17, "fp32"), (65, 64, 32, 2, "fp32")])
def test_bias_gradients_over_row_slices(vd, ctx, B, n, d, H, dtype):
    """Column sums of 127 rows (one slice), 128 and 129 (two, the second one row short or not), more columns than a
    workgroup takes at once, and the largest number of slices."""
    xs, W, dy, b = random_case(B + n, B, n, d, dtype, bias=True)
    want = oracle_attention(xs, W, H, dy, tuple(b))
    got = run_gpu(vd, ctx, xs, W, H, dy, dtype, biases=b)
    compare(got, want, dtype, ("dbq", "dbk", "dbv", "dbo"))


@pytest.mark.parametrize("B,n,d", [(7, 150, 192), (40, 129, 256), (86, 193, 512)])
def test_gradients_do_not_depend_on_the_place_in_the_batch(vd, ctx, B, n, d):
    """Equal windows get equal bits wherever they lie in the batch: 64- and 128-row tiles of dO, windows that share tiles."""
    xs, W, dy, _ = random_case(B + n, 1, n, d, "bf16", bias=False)
    td = torch.bfloat16
    rep = lambda a: to_dev(a, td).expand(B, n, d).contiguous()
    xs_t, dy_t, W_t = rep(xs), rep(dy), [to_dev(w, td) for w in W]
    y, saved = vd.vardrop_attn_fwd(ctx, xs_t, *W_t, d // 64)
    dxs = vd.vardrop_attn_bwd(ctx, dy_t, xs_t, *W_t, d // 64, saved)[0]
    assert torch.equal(y, y[:1].expand_as(y)) and torch.equal(dxs, dxs[:1].expand_as(dxs))


@pytest.mark.parametrize("B,n,d", [(1, 1, 64), (1, 63, 64), (3, 43, 192), (5, 129, 128), (32, 145, 128), (65, 160, 256), (20, 480, 512)])
def test_bias_gradients_beside_the_weight_gradients(vd, ctx, B, n, d):
    """bf16 column sums come from the tiles of the weight gradients, at 32 x 145 x 128 from launches of their own: K slices of one row to several slices, a last slice a row short
    or over, few- and many-token tiles, a width whose last tile is half empty.  dbo = colsum(dy) against float64 (sums of some
    1e4 positive terms in groups of four: below 1e-6); with the count on the device and with one sum left out the same bits."""
    xs, W, dy, _ = random_case(B + n, B, n, d, "bf16", bias=False)
    td = torch.bfloat16
    xs_t, W_t, dy_t = to_dev(xs, td), [to_dev(w, td) for w in W], to_dev(np.abs(dy), td)
    H = d // 64
    y, saved = vd.vardrop_attn_fwd(ctx, xs_t, *W_t, H)
    out = vd.vardrop_attn_bwd(ctx, dy_t, xs_t, *W_t, H, saved, bias_grads=True)
    want = dy_t.double().reshape(-1, d).sum(0)
    assert ((out[8].double() - want).abs() / want).max().item() <= 1e-6
    ws = torch.empty(vd.load_library().vardrop_attn_workspace_bytes(B, n, d, H, vd.BF16), dtype=torch.uint8, device="cuda")
    n_dev = torch.tensor([n], dtype=torch.int32, device="cuda")
    again = [torch.full_like(t, float("nan")) for t in out]
    again[6] = None
    vd.vardrop_attn_bwd_dev(ctx, dy_t, xs_t, n_dev, n, *W_t, H, saved, ws, tuple(again))
    assert all(b is None or torch.equal(a, b) for a, b in zip(out, again))


@pytest.mark.parametrize("B,n,d,H", [(2, 32, 64, 1), (2, 33, 64, 1), (1, 128, 128, 1), (2, 129, 32, 2), (3, 97, 192, 3),
                                     (1, 257, 128, 1), (2, 65, 96, 3), (4, 128, 64, 1), (9, 300, 80, 5)])
def test_fp32_matrix_core_tiles(vd, ctx, B, n, d, H):
    """Token blocks of 32 and 128 ended exactly and one past, all head sizes, widths off the 64-wide product tiles, and
    weight gradients in one K slice (up to 291 rows), two (512) and ten with a short last one (2700)."""
    xs, W, dy, b = random_case(3 * d + n, B, n, d, "fp32", bias=True)
    want = oracle_attention(xs, W, H, dy, tuple(b))
    got = run_gpu(vd, ctx, xs, W, H, dy, "fp32", biases=b)
    compare(got, want, "fp32", ("y",) + GRADS + ("dbq", "dbk", "dbv", "dbo"))


@pytest.mark.parametrize("d", [64, 128])
def test_weight_gradients_of_many_rows_stay_in_their_workspace(vd, ctx, d):
    """37152 rows of one column of tiles: nine partial products per weight, one more than any wider model has, with a host
    and a device-side count.  What lies behind the workspace stays as it was."""
    B, n, H, dtype = 288, 129, d // 64, "bf16"
    xs, W, dy, _ = random_case(d, B, n, d, dtype, bias=False)
    want = oracle_attention(xs, W, H, dy)
    td = torch_dtype(dtype)
    xs_t, dy_t, W_t = to_dev(xs, td), to_dev(dy, td), [to_dev(w, td) for w in W]
    need = vd.load_library().vardrop_attn_workspace_bytes(B, n, d, H, vd.BF16)
    status = torch.zeros(1, dtype=torch.int32, device="cuda")
    n_dev = torch.full((1,), n, dtype=torch.int32, device="cuda")
    y, saved = vd.vardrop_attn_fwd(ctx, xs_t, *W_t, H)
    for device_count in (False, True):
        buf = torch.full((need + (4 << 20),), 0x5A, dtype=torch.uint8, device="cuda")   # (a partial product more would fit)
        out = (torch.empty_like(xs_t), *[torch.empty((d, d), device="cuda") for _ in range(4)])
        if device_count:
            vd.vardrop_attn_bwd_dev(ctx, dy_t, xs_t, n_dev, n, *W_t, H, saved, buf[:need], out, status=status)
        else:
            vd.vardrop_attn_bwd(ctx, dy_t, xs_t, *W_t, H, saved, ws=buf[:need], out=out)
        torch.cuda.synchronize()
        assert int(status[0]) == 0 and bool((buf[need:] == 0x5A).all())
        compare(dict(zip(GRADS, out), y=y), want, dtype, ("y",) + GRADS)


@pytest.mark.parametrize("B,d", [(73, 384), (76, 384), (190, 256), (192, 256), (36, 704), (37, 704)])
def test_gradient_launch_on_both_sides_of_its_rounds(vd, ctx, B, d):
    """129 tokens a window: the last row counts whose many-token workgroups fit the chip in one round and the first that
    take the few-token tiles instead (in three, six and two slices)."""
    xs, W, dy, _ = random_case(B + d, B, 129, d, "bf16", bias=False)
    want = oracle_attention(xs, W, d // 64, dy)
    got = run_gpu(vd, ctx, xs, W, d // 64, dy, "bf16")
    compare(got, want, "bf16", ("y",) + GRADS)


def test_dense_mode_equals_identity_selection(vd, ctx):
    """Inference path of the paper: no variate dropped, all N tokens attend."""
    w = wl.WORKLOADS["electricity"]
    from util_gpu import workload_inputs
    _, x, *_ = workload_inputs("electricity")
    tok = wl.make_tokens(w, x)[:4]
    W = wl.make_weights(w)
    dy = wl.make_upstream(w, w.N)[:4]
    want = oracle_attention(tok, W, w.H, dy)
    got = run_gpu(vd, ctx, tok, W, w.H, dy, "bf16")
    compare(got, want, "bf16", ("y",) + GRADS)


def test_softmax_with_large_logits_stays_finite(vd, ctx):
    xs, W, dy, _ = random_case(1, 2, 40, 64, "bf16", bias=False)
    xs = wl.quantise(xs * 30.0, "bf16")                     # logits of a few hundred: one-hot-like rows
    want = oracle_attention(xs, W, 1, dy)
    got = run_gpu(vd, ctx, xs, W, 1, dy, "bf16")
    assert all(torch.isfinite(v.float()).all() for v in got.values())
    assert rel_err(got["y"], want["y"]) <= 5e-2             # near-ties between keys amplify bf16 rounding of Q, K


# (bf16: the kernel of short selections below 129 tokens, those of long ones from there on)
@pytest.mark.parametrize("sign", [-1.0, 1.0])
@pytest.mark.parametrize("n,d,H,dtype", [(5, 16, 1, "fp32"), (33, 32, 1, "fp32"), (33, 64, 1, "fp32"), (33, 128, 1, "fp32"), (40, 96, 3, "fp32"),
                                         (129, 16, 1, "fp32"), (129, 256, 2, "fp32"), (31, 64, 1, "bf16"), (129, 128, 2, "bf16"), (200, 64, 1, "bf16")])
def test_all_logits_of_every_query_far_from_zero(vd, ctx, n, d, H, dtype, sign):
    """Every logit lies near -110 (or 110), where exp(-logit) of an absent key's zero score overflows, at token counts
    that end a block of keys early.  The last dimension of a head is a constant of Q and of K, so the others behave as
    usual."""
    B, dk = 2, d // H
    xs, W, dy, b = random_case(n + d, B, n, d, dtype, bias=True)
    const = np.arange(d) % dk == dk - 1
    a = np.ceil(np.sqrt(110.0 * np.sqrt(dk)))                    # a whole number: a bf16 value too
    W[0][:, const] = W[1][:, const] = 0.0
    b[0][const], b[1][const] = a, sign * a
    want = oracle_attention(xs, W, H, dy, tuple(b))
    got = run_gpu(vd, ctx, xs, W, H, dy, dtype, biases=b)
    assert all(torch.isfinite(v.float()).all() for v in got.values())
    for name in ("dWq", "dWk"):                                  # (the constants' columns cancel to rounding)
        got[name], want[name] = got[name][:, to_dev(~const)], want[name][:, ~const]
    # A score and a log-sum-exp of magnitude a^2 / sqrt(dk) carry a few roundings of 2^-24 of it into the exponent, so
    # that much relative error enters every probability, on top of what the tensors have anyway.
    tol = TOL[dtype] + 8.0 * (a * a / np.sqrt(dk)) * 2.0 ** -24
    errs = {k: rel_err(got[k], want[k]) for k in ("y",) + GRADS}
    assert all(e <= tol for e in errs.values()), (tol, errs)


@pytest.mark.parametrize("dtype", ["bf16", "fp32"])
@pytest.mark.parametrize("B,n,bias", [(2, 1, False), (3, 61, True), (2, 128, False), (2, 129, True), (5, 300, False)])
def test_saved_holds_q_k_v(vd, ctx, dtype, B, n, bias):
    """`saved` begins with Q, K and V as documented.  Weights that permute and scale by powers of two, and biases of a few
    bits, leave one rounding: that of the result."""
    d, H = 128, 2
    rng = np.random.default_rng(n)
    td = torch_dtype(dtype)
    xs = wl.quantise(rng.standard_normal((B, n, d)), "bf16")
    W = [np.eye(d)[rng.permutation(d)] * 2.0 ** rng.integers(-2, 3, d) for _ in range(4)]
    b = [rng.integers(-8, 9, d) / 4.0 for _ in range(4)] if bias else [np.zeros(d)] * 4
    args = [to_dev(w, td) for w in W] + [H] + ([to_dev(v, td) for v in b] if bias else [])
    y, saved = vd.vardrop_attn_fwd(ctx, to_dev(xs, td), *args)
    torch.cuda.synchronize()
    got = saved[:3 * B * n * d * y.element_size()].view(td).reshape(3, B, n, d).cpu()
    for z in range(3):
        assert torch.equal(got[z], torch.from_numpy(xs @ W[z] + b[z]).float().to(td)), "QKV"[z]


@pytest.mark.parametrize("B,n", [(2, 129), (2, 192), (3, 300), (256, 300)])
def test_softmax_reference_moves_between_key_blocks(vd, ctx, B, n):
    """Scores that leave the reference taken in an earlier block of 64 keys behind: by less than what the forward lets
    pass, by more, by enough to overflow an exponential, and back down (two and four wavefronts per workgroup).
    Wq = Wk = 1, so Q and K hold the tokens exactly and the usual bounds apply to what follows the scores."""
    rng = np.random.default_rng(n + B)
    xs = 0.5 * rng.standard_normal((B, n, 64))
    top = np.array([1.0, 5.0, 25.0, 150.0, 2.0])[np.arange(n) // 64]
    xs[:, :, 0] = top * rng.uniform(-1.0, 1.0, (B, n))
    xs = wl.quantise(xs, "bf16")
    W = [np.eye(64), np.eye(64)] + [wl.quantise(rng.standard_normal((64, 64)) / 8.0, "bf16") for _ in range(2)]
    dy = wl.quantise(rng.standard_normal((B, n, 64)), "bf16")
    want = oracle_attention(xs, W, 1, dy)
    got = run_gpu(vd, ctx, xs, W, 1, dy, "bf16")
    compare(got, want, "bf16", ("y", "dWv", "dWo"))


def placed_logits(seed, B, n, x0):
    """One head whose logit for key j is x0[j] plus noise of standard deviation 1/4: Q's first dimension is 8, K's is x0,
    held exactly."""
    rng = np.random.default_rng(seed)
    xs = 0.5 * rng.standard_normal((B, n, 64))
    xs[:, :, 0], xs[:, :, 1] = x0, 8.0
    Wq, Wk = np.eye(64), np.eye(64)
    Wq[0] = Wk[1] = Wq[1] = 0.0
    Wq[1, 0] = 1.0
    Wv, Wo = (wl.quantise(rng.standard_normal((64, 64)) / 8.0, "bf16") for _ in range(2))
    Wv[0] = Wv[1] = 0.0
    return wl.quantise(xs, "bf16"), [Wq, Wk, Wv, Wo], wl.quantise(rng.standard_normal((B, n, 64)), "bf16")


def check_placed(got, want, gradients):
    """All finite, y, dWv and dWo within the usual bounds, and the gradients that go through the probabilities within the
    RMS bound, the placed dimension apart from the others: it is 16 times as large.  (The worst element has no bound
    against a tensor's RMS here, since tokens differ by the weight they take, and what belongs to the constant token
    dimension vanishes identically, a row of dS summing to zero, so that only rounding is left of it.)"""
    assert all(torch.isfinite(v.float()).all() for v in got.values())
    compare(got, want, "bf16", ("y", "dWv", "dWo"))
    if gradients:
        for k, cut in (("dxs", (np.s_[..., 2:], np.s_[..., 0])), ("dWq", (np.s_[2:, 1:], np.s_[2:, 0])),
                       ("dWk", (np.s_[2:, 1:], np.s_[2:, 0]))):
            for at in cut:
                rms, _ = elem_err(got[k][at], want[k][at], "bf16")
                assert rms <= 1.0, (k, at, rms)


@pytest.mark.parametrize("B", [2, 256])
@pytest.mark.parametrize("slope", [0.02, 0.05, 0.125, 0.5, 2.0, -0.125])
def test_logits_that_rise_over_the_keys(vd, ctx, B, slope):
    """The reference is left behind a little, enough to move, and beyond an exponential's range in every block of 64 keys
    (and never, when they fall).  Up to 0.5 a key several neighbours share the weight; with 2 the last key has nearly all
    of it, and what is left of dQ and dK is rounding."""
    n = 270
    j = np.arange(n)
    xs, W, dy = placed_logits(int(1000 * slope) % 977, B, n, slope * (j - (n - 1) if slope > 0 else j))
    want = oracle_attention(xs, W, 1, dy)
    check_placed(run_gpu(vd, ctx, xs, W, 1, dy, "bf16"), want, gradients=slope <= 0.5)


@pytest.mark.parametrize("at", [64, 130, 199])
@pytest.mark.parametrize("above", [7.5, 9.0, 11.0, 12.5, 14.0, 20.0, 140.0])
def test_one_key_above_all_before_it(vd, ctx, above, at):
    """A single key of a later block `above` (log2) over the others: its probability alone is let pass up to 2^13, moves the
    reference beyond that, and would overflow.  From 11 on it takes nearly all the weight."""
    x0 = np.zeros(200)
    x0[at] = above * np.log(2.0)
    xs, W, dy = placed_logits(at, 3, 200, x0)
    want = oracle_attention(xs, W, 1, dy)
    check_placed(run_gpu(vd, ctx, xs, W, 1, dy, "bf16"), want, gradients=above <= 9.0)


def test_determinism(vd, ctx):
    xs, W, dy, _ = random_case(9, 4, 130, 512, "bf16", bias=False)
    a = run_gpu(vd, ctx, xs, W, 8, dy, "bf16")
    b = run_gpu(vd, ctx, xs, W, 8, dy, "bf16")
    for k in a:
        assert torch.equal(a[k], b[k]), k


def test_empty_and_error_cases(vd, ctx):
    d, H = 64, 1
    W = [torch.zeros((d, d), dtype=torch.bfloat16, device="cuda") for _ in range(4)]
    xs = torch.zeros((2, 0, d), dtype=torch.bfloat16, device="cuda")
    y, saved = vd.vardrop_attn_fwd(ctx, xs, *W, H)
    out = vd.vardrop_attn_bwd(ctx, xs, xs, *W, H, saved)
    assert y.shape == (2, 0, d) and all(float(t.abs().sum()) == 0 for t in out[1:])
    with pytest.raises(vd.VarDropError) as e:                                   # d_k = 32 is not built for bf16
        vd.vardrop_attn_fwd(ctx, torch.zeros((1, 4, 64), dtype=torch.bfloat16, device="cuda"), *W, 2)
    assert e.value.code == -4
    with pytest.raises(vd.VarDropError) as e:                                   # H does not divide d
        vd.vardrop_attn_fwd(ctx, torch.zeros((1, 4, 64), dtype=torch.bfloat16, device="cuda"), *W, 3)
    assert e.value.code == -1


def test_bf16_backward_is_bit_reproducible(vd, ctx):
    """Sliced weight gradients are summed in a fixed order, whichever workgroup finishes last: equal bits on every call."""
    xs, W, dy, _ = random_case(77, 8, 113, 512, "bf16", bias=False)
    first = run_gpu(vd, ctx, xs, W, 8, dy, "bf16")
    for _ in range(3):
        again = run_gpu(vd, ctx, xs, W, 8, dy, "bf16")
        for k in GRADS + ("y",):
            assert torch.equal(first[k], again[k]), k
