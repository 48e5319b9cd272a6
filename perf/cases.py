"""Performance cases of the VarDrop hot path: what a training or inference program calls, over its range of sizes.

A case is one of five programs ("path"), all through the public calls of paper_2501_14183_amd:

  step     one training step with the count of kept tokens on the device: vardrop_hash -> vardrop_sample ->
           vardrop_gather_attn_fwd_dev -> vardrop_attn_bwd_dev (-> vardrop_scatter_dev when the embedding in front is
           trained too); with "embed" the tokens are formed inside the step from the raw windows
           (vardrop_embed_fwd_dev / vardrop_embed_bwd_dev around the attention)
  dense    attention forward and backward over all N variate tokens, with biases: training without dropping
  infer    attention forward over all N variate tokens: what the trained model runs when it forecasts
  embed    token embedding of a host-known selection from raw windows, forward and weight gradients
  select   fixed representatives: spectra and hashes of a time-major batch, then vardrop_sample_nearest

Windows are sums of sinusoids of shared templates plus noise, as in `workloads`, made on the GPU.  A template's
components lie on bins of the window and are well separated in amplitude, so that rounding decides no rank.
"""
import math

import torch

import paper_2501_14183_amd as vd


def listed():
    return [
        # The smallest problem of the repository (4 windows, 32 variates, fp32): unit tests, first runs; launches count.
        dict(name="step_tiny_fp32", path="step", B=4, N=32, L=96, k=3, gs=0, num=1, den=4, templates=4, own=0,
             d=64, H=2, dtype="fp32", embed=False, scatter=False),
        # A small dataset (137 variates, 20 members a group) trained in fp32 at the full model width.
        dict(name="step_solar_fp32", path="step", B=32, N=137, L=96, k=3, gs=20, num=1, den=1, templates=5, own=6,
             d=512, H=8, dtype="fp32", embed=False, scatter=False),
        # The two everyday training shapes at their configured keep ratios (about 90 and 115 kept tokens).
        dict(name="step_electricity", path="step", B=32, N=321, L=96, k=3, gs=0, num=1, den=5, templates=30, own=17,
             d=512, H=8, dtype="bf16", embed=False, scatter=False),
        dict(name="step_traffic", path="step", B=32, N=862, L=96, k=3, gs=0, num=1, den=10, templates=30, own=17,
             d=512, H=8, dtype="bf16", embed=False, scatter=False),
        # The same data under Eq. 1 as printed (k = 4, gs = 10; about 190 kept tokens) with a trained embedding in
        # front of the path, so that the token gradients of all variates are wanted.
        dict(name="step_traffic_gs10", path="step", B=32, N=862, L=96, k=4, gs=10, num=1, den=1, templates=18, own=17,
             d=512, H=8, dtype="bf16", embed=False, scatter=True),
        # The everyday shape with the embedding of the kept variates inside the step.
        dict(name="step_traffic_embed", path="step", B=32, N=862, L=96, k=3, gs=0, num=1, den=10, templates=30, own=17,
             d=512, H=8, dtype="bf16", embed=True, scatter=False),
        # Longer windows and more variates; about 240 kept tokens.
        dict(name="step_long", path="step", B=16, N=2048, L=336, k=4, gs=0, num=1, den=10, templates=61, own=0,
             d=512, H=8, dtype="bf16", embed=False, scatter=False),
        # The largest: 8192 variates, 512 samples, about 1950 kept tokens, width 768.
        dict(name="step_stress", path="step", B=8, N=8192, L=512, k=5, gs=0, num=1, den=20, templates=256, own=1500,
             d=768, H=12, dtype="bf16", embed=False, scatter=False),
        # Training without dropping at 321 variates, with biases and their gradients (what the method is compared with).
        dict(name="dense_electricity", path="dense", B=32, N=321, d=512, H=8, dtype="bf16"),
        # Forecasting with all 862 variates.
        dict(name="infer_traffic", path="infer", B=32, N=862, d=512, H=8, dtype="bf16"),
        # Embedding of kept variates from long windows (720 samples is the usual long lookback), with bias.
        dict(name="embed_720", path="embed", B=16, N=862, L=720, n=188, d=512, dtype="bf16"),
        # Choosing fixed representatives once per epoch from a time-major loader batch.
        dict(name="select_nearest", path="select", B=16, N=2048, L=336, k=4, gs=0, num=1, den=10, templates=61, own=60,
             dtype="fp32"),
    ]


# ------------------------------------------------------------------------------------------------ sizes
def _group_sizes(c):
    """Sizes of the groups the generator plants: templates of falling popularity, then variates of their own.  Each has
    an ordered tuple of bins to itself while there are enough of them; from then on they share the tuples in turn."""
    T = min(c["templates"], c["N"])
    own = min(c["own"], c["N"] - T)
    weights = [1.0 / (i + 4) for i in range(T)]
    rest = c["N"] - own - T
    sizes = [1 + int(rest * w / sum(weights)) for w in weights]
    for i in range(c["N"] - own - sum(sizes)):
        sizes[i % T] += 1
    sizes += [1] * own
    total = math.perm(_candidates(c["L"]), c["k"])
    return [sum(sizes[i::total]) for i in range(min(total, len(sizes)))]


def _kept(c):
    """Kept tokens N': the same for every seed."""
    cap = c["gs"] or c["N"]
    return sum(min(g, cap, max(1, -(-g * c["num"] // c["den"]))) for g in _group_sizes(c))


def _es(c):
    return 2 if c["dtype"] == "bf16" else 4


def _candidates(L):
    return (L // 2 + 2) // 2          # the library's default cut-off: half of the positive frequencies, rounded up


def _hash_work(c):
    B, N, L, k = c["B"], c["N"], c["L"], c["k"]
    return 4.0 * B * N * L + N * (8.0 + 4.0 * k), 2.5 * B * N * L * math.log2(L)


def _attn_work(B, n, d, es, backward, biases):
    M = float(B * n)
    nbytes = 2 * M * d * es + 4 * d * d * es + (4 * d * es if biases else 0)       # xs, y, weights
    flops = 8 * M * d * d + 4 * M * n * d
    if backward:
        nbytes += 2 * M * d * es + 16.0 * d * d + (16.0 * d if biases else 0)      # dy, dxs, weight gradients
        flops += 16 * M * d * d + 8 * M * n * d
    return nbytes, flops


def work(c):
    es = _es(c)
    if c["path"] in ("dense", "infer"):
        nbytes, flops = _attn_work(c["B"], c["N"], c["d"], es, c["path"] == "dense", True)
    elif c["path"] == "embed":
        M = float(c["B"] * c["n"])
        nbytes = 4 * M * c["L"] + 2 * M * c["d"] * es + c["L"] * c["d"] * (es + 4)
        flops = 4 * M * c["L"] * c["d"]
    elif c["path"] == "select":
        nbytes, flops = _hash_work(c)
        nbytes += c["N"] * (4.0 * _candidates(c["L"]) + 4) + 4.0 * _kept(c)
        flops += 4.0 * c["N"] * _candidates(c["L"])
    else:
        n = _kept(c)
        M = float(c["B"] * n)
        nbytes, flops = _hash_work(c)
        a_bytes, a_flops = _attn_work(c["B"], n, c["d"], es, True, False)
        nbytes += 4.0 * c["N"] + 4.0 * n + a_bytes
        flops += a_flops
        if c["embed"]:
            nbytes += M * c["d"] * es + c["L"] * c["d"] * (es + 4)
            flops += 4 * M * c["L"] * c["d"]
        else:
            nbytes += M * c["d"] * es                                                # the kept tokens read
        if c["scatter"]:
            nbytes += float(c["B"]) * c["N"] * c["d"] * es
    return {"bytes": nbytes, "flops": flops}


def _cost(c):
    """Seconds at the card's nominal rates: what draws are bounded by."""
    w = work(c)
    return w["bytes"] / 8e12 + w["flops"] / (2.5e15 if c["dtype"] == "bf16" else 1.5e14)


def tolerance(c):
    # About four times the worst output of the listed cases against the same path in float64 from the same inputs:
    # bf16 4.5e-3 relative and 2.7e-2 of the RMS (or of the value) for one element, fp32 1.3e-6 and 9.2e-6, mean
    # amplitudes 5e-8 and 3e-7 (summed in another order they differ by a few times that).
    if c["path"] == "select":
        return {"rel": 1e-6, "max": 1e-5}
    if c["dtype"] == "bf16":
        return {"rel": 1.8e-2, "max": 1.1e-1}
    return {"rel": 5e-6, "max": 4e-5}


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    most = max(_cost(c) for c in listed())
    while True:
        path = rng.choice(("step", "step", "step", "step", "step", "dense", "infer", "embed", "select"))
        c = dict(path=path, B=log_int(1, 64), N=log_int(12, 8192))
        fp32 = path == "select" or rng.random() < 0.2
        if path in ("step", "select"):
            c.update(L=log_int(32, 768), k=rng.randint(1, 5))
            if rng.random() < 0.5:
                c["L"] = rng.choice((48, 96, 168, 192, 336, 512, 720))
            if rng.random() < 0.5:
                c.update(gs=rng.choice((1, 2, 5, 10, 20)), num=1, den=1)
            else:
                c.update(gs=0, num=1, den=rng.randint(2, 20))
            c.update(templates=log_int(2, max(3, c["N"] // 8)), own=int(c["N"] * rng.uniform(0.0, 0.2)))
        if path == "embed":
            c.update(L=8 * log_int(6, 96))
            c.update(n=min(c["N"], log_int(4, 2048)))
        if path != "select":
            dk = rng.choice((16, 32, 64, 128)) if fp32 else 64
            c["d"] = dk * rng.randint(1, 1024 // dk) if fp32 else 64 * rng.randint(1, 16)
            if path != "embed":
                c["H"] = c["d"] // dk
        c["dtype"] = "fp32" if fp32 else "bf16"
        if path == "step":
            c["embed"] = not fp32 and rng.random() < 0.25
            if c["embed"]:
                c["L"] = 8 * (min(c["L"], 376) // 8)
            c["scatter"] = not c["embed"] and rng.random() < 0.25
        if "templates" in c and _kept(c) < 8:          # scores of a few tokens cancel to rounding noise in the gradients
            continue
        if _cost(c) <= most and c["B"] * c["N"] * max(c.get("d", 1), c.get("L", 1)) <= 8 * 8192 * 768:
            return c


# ------------------------------------------------------------------------------------------------ inputs
DEV = "cuda"


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(1000003 * (int(seed) + 1))
    return g


def _windows(c, g, time_major=False):
    """float32 windows [B, N, L]: variate n is scale_n (sum of k + 1 sinusoids of its template + noise) + offset_n."""
    B, N, L, m = c["B"], c["N"], c["L"], c.get("k", 3) + 1
    F = _candidates(L)
    order = torch.rand((F,), generator=g, device=DEV).argsort() + 1
    if "templates" in c:
        # group i leads with the ordered tuple number (step * i + first) of all ordered tuples of bins
        sizes, total = _group_sizes(c), math.perm(F, c["k"])
        step = next(a for a in range(1 + int(0.381966 * total), 2 * total) if math.gcd(a, total) == 1)
        number = (torch.arange(len(sizes), device=DEV) * step + g.initial_seed() % total) % total
        free = torch.ones((len(sizes), F), dtype=torch.int64, device=DEV)
        at = []
        for j in range(c["k"]):
            digit, number = number % (F - j), number // (F - j)
            at.append(((free.cumsum(1) == digit[:, None] + 1) & (free == 1)).int().argmax(1))
            free.scatter_(1, at[j][:, None], 0)
        at.append(free.argmax(1))
        bins = order[torch.stack(at, 1)]
    else:
        sizes = [1] * N
        bins = torch.rand((N, F), generator=g, device=DEV).argsort(1)[:, :m] + 1
    amp = torch.empty((len(sizes), 1), device=DEV).uniform_(1.0, 2.0, generator=g) * 1.5 ** -torch.arange(m, device=DEV)
    of = torch.repeat_interleave(torch.arange(len(sizes), device=DEV), torch.tensor(sizes, device=DEV))
    of = of[torch.randperm(N, generator=g, device=DEV)]
    phase = 6.2831853 * torch.rand((B, N, m), generator=g, device=DEV)
    x = 0.05 * torch.randn((B, N, L), generator=g, device=DEV)
    t = torch.arange(L, device=DEV)
    for j in range(m):
        f = bins[of, j]
        arg = (6.2831853 / L) * (f[:, None] * t[None, :] % L)
        x += amp[of, j][None, :, None] * torch.sin(arg[None] + phase[:, :, j, None])
    scale = torch.empty(N, device=DEV).uniform_(-1.0, 1.0, generator=g).exp_()
    x = x * scale[None, :, None] + torch.randn(N, generator=g, device=DEV)[None, :, None]
    return x.transpose(1, 2).contiguous().transpose(1, 2) if time_major else x


def _prepare_attention(c, g, s, n, biases):
    """Weights and what the calls write: buffers for at most n tokens a window."""
    B, d, H = c["B"], c["d"], c["H"]
    td = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    code = vd.BF16 if c["dtype"] == "bf16" else vd.F32
    lib = vd.load_library()
    s["H"] = H
    s["W"] = [(torch.randn((d, d), generator=g, device=DEV) / math.sqrt(d)).to(td) for _ in range(4)]
    s["b"] = [(0.1 * torch.randn(d, generator=g, device=DEV)).to(td) if biases else None for _ in range(4)]
    s["saved"] = torch.empty(lib.vardrop_attn_saved_bytes(B, n, d, H, code), dtype=torch.uint8, device=DEV)
    s["ws"] = torch.empty(max(256, lib.vardrop_attn_workspace_bytes(B, n, d, H, code)), dtype=torch.uint8, device=DEV)
    s["dy"] = torch.randn((B, n, d), generator=g, device=DEV).to(td)
    s["xs"], s["y"], s["dxs"] = (torch.zeros((B, n, d), dtype=td, device=DEV) for _ in range(3))
    s["dW"] = [torch.zeros((d, d), device=DEV) for _ in range(4)]
    # One buffer for the four bias gradients: the one of the keys is zero but for rounding (softmax does not see a
    # shift of a row's logits), so it is compared at the scale of the four.
    s["db"] = torch.zeros((4, d), device=DEV)


def _embedding(c, g, td):
    L, d = c["L"], c["d"]
    return ((torch.randn((L, d), generator=g, device=DEV) / math.sqrt(L)).to(td),
            (0.1 * torch.randn(d, generator=g, device=DEV)).to(td))


def prepare(case, seed):
    c, g = case, _gen(seed)
    td = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    s = {"path": c["path"], "ctx": vd.Context(0), "seed": int(seed)}
    lib = vd.load_library()
    if c["path"] in ("dense", "infer"):
        n = c["N"]
        _prepare_attention(c, g, s, n, True)
        s["xs"] = torch.randn((c["B"], n, c["d"]), generator=g, device=DEV).to(td)
        s["grads"] = (s["dxs"], *s["dW"], *s["db"])
        return s
    if c["path"] == "embed":
        s["x"] = _windows(c, g)
        s["n"], s["L"] = c["n"], c["L"]
        s["sel"] = torch.randperm(c["N"], generator=g, device=DEV)[: c["n"]].sort().values.to(torch.int32)
        s["We"], s["be"] = _embedding(c, g, td)
        s["dxs"] = torch.randn((c["B"], c["n"], c["d"]), generator=g, device=DEV).to(td)
        code = vd.BF16 if c["dtype"] == "bf16" else vd.F32
        s["saved"] = torch.empty(lib.vardrop_embed_saved_bytes(c["B"], c["n"], c["L"], code), dtype=torch.uint8, device=DEV)
        s["ws"] = torch.empty(max(256, lib.vardrop_embed_workspace_bytes(c["B"], c["n"], c["L"], c["d"], code)),
                              dtype=torch.uint8, device=DEV)
        s["xs"] = torch.zeros((c["B"], c["n"], c["d"]), dtype=td, device=DEV)
        s["dWe"] = (torch.zeros((c["L"], c["d"]), device=DEV), torch.zeros(c["d"], device=DEV))
        return s
    s["rule"] = (c["gs"], c["num"], c["den"])
    s["k"], s["L"] = c["k"], c["L"]
    if c["path"] == "select":
        s["x"] = _windows(c, g, time_major=True)
        s["ws"] = torch.empty(lib.vardrop_hash_strided_workspace_bytes(c["B"], c["N"], c["L"]), dtype=torch.uint8, device=DEV)
        s["n"] = _kept(c)
        return s
    N = c["N"]
    s["x"] = _windows(c, g)
    s["topk"] = torch.zeros((N, c["k"]), dtype=torch.int32, device=DEV)
    s["hash"] = torch.zeros(N, dtype=torch.int64, device=DEV)
    s["gid"], s["sel"] = (torch.zeros(N, dtype=torch.int32, device=DEV) for _ in range(2))
    s["counts"] = torch.zeros(2, dtype=torch.int32, device=DEV)
    s["status"] = torch.zeros(1, dtype=torch.int32, device=DEV)
    # A program knows its token counts from a first selection and sizes its buffers for 128 tokens or whole blocks of 64.
    _select(s)
    n = _kept(c)
    n_max = 128 if c["dtype"] == "bf16" and n <= 128 <= N else min(N, -(-n // 64) * 64)
    s["n_max"] = n_max
    _prepare_attention(c, g, s, n_max, False)
    s["grads"] = (s["dxs"], *s["dW"])
    We, be = _embedding(c, g, td)
    if c["embed"]:
        s["We"], s["be"] = We, be
        code = vd.BF16
        s["esaved"] = torch.empty(lib.vardrop_embed_saved_bytes(c["B"], n_max, c["L"], code), dtype=torch.uint8, device=DEV)
        s["ews"] = torch.empty(max(256, lib.vardrop_embed_workspace_bytes(c["B"], n_max, c["L"], c["d"], code)),
                               dtype=torch.uint8, device=DEV)
        s["dWe"] = (torch.zeros((c["L"], c["d"]), device=DEV), torch.zeros(c["d"], device=DEV))
    else:
        # tokens of all variates, as the embedding in front of the path leaves them
        x = s["x"]
        z = (x - x.mean(-1, keepdim=True)) / x.std(-1, keepdim=True, unbiased=False)
        s["tokens"] = torch.addmm(be, z.to(td).reshape(-1, c["L"]), We).reshape(c["B"], N, c["d"])
    if c["scatter"]:
        s["dtokens"] = torch.zeros((c["B"], N, c["d"]), dtype=td, device=DEV)
    # What the calls write is packed at the front of the buffers: views of that part, for the outputs.
    packed = [s[name].view(-1)[: c["B"] * n * c["d"]].view(c["B"], n, c["d"]) for name in ("xs", "y", "dxs")]
    s["out"] = [s["topk"], s["hash"], s["gid"], s["sel"][:n], s["counts"], s["status"], *packed, *s["dW"]]
    s["out"] += [*s["dWe"]] if c["embed"] else []
    s["out"] += [s["dtokens"]] if c["scatter"] else []
    return s


# ------------------------------------------------------------------------------------------------ one pass
def _select(s):
    vd.vardrop_hash(s["ctx"], s["x"], s["k"], out=(s["topk"], s["hash"]))
    vd.vardrop_sample(s["ctx"], s["hash"], *s["rule"], s["seed"], 1, out=(s["gid"], s["sel"], s["counts"]))


def _select_nearest(s):
    topk, hsh, abar = vd.vardrop_hash(s["ctx"], s["x"], s["k"], want_abar=True, ws=s["ws"])
    gid, sel, counts = vd.vardrop_sample_nearest(s["ctx"], hsh, abar, *s["rule"])
    return topk, hsh, abar, gid, sel, counts


def _run_step(s):
    _select(s)
    ctx, sel, n, n_max, H, W, status = s["ctx"], s["sel"], s["counts"], s["n_max"], s["H"], s["W"], s["status"]
    if "We" in s:
        vd.vardrop_embed_fwd_dev(ctx, s["x"], sel, n, n_max, s["We"], s["be"], s["xs"], s["esaved"], status=status)
        vd.vardrop_attn_fwd_dev(ctx, s["xs"], n, n_max, *W, H, s["y"], s["saved"], status=status)
    else:
        vd.vardrop_gather_attn_fwd_dev(ctx, s["tokens"], sel, n, n_max, *W, H, s["xs"], s["y"], s["saved"], status=status)
    vd.vardrop_attn_bwd_dev(ctx, s["dy"], s["xs"], n, n_max, *W, H, s["saved"], s["ws"], s["grads"], status=status)
    if "We" in s:
        vd.vardrop_embed_bwd_dev(ctx, s["dxs"], n, n_max, s["L"], s["esaved"], s["ews"], s["dWe"])
    if "dtokens" in s:
        vd.vardrop_scatter_dev(ctx, s["dxs"], sel, n, n_max, s["dtokens"], status=status)
    return s["out"]


def run(state):
    s = state
    if s["path"] == "step":
        return _run_step(s)
    if s["path"] == "select":
        topk, hsh, abar, gid, sel, counts = _select_nearest(s)
        return topk, hsh, abar, gid, sel[: s["n"]], counts
    if s["path"] == "embed":
        xs, saved = vd.vardrop_embed_fwd(s["ctx"], s["x"], s["sel"], s["n"], s["We"], s["be"], saved=s["saved"], out=s["xs"])
        dWe, dbe = vd.vardrop_embed_bwd(s["ctx"], s["dxs"], s["L"], saved, ws=s["ws"], out=s["dWe"])
        return xs, dWe, dbe
    bq, bk, bv, bo = s["b"]
    y, saved = vd.vardrop_attn_fwd(s["ctx"], s["xs"], *s["W"], s["H"], bq, bk, bv, bo, saved=s["saved"], out=s["y"])
    if s["path"] == "infer":
        return y
    dxs, dWq, dWk, dWv, dWo, *_ = vd.vardrop_attn_bwd(s["ctx"], s["dy"], s["xs"], *s["W"], s["H"], saved, bias_grads=True,
                                                     ws=s["ws"], out=s["grads"])
    return y, dxs, dWq, dWk, dWv, dWo, s["db"]
