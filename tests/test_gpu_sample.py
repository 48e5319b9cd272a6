"""GPU grouping + stratified sampling (vardrop_sample) against the oracle: bit-exact."""
import numpy as np
import pytest
import torch

import workloads as wl
from oracle import sampling as o_samp

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def vd():
    import paper_2501_14183_amd as m
    return m


@pytest.fixture(scope="module")
def ctx(vd):
    return vd.Context(0)


def run(vd, ctx, hashes, gs, num, den, seed, step, pinned=None):
    h = torch.from_numpy(np.asarray(hashes, dtype=np.uint64).view(np.int64)).cuda()
    gid, sel, counts = vd.vardrop_sample(ctx, h, gs, num, den, seed, step, counts_host=pinned)
    torch.cuda.synchronize()
    n_sel, G = (int(v) for v in counts.cpu())
    return gid.cpu().numpy().astype(np.int64), sel.cpu().numpy()[:n_sel].astype(np.int64), n_sel, G


def check(vd, ctx, hashes, gs, num, den, seed, step):
    want_gid, want_sel, want_G = o_samp.stratified_sample(hashes, gs, num, den, seed, step)
    gid, sel, n_sel, G = run(vd, ctx, hashes, gs, num, den, seed, step)
    assert G == want_G and n_sel == len(want_sel)
    assert np.array_equal(gid, want_gid)
    assert np.array_equal(sel, want_sel)
    return gid, sel


@pytest.mark.parametrize("name", wl.ORDER)
def test_five_workloads_bit_exact(vd, ctx, name):
    from util_gpu import workload_inputs, SEED, STEP
    w, x, info, topk, hsh, abar = workload_inputs(name)
    gid, sel = check(vd, ctx, hsh, 0, w.ratio[0], w.ratio[1], SEED, STEP)           # the configured keep ratio
    sizes = np.bincount(gid)
    kept = np.bincount(gid[sel], minlength=len(sizes))
    assert np.all(kept >= 1)
    assert kept.tolist() == [o_samp.keep_count(int(g), 0, *w.ratio) for g in sizes]
    for gs in (1, 5, 10, 20):                                                       # Eq. 1 as printed
        gid, sel = check(vd, ctx, hsh, gs, 1, 1, SEED, STEP + gs)
        kept = np.bincount(gid[sel], minlength=len(sizes))
        assert kept.tolist() == [min(int(g), gs) for g in sizes]
    print("%s: G=%d N'=%d delta=%.4f" % (name, len(sizes), len(sel), o_samp.reduction_ratio(w.N, len(sel))))


@pytest.mark.parametrize("N,n_distinct", [(1, 1), (2, 1), (3, 3), (64, 5), (65, 7), (129, 129), (1000, 40),
                                          (4097, 300), (8192, 1), (8192, 8192), (8191, 977)])
def test_sizes_and_degenerate_groupings(vd, ctx, N, n_distinct):
    rng = np.random.default_rng(N + n_distinct)
    pool = rng.integers(0, 2 ** 63, size=n_distinct, dtype=np.uint64)
    if n_distinct == N:
        hashes = rng.permutation(np.unique(rng.integers(0, 2 ** 63, size=4 * N, dtype=np.uint64))[:N])
    else:
        hashes = pool[rng.integers(0, n_distinct, size=N)]
    check(vd, ctx, hashes, 0, 1, 10, seed=N, step=3)
    check(vd, ctx, hashes, 3, 1, 1, seed=2 ** 63 + 5, step=2 ** 40 + N)
    check(vd, ctx, hashes, 7, 2, 3, seed=1, step=0)
    gid, sel = check(vd, ctx, hashes, 0, 1, 1, seed=1, step=1)
    assert sel.tolist() == list(range(N))                                           # nothing dropped


def test_extreme_hash_values_and_new_selection_every_step(vd, ctx):
    hashes = np.array([2 ** 64 - 1, 0, 2 ** 63, 2 ** 64 - 1, 0, 1, 2 ** 64 - 2] * 9, dtype=np.uint64)
    check(vd, ctx, hashes, 2, 1, 1, 11, 12)
    sels = set()
    for step in range(20):
        _, sel = check(vd, ctx, hashes, 2, 1, 1, 99, step)
        sels.add(tuple(sel.tolist()))
    assert len(sels) > 10


def test_counts_reach_pinned_host_memory_and_runs_are_deterministic(vd, ctx):
    rng = np.random.default_rng(0)
    hashes = rng.integers(0, 50, size=3000).astype(np.uint64)
    pinned = torch.zeros(2, dtype=torch.int32).pin_memory()
    a = run(vd, ctx, hashes, 4, 1, 3, 5, 6, pinned=pinned)
    assert pinned.tolist() == [a[2], a[3]]
    b = run(vd, ctx, hashes, 4, 1, 3, 5, 6)
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


@pytest.mark.parametrize("N", [63, 192, 193, 255, 256, 257, 1024, 1025, 2047, 2048, 2049, 4096, 5000])
@pytest.mark.parametrize("bits", [17, 32, 33, 40, 57, 64])
def test_counts_at_launch_boundaries_and_hash_widths(vd, ctx, N, bits):
    """Sizes at which the launch shape changes or a workgroup's share ends early, with hashes of every width class:
    among the widest, neighbours that agree in the 32 topmost bits in use and differ below, one large group, singletons."""
    rng = np.random.default_rng(N * 100 + bits)
    top = rng.integers(0, 2 ** min(bits, 32), size=max(2, N // 40), dtype=np.uint64) << np.uint64(max(0, bits - 32))
    low = rng.integers(0, 3, size=N, dtype=np.uint64) if bits > 34 else np.zeros(N, dtype=np.uint64)
    hashes = top[rng.integers(0, len(top), size=N)] + low
    hashes[rng.random(N) < 0.3] = top[0]
    hashes[N // 2] = np.uint64(2 ** bits - 1)
    check(vd, ctx, hashes, 0, 1, 7, seed=bits, step=N)
    check(vd, ctx, hashes, 4, 1, 1, seed=3, step=2 ** 33)


def test_both_launches_of_a_sample_carry_one_signal_and_one_time(vd, ctx):
    h = torch.arange(1000, device="cuda") % 90
    kid = {vd.vardrop_kernel_name(k): k for k in range(64) if vd.vardrop_kernel_name(k)}["sample"]
    want = vd.vardrop_sample(ctx, h, 0, 1, 5, 1, 2)
    out = tuple(torch.full_like(t, -1) for t in want)
    copy = torch.empty_like(out[2])
    main, side = torch.cuda.Stream(), torch.cuda.Stream()
    ev = torch.cuda.Event()
    ev.record(main)
    torch.cuda.synchronize()
    vd.vardrop_signal_after(ctx, kid, ev.cuda_event)
    vd.vardrop_sample(ctx, h, 0, 1, 5, 1, 2, out=out, stream=main.cuda_stream)
    side.wait_event(ev)
    with torch.cuda.stream(side):
        copy.copy_(out[2])                      # the counts: what the second launch writes
    side.synchronize()
    assert copy.tolist() == want[2].tolist()
    main.synchronize()
    n = int(copy[0])
    assert torch.equal(out[0], want[0]) and torch.equal(out[1][:n], want[1][:n])
    vd.vardrop_profile_select(ctx, kid)
    for _ in range(3):
        vd.vardrop_sample(ctx, h, 0, 1, 5, 1, 2, out=out, stream=main.cuda_stream)
    main.synchronize()
    ms, launches = vd.vardrop_profile_read(ctx)
    vd.vardrop_profile_select(ctx, -1)
    print("sample: %.2f us" % (1e3 * ms / launches))
    assert launches == 3 and ms > 0


def test_error_codes(vd, ctx):
    h = torch.zeros(10, dtype=torch.int64, device="cuda")
    for args, code in [((0, 2, 1, 0, 0), -1), ((0, 1, 0, 0, 0), -1)]:
        with pytest.raises(vd.VarDropError) as e:
            vd.vardrop_sample(ctx, h, *args)
        assert e.value.code == code
    with pytest.raises(vd.VarDropError) as e:
        vd.vardrop_sample(ctx, torch.zeros(8193, dtype=torch.int64, device="cuda"), 0, 1, 1, 0, 0)
    assert e.value.code == -4


# ---------------------------------------------------------------- deterministic representatives
U32 = 2.0 ** -24          # unit round-off of IEEE single precision


def single_precision_error_bound(abar, gid, G, d):
    """A-priori bound on |d_kernel[n] - d[n]| for a kernel that evaluates the distances in single precision:
    the group mean as a running sum of g members and a division (relative error <= g u), the difference, its
    square, and a running sum over F bins.  With t = a - mean:  |dt| <= g u mean + u |t|, so
        E[n] = u (2 g sum_f |t_f| mean_f + (3 + F) d[n]).
    """
    A = np.asarray(abar, dtype=np.float64)
    F = A.shape[1]
    E = np.zeros(len(gid))
    for g in range(G):
        members = np.nonzero(gid == g)[0]
        mean = A[members].mean(axis=0)
        t = np.abs(A[members] - mean)
        E[members] = U32 * (2.0 * len(members) * (t * mean).sum(axis=1) + (3.0 + F) * d[members])
    return E


def check_nearest(vd, ctx, hashes, abar, gs, num, den):
    """The oracle states the sampler in float64; the kernel evaluates the distances in single precision.  Where
    floating point decides an integer, the comparison is exact wherever the decision is clear of the kernel's
    rounding: a group is `decided` when the distance gap at its keep boundary (between the n_i-th and the
    (n_i + 1)-th closest member) exceeds four times the summed error bounds of the two members, or the two
    members have identical spectra (the tie rule decides in any arithmetic).  Decided groups must match the
    oracle bit for bit; in the others every kept member must be within the bound of the boundary, and the
    number of members that differ is returned."""
    abar32 = np.ascontiguousarray(abar, dtype=np.float32)
    want_gid, want_sel, want_G = o_samp.representative_sample(hashes, abar32, gs, num, den)
    h = torch.from_numpy(np.asarray(hashes, dtype=np.uint64).view(np.int64)).cuda()
    gid, sel, counts = vd.vardrop_sample_nearest(ctx, h, torch.from_numpy(abar32).cuda(), gs, num, den)
    torch.cuda.synchronize()
    n_sel, G = (int(v) for v in counts.cpu())
    assert G == want_G and n_sel == len(want_sel)
    gid = gid.cpu().numpy().astype(np.int64)
    sel = sel.cpu().numpy()[:n_sel].astype(np.int64)
    assert np.array_equal(gid, want_gid)
    assert np.all(np.diff(sel) > 0)
    d = o_samp.spectrum_distances(abar32, want_gid, want_G)
    E = single_precision_error_bound(abar32, want_gid, want_G, d)
    got, want = set(sel.tolist()), set(want_sel.tolist())
    flips = undecided = 0
    for g in range(want_G):
        members = np.nonzero(want_gid == g)[0].tolist()
        n_i = o_samp.keep_count(len(members), gs, num, den)
        kept = [n for n in members if n in got]
        assert len(kept) == n_i
        order = sorted(members, key=lambda n: (d[n], n))
        decided = True
        if n_i < len(members):
            a, b = order[n_i - 1], order[n_i]
            identical = np.array_equal(abar32[a], abar32[b])
            decided = identical or (d[b] - d[a]) > 4.0 * (E[a] + E[b])
        if decided:
            assert kept == sorted(order[:n_i]), "group %d" % g
        else:
            undecided += 1
            limit = d[order[n_i - 1]]
            for n in kept:
                if n not in want:
                    flips += 1
                    assert d[n] <= limit + 4.0 * (E[n] + E[order[n_i - 1]])
    return flips, undecided, want_G


@pytest.mark.parametrize("name", wl.ORDER)
def test_representatives_of_the_five_workloads(vd, ctx, name):
    """Hashes and mean amplitude spectra from the oracle's k-DFH (rounded once to float32, which both sides
    receive): the kept members match the oracle's float64 evaluation in every group whose keep boundary is clear
    of single-precision rounding, under the keep ratio and under Eq. 1 with gs = 1."""
    import util_gpu
    w, x, info, topk, hsh, abar = util_gpu.workload_inputs(name)
    for gs, num, den in ((0, w.ratio[0], w.ratio[1]), (1, 1, 1)):
        flips, undecided, G = check_nearest(vd, ctx, hsh, abar, gs, num, den)
        print("%s gs=%d ratio=%d/%d: %d groups, %d undecided by the gap screen, %d members differ"
              % (name, gs, num, den, G, undecided, flips))
        assert undecided <= 2 + G // 4          # the screen must leave most groups to the exact comparison


@pytest.mark.parametrize("N,F,n_distinct,gs,num,den", [(1, 1, 1, 0, 1, 1), (5, 3, 1, 2, 1, 1), (64, 25, 5, 0, 1, 3),
                                                       (129, 7, 129, 1, 1, 1), (1000, 85, 40, 5, 1, 1),
                                                       (3000, 129, 7, 0, 1, 10)])
def test_representatives_sizes_ties_and_large_groups(vd, ctx, N, F, n_distinct, gs, num, den):
    rng = np.random.default_rng([N, F, n_distinct])
    pool = rng.integers(0, 2 ** 62, size=n_distinct, dtype=np.uint64)
    h = pool[rng.integers(0, n_distinct, size=N)]
    A = np.abs(rng.standard_normal((N, F))) + 1.0
    A[::3] = A[0]                                   # many identical spectra: ties go to the lower index
    check_nearest(vd, ctx, h, A, gs, num, den)


@pytest.mark.parametrize("N", [255, 256, 257, 513, 1024, 1025, 1280, 1281, 2305])
def test_representatives_groups_across_blocks_of_variates(vd, ctx, N):
    """Group lists are made from blocks of 256 variates, four at a time and the last one alone: groups that begin and end at either side
    of a block, one that spans all."""
    rng = np.random.default_rng(N)
    h = np.full(N, 3, dtype=np.uint64)
    for i, at in enumerate(range(255, N, 256)):
        h[at - 2:at + 3] = 10 + i
    h[-1] = h[N // 2] = 7
    A = np.abs(rng.standard_normal((N, 19))) + 1.0
    check_nearest(vd, ctx, h, A, 0, 1, 4)
    check_nearest(vd, ctx, h, A, 2, 1, 1)


def test_representatives_clear_gaps_are_exact(vd, ctx):
    """Members at well separated distances from the group mean (geometric spacing): every group is decided, so the
    selection equals the oracle's exactly."""
    rng = np.random.default_rng(77)
    N, F, n_groups = 600, 25, 30
    h = rng.integers(0, n_groups, size=N).astype(np.uint64)
    centre = rng.uniform(5.0, 10.0, (n_groups, F))
    direction = rng.standard_normal((N, F))
    direction /= np.linalg.norm(direction, axis=1, keepdims=True)
    radius = 0.01 * 1.3 ** rng.permutation(N).astype(np.float64).__mod__(20)      # twenty radii, ratio 1.3
    radius = radius * (1.0 + 0.02 * rng.random(N))
    A = centre[h.astype(np.int64)] + radius[:, None] * direction
    for gs, num, den in ((1, 1, 1), (3, 1, 1), (0, 1, 4)):
        flips, undecided, G = check_nearest(vd, ctx, h, A, gs, num, den)
        assert flips == 0


def test_representatives_error_codes(vd, ctx):
    lib = vd.load_library()
    h = torch.zeros(4, dtype=torch.int64, device="cuda")
    A = torch.ones((4, 3), device="cuda")
    out = [torch.empty(4, dtype=torch.int32, device="cuda") for _ in range(2)] + [torch.empty(2, dtype=torch.int32, device="cuda")]
    rc = lib.vardrop_sample_nearest(ctx.handle, h.data_ptr(), A.data_ptr(), 4, 3, 0, 1, 1, out[0].data_ptr(), out[1].data_ptr(),
                                    out[2].data_ptr(), None, None, 0, None)
    assert rc == -2                                 # no workspace
    ws = torch.empty(4096, dtype=torch.uint8, device="cuda")
    rc = lib.vardrop_sample_nearest(ctx.handle, h.data_ptr(), A.data_ptr(), 4, 3, 0, 2, 1, out[0].data_ptr(), out[1].data_ptr(),
                                    out[2].data_ptr(), None, ws.data_ptr(), ws.numel(), None)
    assert rc == -1                                 # ratio above one
