"""GPU: kernel variants and dispatch rules at the edges of their tiles.

Each test compares a kernel that a rule selects with the general path of the
same library (itself checked against the oracle in test_gpu_parity.py) or with
the oracle, at sizes where tiles, remainders and window widths can go wrong.
"""
import numpy as np
import pytest

import oracle as O
from paper_2407_03608_amd import inputs
from tests.gpu_common import cuda, host, max_rel, oracle_params, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gp():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2407_03608_amd import gp as g
    g.load()
    return g


def _matvec(gp, prob, a, **kw):
    P = gp.Plan(cuda(prob.x), cuda(prob.sigma), cuda(prob.l), prob.nu, prob.eta, **kw)
    return host(P.matvec(cuda(a), add_noise=True)), P.info()


# Sums of w^d N_sigma products in another order: below 4e-14 (fp64, 343 terms of
# rounding 1.1e-16) and 2e-5 (fp32, 6e-8) of the largest value, with a factor for
# the cancellation among the weights w_k.
ORDER_FP64 = 2e-13
ORDER_FP32 = 3e-5


@pytest.mark.parametrize("d,n,M,tol,prec", [
    # window widths of fp64 and fp32 plans, points dense enough for staged blocks
    (2, 1500, 24, 1e-2, 0), (2, 1500, 24, 1e-5, 0), (2, 1700, 30, 1e-8, 0), (2, 1300, 40, 1e-11, 0),
    (2, 1500, 24, 1e-2, 1), (2, 2100, 40, 1e-4, 1), (2, 1500, 33, 1e-6, 1),
    # the same grids with few points: a group of lanes per point
    (2, 1, 24, 1e-8, 0), (2, 37, 60, 1e-8, 0), (2, 37, 60, 1e-4, 1),
    (3, 4000, 8, 1e-2, 0), (3, 6000, 10, 1e-6, 0), (3, 3000, 10, 1e-9, 0), (3, 25, 12, 1e-8, 0),
    (3, 4000, 8, 1e-2, 1), (3, 6000, 12, 1e-4, 1), (3, 9000, 9, 1e-6, 1), (3, 25, 12, 1e-4, 1),
    (1, 1, 20, 1e-8, 0), (1, 300, 150, 1e-3, 1), (1, 777, 9000, 1e-8, 0), (1, 5000, 60, 1e-12, 0),
])
def test_interp_default_matches_per_bin(gp, d, n, M, tol, prec):
    """The default interpolation (staged blocks or lane groups, by density)
    against the per-bin kernel, on clustered and uniform points."""
    for clustered in (False, True):
        prob = inputs.random_small(d, n, seed=7 * d + n, nu=1.5, lmin=0.1, lmax=0.25)
        if clustered:  # a third of the points in one cell-sized cluster, corners included
            rng = np.random.default_rng(n)
            k = max(1, n // 3)
            prob.x[:k] = 0.5 + 1e-3 * rng.standard_normal((k, d))
            prob.x[0], prob.x[-1] = 0.0, 1.0
        a = np.random.default_rng(1).standard_normal(n)
        got, info = _matvec(gp, prob, a, tol=tol, precision=prec, M=M)
        ref, _ = _matvec(gp, prob, a, tol=tol, precision=prec, M=M, interp=2)
        e = max_rel(got, ref)
        say(f"interp d={d} n={n} w={info['w']} na={info['na']} prec={prec} clustered={clustered}: {e:.2e}")
        assert e <= (ORDER_FP32 if prec else ORDER_FP64), e


@pytest.mark.parametrize("d,M,tol,n_sigma,upsample", [
    (2, 40, 1e-3, 0, 0), (2, 40, 1e-4, 0, 0), (2, 40, 1e-6, 0, 1.25), (2, 40, 1e-4, 9, 0),
    (3, 10, 1e-6, 27, 0), (3, 10, 1e-6, 0, 1.5), (3, 10, 1e-6, 5, 1.5),
])
def test_interp_fp32_joins_rows_in_fp64(gp, d, M, tol, n_sigma, upsample):
    """Staged interpolation of fp32 grids in 2-D, and in 3-D from w = 8 on (w = 7: rows
    of 26 weights on), against the per-bin kernel: both add a window row in fp32, in
    order, and the rows in fp64.  2-D: the same to fp64 rounding.  3-D: the per-bin
    kernel rounds the product of a row's two window values to fp32, an error of at
    most 2^-24 / sqrt(12) of each row's share, of rows of one sign."""
    n = 40000
    prob = inputs.random_small(d, n, seed=3, nu=0.5, lmin=0.1, lmax=0.25, constant_scales=n_sigma == 0)
    kw = dict(tol=tol, nufft_tol=tol, precision=1, M=M, dw=0.25, n_sigma=n_sigma)
    if upsample:
        kw["upsample"] = upsample
    a = np.random.default_rng(1).standard_normal(n)
    got, info = _matvec(gp, prob, a, **kw)
    ref, _ = _matvec(gp, prob, a, interp=2, **kw)
    e = np.sqrt(np.mean((got - ref) ** 2) / np.mean(ref ** 2)) * 2 ** 24
    say(f"fp32 rows d={d} w={info['w']} nk={n_sigma + 1}: {e:.4f} of 2^-24")
    assert d == 2 or info["w"] >= 7
    assert e <= (1e-6 if d == 2 else 2 / np.sqrt(12)), e


@pytest.mark.parametrize("n,M,staged", [(100000, 300, True), (60000, 100, True), (300, 300, False)])
def test_interp_rule_counts_blocks_with_points(gp, n, M, staged):
    """Points in one cluster of a large grid: the staged kernel where its blocks, those
    that hold points, are full (fp32 in 2-D: then the rows are joined as the per-bin kernel
    joins them, to fp64 rounding), lane groups where they are few."""
    prob = inputs.random_small(2, n, seed=4, nu=0.5, lmin=0.1, lmax=0.25, constant_scales=True)
    rng = np.random.default_rng(n)
    prob.x[:] = np.clip(0.4 + 0.01 * rng.standard_normal((n, 2)), 0, 1)
    prob.x[0], prob.x[-1] = 0.0, 1.0
    kw = dict(tol=1e-4, precision=1, M=M, dw=0.25)
    a = rng.standard_normal(n)
    got, info = _matvec(gp, prob, a, **kw)
    ref, _ = _matvec(gp, prob, a, interp=2, **kw)
    e = np.sqrt(np.mean((got - ref) ** 2) / np.mean(ref ** 2)) * 2 ** 24
    say(f"clustered n={n} M={M} na={info['na']}: {e:.4f} of 2^-24")
    assert e <= 1e-6 if staged else 1e-3 < e <= 4, e


@pytest.mark.parametrize("tol,n", [(1e-8, 120000), (1e-9, 120000), (1e-9, 500), (1e-8, 1000000), (1e-9, 1000000)])
def test_interp_wide_windows_3d(gp, tol, n):
    """fp64 in 3-D at w = 9 and 10 below and above the density at which blocks are
    staged: the per-bin kernel's values, in clearly less than its time."""
    prob = inputs.random_small(3, n, seed=6, nu=2.5, lmin=0.3, lmax=0.5)
    a = np.random.default_rng(1).standard_normal(n)
    out, ms = [], []
    for interp in (0, 2):
        P = gp.Plan(cuda(prob.x), cuda(prob.sigma), cuda(prob.l), prob.nu, prob.eta, tol, M=60, dw=0.25, interp=interp)
        v = cuda(a)
        out.append(host(P.matvec(v)))
        P.set_timing(True)
        for _ in range(3):
            P.matvec(v)
        ms.append(P.timing()["interp"][1] / 3)
        P.set_timing(False)
    say(f"3-D w={P.info()['w']} n={n}: {ms[0]:.3f} ms, per-bin kernel {ms[1]:.3f}")
    assert max_rel(out[0], out[1]) <= ORDER_FP64
    if n > 1000:
        assert ms[0] < 0.8 * ms[1], ms


def test_interp_many_points(gp):
    """270 million points (16 lanes each: more threads than one launch can have): outputs
    at both ends and between them against the posterior mean at those points."""
    import torch
    n = 270_000_000
    g = torch.Generator("cuda").manual_seed(0)
    x = torch.rand(n, 1, dtype=torch.float64, device="cuda", generator=g)
    one = torch.ones(n, dtype=torch.float64, device="cuda")
    l = 0.05 * one
    a = torch.randn(n, dtype=torch.float64, device="cuda", generator=g)
    P = gp.Plan(x, one, l, 1.5, 0.1, 1e-8, M=100_000, n_sigma=0)
    assert P.info()["w"] > 8
    y = P.matvec(a)
    i = torch.cat([torch.arange(500), torch.arange(0, n, n // 999), torch.arange(n - 500, n)]).cuda()
    ref = P.posterior_mean(a, x[i].contiguous(), one[i].contiguous(), l[i].contiguous())
    e = float((y[i] - ref).abs().max() / ref.abs().max())
    say(f"{n} points: {e:.2e}")
    assert e <= ORDER_FP64
    P.close()
    del P, x, one, l, a, y
    torch.cuda.empty_cache()


@pytest.mark.parametrize("n,M,tol,prec", [
    (150, 4200, 1e-8, 0), (150, 6200, 1e-8, 0), (90, 15000, 1e-8, 0), (60, 50000, 1e-8, 0),
    (150, 4200, 1e-4, 1), (90, 33000, 1e-4, 1),
])
def test_four_step_against_oracle(gp, n, M, tol, prec):
    """1-D grids over 8192 points: passes over rows of the active box and the
    band of kept modes only, on splits L1 x L2 of several shapes.  A product
    after another one (whose spectrum is still in the grids) has the same bits."""
    prob = inputs.random_small(1, n, seed=M, nu=1.5, lmin=0.1, lmax=0.25)
    P = gp.Plan(cuda(prob.x), cuda(prob.sigma), cuda(prob.l), prob.nu, prob.eta, tol, precision=prec, M=M)
    info = P.info()
    assert info["nf"][0] > 8192
    rng = np.random.default_rng(2)
    a, b = rng.standard_normal(n), rng.standard_normal(n)
    got = host(P.matvec(cuda(a)))
    P.matvec(cuda(1e3 * b))
    assert np.array_equal(got, host(P.matvec(cuda(a))))
    e = max_rel(got, O.ktilde_matvec(oracle_params(info), prob.x, prob.sigma, prob.l, a))
    say(f"four-step nf={info['nf'][0]} M={M} prec={prec}: {e:.2e}")
    assert e <= (2e-4 if prec else 1e-6), e


@pytest.mark.parametrize("d,M,tol,prec", [
    # every remainder of the columns by blocks of 8, lengths 24 .. 1536
    (2, 4, 1e-4, 0), (2, 11, 1e-6, 0), (2, 18, 1e-6, 0), (2, 33, 1e-4, 0), (2, 62, 1e-8, 0), (2, 126, 1e-6, 0),
    (2, 5, 1e-3, 1), (2, 24, 1e-4, 1), (2, 60, 1e-4, 1), (2, 129, 1e-4, 1), (2, 302, 1e-4, 1), (2, 301, 1e-8, 0),
    # 2048 .. 8192: several columns per thread, per workgroup and one (M odd: against blocks
    # of 4 columns, M even: against whole rows)
    (2, 801, 1e-8, 0), (2, 1100, 1e-6, 0), (2, 1701, 1e-6, 0), (2, 2501, 1e-6, 0), (2, 3001, 1e-4, 0),
    (2, 800, 1e-8, 0), (2, 1600, 1e-6, 0), (2, 1702, 1e-6, 0), (2, 2046, 1e-8, 0), (2, 3000, 1e-4, 0),
    (2, 802, 1e-4, 1), (2, 1104, 1e-4, 1), (2, 1905, 1e-4, 1), (2, 2400, 1e-4, 1), (2, 3002, 1e-4, 1),
    (2, 1602, 1e-4, 1), (2, 2046, 1e-4, 1),
    # rows of modes unpadded and padded to whole lines
    (3, 4, 1e-4, 0), (3, 13, 1e-6, 0), (3, 66, 1e-6, 0), (3, 90, 1e-4, 0),
    (3, 5, 1e-3, 1), (3, 71, 1e-4, 1), (3, 116, 1e-4, 1),
])
def test_fft_layouts(gp, d, M, tol, prec):
    """Transforms through blocks of columns (2-D) and padded rows of modes (3-D)
    against the oracle or, at sizes beyond it, against the plan whose byte limit
    leaves no room for them, with the same spreading (the LDS-atomic variant): rows of B
    whole, in 2-D where M is even, or in blocks of 4 columns, and rows of modes unpadded."""
    n = 200 if (2 * M + 1) ** d < 20000 else 20000
    prob = inputs.random_small(d, n, seed=M, nu=1.5, lmin=0.1, lmax=0.25)
    kw = dict(tol=tol, precision=prec, M=M, dw=0.25)
    a = np.random.default_rng(3).standard_normal(n)
    if n == 200:
        got, info = _matvec(gp, prob, a, **kw)
        ref, bar = O.ktilde_matvec(oracle_params(info), prob.x, prob.sigma, prob.l, a), 100 * tol
        ref = ref + prob.eta ** 2 * a
    else:
        kw["spread"] = 1
        got, info = _matvec(gp, prob, a, **kw)
        ref, linfo = _matvec(gp, prob, a, max_device_bytes=info["device_bytes"] - 1, **kw)
        assert linfo["device_bytes"] < info["device_bytes"]
        if d == 2:  # what the limit leaves: rows whole (mc + 1 columns counted) or blocks of 4
            mc, na1 = 2 * M + 1, info["na"][1]
            blocks = info["n_pairs"] * na1 * ((mc + 7) // 8 * 8 - (mc + 1)) * (8 if prec else 16)
            assert info["device_bytes"] - linfo["device_bytes"] == blocks
            assert (mc + 3) // 4 * 4 > mc + 1 or M % 2 == 1
        bar = ORDER_FP32 if prec else ORDER_FP64
    e = max_rel(got, ref)
    say(f"layouts d={d} M={M} nf={info['nf'][0]} na={info['na']} prec={prec}: {e:.2e}")
    assert e <= bar, e


@pytest.mark.parametrize("d,M,n_sigma", [
    # rows of 3, 10, 21, 36, 55, 105, 210 and 300 entries: whole and partial pieces and chunks
    (2, 3, 1), (2, 40, 3), (2, 63, 5), (2, 64, 7), (2, 130, 9), (2, 65, 13), (2, 20, 19), (2, 31, 23),
    (3, 3, 1), (3, 12, 3), (3, 16, 5), (3, 21, 7), (3, 9, 9), (3, 15, 13), (3, 8, 19), (3, 5, 23),
])
def test_mode_rows(gp, d, M, n_sigma):
    """Step 3 with the table's rows staged through LDS against the direct sum over
    the t nodes, and one vector against several (other step-3 kernels in 2-D, more
    transforms per FFT pass): the same bits."""
    n = 500
    prob = inputs.random_small(d, n, seed=M + n_sigma, nu=1.5, lmin=0.1, lmax=0.25)
    kw = dict(tol=1e-6, M=M, dw=0.2, n_sigma=n_sigma)
    a = np.random.default_rng(4).standard_normal(n)
    got, info = _matvec(gp, prob, a, **kw)
    ref, _ = _matvec(gp, prob, a, step3=1, **kw)
    e = max_rel(got, ref)
    say(f"mode rows d={d} M={M} pairs={info['n_pairs']} t nodes={info['n_t']}: {e:.2e}")
    # n_t N_sigma products in another order, cancellation among the w_k as above
    assert e <= ORDER_FP64, e
    P = gp.Plan(cuda(prob.x), cuda(prob.sigma), cuda(prob.l), prob.nu, prob.eta, **kw)
    A, _, _, _ = P.cg_solve_multi(cuda(np.stack([a, prob.y, -a])), tol=1e-14, max_iter=3)
    a1, _ = P.cg_solve(cuda(prob.y), tol=1e-14, max_iter=3)
    assert np.array_equal(host(A)[1], host(a1))


@pytest.mark.parametrize("n", [1, 2, 1023, 1025, 4095, 4096, 4097, 5000])
def test_cg_vector_kernels(gp, n):
    """One launch per iteration up to 4096 points, three beyond: K iterations
    against the same recurrence on the host with the plan's own products, and a
    lockstep solve of two columns (bit for bit the single solves).  Bound: the
    two recurrences differ by the rounding of sums of n terms, amplified over
    K = 4 steps of a well-conditioned system (eta = 1)."""
    prob = inputs.random_small(1, n, seed=n, nu=2.5, lmin=0.1, lmax=0.25, eta=1.0)
    P = gp.Plan(cuda(prob.x), cuda(prob.sigma), cuda(prob.l), prob.nu, prob.eta, 1e-8, M=60)
    y = np.random.default_rng(n).standard_normal((2, n))
    k = min(4, n)
    got = [host(P.cg_solve(cuda(v), tol=1e-15, max_iter=k)[0]) for v in y]
    both = host(P.cg_solve_multi(cuda(y), tol=1e-15, max_iter=k)[0])
    for j in range(2):
        assert np.array_equal(both[j], got[j])
        x, r = np.zeros(n), y[j].copy()
        p, rr = r.copy(), r @ r
        for _ in range(k):
            Ap = host(P.matvec(cuda(p), add_noise=True))
            a = rr / (p @ Ap)
            x += a * p
            r -= a * Ap
            rr, old = r @ r, rr
            p = r + (rr / old) * p
            if rr <= 1e-30 * (y[j] @ y[j]):
                break
        assert max_rel(got[j], x) < 1e-11, (n, j, max_rel(got[j], x))


@pytest.mark.parametrize("n,replace", [(300, 0), (300, 3), (4096, 0), (4097, 0), (4097, 3), (6000, 2)])
def test_cg_stops_once(gp, n, replace):
    """Iterations queued beyond the last one change nothing, whichever parity the last
    has: K iterations with max_iter = K have the bits of the converged solve, and a
    column of a lockstep solve that is done (at once: b = 0, or at another iteration than
    its neighbours) keeps its iterate and its count while the others go on."""
    prob = inputs.random_small(1, n, seed=n, nu=2.5, lmin=0.1, lmax=0.25, eta=0.3)
    P = gp.Plan(cuda(prob.x), cuda(prob.sigma), cuda(prob.l), prob.nu, prob.eta, 1e-8, M=60)
    rng = np.random.default_rng(n)
    smooth = np.sin(3 * prob.x[:, 0])
    B = np.stack([rng.standard_normal(n), np.zeros(n), smooth, smooth + 0.01 * rng.standard_normal(n)])
    counts = set()
    single = []
    for tol in (1e-3, 1e-5, 1e-6, 1e-8):
        for b in B[[0, 2, 3]]:
            full, info = P.cg_solve(cuda(b), tol=tol, max_iter=500, replace_every=replace)
            k = info["iters"]
            counts.add(k % 2)
            if k == 0:
                continue
            try:
                part, pinfo = P.cg_solve(cuda(b), tol=tol, max_iter=k, replace_every=replace)
            except gp.GpError as e:
                raise AssertionError((n, tol, k)) from e
            assert pinfo["iters"] == k and np.array_equal(host(full), host(part))
    assert counts == {0, 1}
    if replace == 0:
        X, iters, _, _ = P.cg_solve_multi(cuda(B), tol=1e-6, max_iter=500)
        single = [P.cg_solve(cuda(b), tol=1e-6, max_iter=500) for b in B]
        assert len({int(i) for i in iters}) > 2
        for j in range(4):
            assert int(iters[j]) == single[j][1]["iters"] and np.array_equal(host(X)[j], host(single[j][0])), j


@pytest.mark.parametrize("d,n,M,n_sigma,tol,prec", [
    # 1 .. 12 grid pairs (one chunk of up to 8, two chunks, a chunk that overlaps the other)
    (1, 700, 60, 1, 1e-8, 0), (1, 700, 5000, 23, 1e-8, 0), (1, 2500, 40, 17, 1e-4, 1), (1, 300, 6, 3, 1e-3, 1),
    (2, 900, 24, 1, 1e-8, 0), (2, 900, 24, 13, 1e-8, 0), (2, 700, 20, 19, 1e-11, 0), (2, 5, 40, 5, 1e-4, 0),
    (2, 900, 24, 1, 1e-4, 1), (2, 900, 24, 3, 1e-4, 1), (2, 900, 30, 9, 1e-6, 1), (2, 900, 30, 15, 1e-3, 1),
    (3, 900, 8, 1, 1e-6, 0), (3, 500, 8, 11, 1e-9, 0), (3, 900, 8, 7, 1e-4, 1), (3, 900, 10, 21, 1e-5, 1),
])
def test_spread_lists_match_atomics(gp, d, n, M, n_sigma, tol, prec):
    """Spreading from sub-tile lists by matrix instructions (whole and split
    lists) against the LDS-atomic variant, uniform points and all in one cell."""
    for clustered in (False, True):
        prob = inputs.random_small(d, n, seed=3 * d + n_sigma, nu=1.5, lmin=0.1, lmax=0.25)
        if clustered:  # lists longer than a chunk beside empty ones
            rng = np.random.default_rng(n)
            prob.x[: n - n // 4] = 0.37 + 1e-4 * rng.standard_normal((n - n // 4, d))
            prob.x[0], prob.x[-1] = 0.0, 1.0
        a = np.random.default_rng(2).standard_normal(n)
        kw = dict(tol=tol, precision=prec, M=M, n_sigma=n_sigma)
        got, info = _matvec(gp, prob, a, **kw)
        ref, _ = _matvec(gp, prob, a, spread=1, **kw)
        # without room for the lists: tiles that filter their source bins
        lean, linfo = _matvec(gp, prob, a, max_device_bytes=info["device_bytes"] - 1, **kw) \
            if _fits_lean(gp, prob, info, kw) else (got, info)
        e, el = max_rel(got, ref), max_rel(lean, ref)
        say(f"spread d={d} n={n} w={info['w']} pairs={info['n_pairs']} prec={prec} clustered={clustered}: "
            f"{e:.2e}, lean {el:.2e} ({linfo['device_bytes']} of {info['device_bytes']} bytes)")
        bar = ORDER_FP32 if prec else ORDER_FP64
        assert e <= bar and el <= bar, (e, el)


def test_spread_many_sub_tiles(gp):
    """A 3-D grid of 1648^3 cells: more than 2^32 / 64 sub-tiles, so that a launch of a
    wavefront each has more threads than one launch can have."""
    n = 3000
    prob = inputs.random_small(3, n, seed=11, nu=1.5, lmin=0.1, lmax=0.25, constant_scales=True)
    prob.x[: n // 2] = 0.5 + 0.5 * prob.x[: n // 2]  # more of them where the sub-tiles' numbers are high
    prob.x[0], prob.x[-1] = 0.0, 1.0
    a = np.random.default_rng(2).standard_normal(n)
    kw = dict(tol=1e-4, precision=1, M=385, dw=0.4)
    got, info = _matvec(gp, prob, a, **kw)
    assert info["na"][0] * info["na"][1] * info["na"][2] / 64 * 64 >= 2 ** 32
    ref, _ = _matvec(gp, prob, a, spread=1, **kw)
    e = max_rel(got, ref)
    say(f"na={info['na']} {info['device_bytes'] / 2**30:.0f} GiB: {e:.2e}")
    assert e <= ORDER_FP32


def _fits_lean(gp, prob, info, kw):
    """Whether the plan without lists is the smaller one (dense points)."""
    kw = dict(kw)
    b = gp.plan_query(cuda(prob.x), cuda(prob.sigma), cuda(prob.l), prob.nu, prob.eta, kw.pop("tol"),
                      max_device_bytes=info["device_bytes"] - 1, **kw)
    return b < info["device_bytes"]


@pytest.mark.parametrize("d,n,M,n_sigma,m,prec", [
    (2, 60000, 24, 13, 6, 0), (1, 30000, 60, 23, 3, 0), (2, 60000, 24, 13, 5, 1), (3, 40000, 8, 7, 4, 0),
])
def test_multi_split_lists_memory(gp, d, n, M, n_sigma, m, prec):
    """Several vectors on a plan whose lists are split (most points in one cell):
    the bits of single solves, and beside the grids and the solver's vectors at most
    64 MB for partial tiles however many vectors there are; single products
    before and after have the same bits."""
    import torch
    rng = np.random.default_rng(n)
    prob = inputs.random_small(d, n, seed=d, nu=1.5, lmin=0.1, lmax=0.25, eta=1.0)
    prob.x[: n - n // 4] = 0.37 + 1e-2 * rng.standard_normal((n - n // 4, d))
    prob.x[0], prob.x[-1] = 0.0, 1.0
    P = gp.Plan(cuda(prob.x), cuda(prob.sigma), cuda(prob.l), prob.nu, prob.eta, 1e-4 if prec else 1e-8,
                precision=prec, M=M, n_sigma=n_sigma)
    info = P.info()
    y = rng.standard_normal((m, n))
    Y = cuda(y)
    before = host(P.matvec(Y[0]))
    torch.cuda.synchronize()
    _trim_pool()
    free = torch.cuda.mem_get_info()[0]
    X = host(P.cg_solve_multi(Y, tol=1e-14, max_iter=2)[0])
    torch.cuda.synchronize()
    used = free - torch.cuda.mem_get_info()[0]
    # grids A, B, B2, C are at most the transform's size each; the solver keeps
    # five vectors per column and torch the result
    cs = 8 if prec else 16
    nf, na, mc = info["nf"][0], info["na"], 2 * info["M"] + 1
    grids = {1: na[0] + 2 * mc, 2: na[0] * na[1] + (max(na) + 8) * (mc + 8) + mc ** 2,
             3: na[0] * na[1] * na[2] + na[2] * na[1] * mc + na[2] * mc ** 2 + mc ** 3}[d]
    if nf > 8192:
        grids = 3 * nf
    bound = m * (info["n_pairs"] * grids * cs + 6 * n * 8) + (64 << 20)
    say(f"multi d={d} prec={prec} m={m}: {used / 2**20:.0f} MB used, {bound / 2**20:.0f} MB allowed")
    assert used <= bound + (32 << 20), (used, bound)  # the pool takes whole blocks
    for j in range(m):
        assert np.array_equal(X[j], host(P.cg_solve(Y[j], tol=1e-14, max_iter=2)[0])), j
    assert np.array_equal(before, host(P.matvec(Y[0])))


@pytest.mark.parametrize("d,n,M,tol,prec,dw,n_sigma,nbytes", [
    # nbytes: what a plan without lists, column blocks and padded rows has always counted
    (1, 2, 20, 1e-08, 0, 0.25, 5, 24528),
    (1, 300, 60, 1e-08, 0, 0.25, 7, 166728),
    (1, 70000, 6200, 1e-08, 0, 0.25, 5, 22915152),
    (1, 5000, 60, 0.0001, 1, 0.25, 5, 697788),
    (2, 2, 3, 0.0001, 0, 0.25, 3, 65772),
    (2, 500, 40, 1e-08, 0, 0.25, 7, 1873576),
    (2, 70000, 130, 1e-06, 0, 0.25, 5, 32328992),
    (2, 500, 41, 0.0001, 1, 0.25, 4, 749500),
    (2, 300, 5, 0.001, 1, 0.45, 3, 400576),
    (2, 300, 3, 0.0001, 1, 0.45, 3, 739596),
    (2, 300, 2, 0.01, 1, 0.45, 3, 261988),
    (2, 300, 6, 1e-05, 1, 0.4, 3, 284880),
    (2, 70000, 100, 0.0001, 1, 0.25, 5, 17676816),
    (3, 2, 4, 0.0001, 0, 0.25, 3, 736500),
    (3, 2000, 12, 1e-06, 0, 0.25, 5, 13639672),
    (3, 70000, 66, 1e-06, 0, 0.25, 5, 1130798784),
    (3, 2000, 12, 0.0001, 1, 0.25, 5, 7017752),
    (3, 300, 3, 0.0001, 1, 0.45, 3, 15828404),
    (3, 300, 2, 0.001, 1, 0.45, 3, 15489120),
    (3, 300, 5, 1e-05, 1, 0.45, 3, 37753460),
    (3, 70000, 64, 0.0001, 1, 0.25, 5, 559441452),
])
def test_byte_limit_admits_plans_without_lists(gp, d, n, M, tol, prec, dw, n_sigma, nbytes):
    """max_device_bytes admits every plan whose form without spreading lists fits."""
    prob = inputs.random_small(d, n, seed=d, nu=1.5, lmin=0.1, lmax=0.25)
    arg = [cuda(prob.x), cuda(prob.sigma), cuda(prob.l), prob.nu, prob.eta, tol]
    kw = dict(precision=prec, M=M, dw=dw, n_sigma=n_sigma)
    assert gp.plan_query(*arg, max_device_bytes=1, **kw) == nbytes
    least = min(nbytes, gp.plan_query(*arg, **kw))  # few points: the form with lists may be the smaller one
    a = cuda(np.random.default_rng(2).standard_normal(n))
    got = host(gp.Plan(*arg, max_device_bytes=nbytes, **kw).matvec(a))
    ref = host(gp.Plan(*arg, **kw).matvec(a))
    assert max_rel(got, ref) <= (ORDER_FP32 if prec else ORDER_FP64)
    with pytest.raises(gp.GpError):
        gp.Plan(*arg, max_device_bytes=least - 1, **kw)


def _hip():
    """The HIP runtime of this process."""
    import ctypes
    return ctypes.CDLL(next(line.split()[-1] for line in open("/proc/self/maps") if "libamdhip64" in line))


def _trim_pool():
    """Hands the memory that the runtime's pool keeps for reuse back to the device."""
    import ctypes
    hip = _hip()
    pool = ctypes.c_void_p()
    assert hip.hipDeviceGetDefaultMemPool(ctypes.byref(pool), 0) == 0
    assert hip.hipMemPoolTrimTo(pool, ctypes.c_size_t(0)) == 0


def test_plan_where_lists_do_not_fit_the_device(gp):
    """A plan without a byte limit on a device whose free memory holds its form without
    spreading lists, but not the one with them: built, as it was before there were
    lists, with the values of the plan with lists."""
    import ctypes

    import torch
    n = 6_000_000
    g = torch.Generator("cuda").manual_seed(1)
    x = torch.rand(n, 3, dtype=torch.float64, device="cuda", generator=g)
    one = torch.ones(n, dtype=torch.float64, device="cuda")
    l = 0.2 * one
    a = torch.randn(n, dtype=torch.float64, device="cuda", generator=g)
    arg = (x, one, l, 2.5, 0.1, 1e-8)
    kw = dict(M=60, dw=0.25, n_sigma=0)
    P = gp.Plan(*arg, **kw)
    full = P.info()["device_bytes"]
    want = P.matvec(a)
    P.close()
    lean = gp.plan_query(*arg, max_device_bytes=1, **kw)
    # what the runtime's pool still holds is not known, so the room shrinks in steps until
    # the form with lists (a few hundred MB more) does not fit any more
    hip, fill = _hip(), []

    def leave(room):
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        _trim_pool()
        p, free = ctypes.c_void_p(), torch.cuda.mem_get_info()[0]
        if free > room:
            assert hip.hipMalloc(ctypes.byref(p), ctypes.c_size_t(free - room)) == 0
            fill.append(p)

    try:
        for k in range(40):
            room = full + (full >> 2) - k * (96 << 20)
            leave(room)
            P = gp.Plan(*arg, **kw)
            info = P.info()
            if info["device_bytes"] == lean:
                break
            P.close()
        say(f"lists at most {full >> 20} MB, without {lean >> 20} MB counted; built without at {room >> 20} MB free")
        assert info["device_bytes"] == lean
        got = P.matvec(a)
        assert float((got - want).abs().max() / want.abs().max()) <= ORDER_FP64
        P.close()
    finally:
        for p in fill:
            assert hip.hipFree(p) == 0


@pytest.mark.parametrize("d,n,m,prec", [(1, 300, 1, 0), (2, 3000, 5000, 0), (2, 900, 40, 1), (3, 500, 300, 0)])
def test_posterior_mean_streams(gp, d, n, m, prec):
    """The targets are read on a stream beside the plan's: they may be written by
    work still queued on the plan's stream, and after a refused call the
    plan gives the same bits as before."""
    import torch
    prob = inputs.random_small(d, n, seed=5 * d, nu=1.5, lmin=0.1, lmax=0.25)
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        P = gp.Plan(cuda(prob.x), cuda(prob.sigma), cuda(prob.l), prob.nu, prob.eta, 1e-6 if prec == 0 else 1e-4,
                    precision=prec, M={1: 100, 2: 40, 3: 12}[d])
        i = np.random.default_rng(6).integers(0, n, m)
        true = [cuda(v[i]) for v in (prob.x, prob.sigma, prob.l)]
        al = cuda(np.random.default_rng(7).standard_normal(n))
        s.synchronize()
        want = host(P.posterior_mean(al, *true))
        work = torch.rand(2048, 2048, device="cuda")
        for _ in range(3):
            t = [v.clone() for v in true]
            t[0].fill_(0.5)
            s.synchronize()
            for _ in range(20):
                work = work @ work
                work = work / work.abs().max()
            t[0].copy_(true[0])
            got = P.posterior_mean(al, *t)
            assert np.array_equal(host(got), want)
            bad = true[0].clone()
            bad[m // 2, 0] = 7.0
            with pytest.raises(gp.GpError):
                P.posterior_mean(al, bad, *true[1:])


def test_posterior_mean_plans_and_threads(gp):
    """The first prediction of a plan, later ones and those of several plans in as many
    threads (more than streams are kept idle): the same bits, refused calls between them."""
    import threading

    import torch
    prob = inputs.random_small(2, 4000, seed=8, nu=1.5, lmin=0.1, lmax=0.25)
    rng = np.random.default_rng(9)
    al = cuda(rng.standard_normal(4000))
    i = rng.integers(0, 4000, 700)
    t = [cuda(v[i]) for v in (prob.x, prob.sigma, prob.l)]
    bad = [t[0] + 3.0, t[1], t[2]]
    torch.cuda.synchronize()

    def plan(stream):
        return gp.Plan(cuda(prob.x), cuda(prob.sigma), cuda(prob.l), prob.nu, prob.eta, 1e-6, M=60, stream=stream)

    want = host(plan(torch.cuda.Stream()).posterior_mean(al, *t))
    out, err = [[] for _ in range(6)], []

    def work(k):
        try:
            s = torch.cuda.Stream()
            with torch.cuda.stream(s):
                P = plan(s)
                for r in range(4):
                    out[k].append(host(P.posterior_mean(al, *t)))
                    if (k + r) % 3 == 0:
                        with pytest.raises(gp.GpError):
                            P.posterior_mean(al, *bad)
        except BaseException as e:  # noqa: BLE001
            err.append(e)

    ts = [threading.Thread(target=work, args=(k,)) for k in range(6)]
    for th in ts:
        th.start()
    for th in ts:
        th.join()
    assert not err, err
    for o in out:
        assert len(o) == 4 and all(np.array_equal(v, want) for v in o)
