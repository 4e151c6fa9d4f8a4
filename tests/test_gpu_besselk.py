"""GPU parity of standalone K_nu(x) and the window export against the CPU oracle.

The oracle computes the defining integral of Sec. IV-B by adaptive Gauss-Kronrod
in long double; the GPU computes the windowed trapezoid sum of Eq. "refined".
"""
import numpy as np
import pytest

from gpu_util import DBL_MIN, TOL_MIXED, TOL_PLAIN, re_metric, rel_err, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_00356_amd import api
    return api


def _gpu(api, nu, x, mode, result=0, **kw):
    import torch
    out = api.besselk(to_dev(nu), to_dev(x), mode=mode, result=result, **kw)
    torch.cuda.synchronize()
    return out.cpu().numpy()


def _check_form(api, orc, nu, x, mode, tol):
    k, lk, ks = orc.besselk(nu, x)
    got_k = _gpu(api, nu, x, mode, 0)
    got_s = _gpu(api, nu, x, mode, 1)
    got_l = _gpu(api, nu, x, mode, 2)
    normal = k >= DBL_MIN
    ek = rel_err(got_k[normal], k[normal])
    es = rel_err(got_s, ks)
    el = np.abs(got_l - lk)
    assert np.all(np.isfinite(got_s))
    assert ek.max() <= tol, ("K", ek.max(), nu[normal][ek.argmax()], x[normal][ek.argmax()])
    assert es.max() <= tol, ("scaled", es.max(), nu[es.argmax()], x[es.argmax()])
    # log K: absolute error tol (the relative error of K) plus the rounding of |log K|
    assert np.all(el <= tol + 4 * np.finfo(float).eps * np.abs(lk))
    # underflow zone: K below DBL_MIN is compared through e^x K above; here it must
    # at least be a non-negative number no larger than DBL_MIN * (1 + tol)
    assert np.all((got_k[~normal] >= 0) & (got_k[~normal] <= DBL_MIN * 2))
    return ek, es


def test_small_pairs_plain(api, orc):
    from paper_2502_00356_amd import workloads as w
    nu, x = w.small_pairs()
    ek, es = _check_form(api, orc, nu, x, "plain", TOL_PLAIN)
    # RE metric of Sec. IV-C on log K, reported for context
    _, lk, _ = orc.besselk(nu, x)
    re = re_metric(_gpu(api, nu, x, "plain", 2), lk)
    print("small pairs plain: max rel %.3g, max RE %.3f" % (max(ek.max(), es.max()), re.max()))


def test_small_pairs_mixed(api, orc):
    from paper_2502_00356_amd import workloads as w
    nu, x = w.small_pairs()
    ek, es = _check_form(api, orc, nu, x, "mixed", TOL_MIXED)
    print("small pairs mixed: max rel %.3g" % max(ek.max(), es.max()))


@pytest.mark.parametrize("mode,tol", [("plain", TOL_PLAIN), ("mixed", TOL_MIXED)])
def test_grid_law_sample(api, orc, mode, tol):
    """The standalone grid's law (nu in [0.01, 10], x in [1e-4, 1e3], 1% half-integer
    orders) on a 2^16 sample, with per-region maxima printed."""
    from paper_2502_00356_amd import workloads as w
    nu, x, hidx = w.grid_pairs(1 << 16, seed=2)
    ek, es = _check_form(api, orc, nu, x, mode, tol)
    lx = np.log10(x)
    regions = []
    for lo in range(-4, 3):
        sel = (lx >= lo) & (lx < lo + 1)
        regions.append("x~1e%d: %.2g" % (lo, es[sel].max()))
    print(mode, " | ".join(regions), "| half-int: %.2g" % es[hidx].max())


@pytest.mark.parametrize("mode,tol", [("plain", TOL_PLAIN), ("mixed", TOL_MIXED)])
def test_half_integer_closed_forms(api, mode, tol):
    """e^x K_{n+1/2}(x) = sqrt(pi/2x) sum_k (n+k)! / (k! (n-k)! (2x)^k) (DLMF 10.49.12)."""
    import math
    xs = np.geomspace(1e-4, 1e3, 97)
    for n in range(10):
        ref = np.array([math.sqrt(math.pi / (2 * x)) * sum(
            math.factorial(n + k) / (math.factorial(k) * math.factorial(n - k)) / (2 * x) ** k
            for k in range(n + 1)) for x in xs])
        got = _gpu(api, np.full(xs.shape, n + 0.5), xs, mode, 1)
        assert rel_err(got, ref).max() <= tol, (n, rel_err(got, ref).max())


@pytest.mark.parametrize("n", [0, 1, 63, 255, 256, 257, 1000, 4099])
def test_ragged_sizes(api, orc, n):
    import torch
    rng = np.random.default_rng(100 + n)
    nu = rng.uniform(0.01, 10, n); x = 10 ** rng.uniform(-4, 3, n)
    if n == 0:
        out = api.besselk(to_dev(nu), to_dev(x))
        assert out.numel() == 0
        return
    got = _gpu(api, nu, x, "plain", 1)
    _, _, ks = orc.besselk(nu, x)
    assert rel_err(got, ks).max() <= TOL_PLAIN
    # the fixed-signature entry point is the plain form with defaults, bit for bit
    out = torch.empty(n, dtype=torch.float64, device="cuda")
    api.besselk_plain(to_dev(nu), to_dev(x), out)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(out.cpu().numpy(), _gpu(api, nu, x, "plain", 0))


@pytest.mark.parametrize("L,Lq", [(1e-3, 35.0), (0.01, 35.0), (0.05, 35.0), (0.08, 8.0), (0.3, 35.0), (0.999, 0.999),
                                  (36.0, 1e-3), (36.0, 0.3), (1.0, 1.0), (3.0, 30.0), (8.0, 1.0)])
def test_plain_small_thresholds(api, orc, L, Lq):
    """Thresholds below 1: the trapezoid sum over the solved window's own nodes (bk_window),
    formed here in long double (node positions rounded at 2^-52 t, up to 15, of a width down
    to 3e-3: 1e-12). From 1 on the window may be wider, so the sum lies between that window's
    integral and K, up to its own discretisation (Lq: half of K at most for Lq >= 1)."""
    import torch
    nu = np.array([0.0, 0.3, 0.9, 2.0, 9.0, 9.9, 100.0, 300.0, 300.0, 9900.0, 9900.0])
    x = np.array([1.0, 0.2, 0.95, 5.0, 90.0, 100.0, 40.0, 60.0, 9.1e4, 9e4, 6e4])
    got = api.besselk(to_dev(nu), to_dev(x), result=api.RESULT_LOG, L_window=L, L_quad=Lq)
    t0, t1, N = api.window(to_dev(nu), to_dev(x), L_window=L, L_quad=Lq)
    torch.cuda.synchronize()
    got, t0, t1, N = (a.cpu().numpy() for a in (got, t0, t1, N))

    def log_sum(v, z, a, b, n):
        a, h = np.longdouble(a), (np.longdouble(b) - np.longdouble(a)) / n
        t = a + np.arange(n + 1) * h
        e = v * t - np.log(np.longdouble(2)) - 2 * z * np.sinh(t / 2) ** 2 + np.log1p(np.exp(-2 * v * t))
        w = np.ones(n + 1, np.longdouble)
        w[0] = w[-1] = 0.5
        return float(e.max() + np.log((w * np.exp(e - e.max())).sum() * h) - z)

    solved = t1 > t0          # the solver itself loses windows that short at large orders
    assert solved.sum() >= 7
    _, lk, _ = orc.besselk(nu, x)
    for v, z, a, b, n, g, k in zip(*(q[solved] for q in (nu, x, t0, t1, N, got, lk))):
        if L >= 1 and Lq >= 1:
            assert log_sum(v, z, a, b, 4000) - np.log(2.0) <= g <= k + np.log(2.0), (v, z)
        else:
            s = log_sum(v, z, a, b, n)
            assert abs(s - g) <= 1e-11 + 4e-16 * abs(s), (v, z)


def test_plain_large_order_windows(api, orc):
    """Orders up to 10,000: the FP32 window has about the nodes of the solved one (within a
    tenth, and the two's own rounding up), and K is the oracle's (which converges up to
    nu = 1,000)."""
    import torch
    rng = np.random.default_rng(31)
    n = 3000
    nu = 10 ** rng.uniform(1.7, 4.0, n)
    x = nu * 10 ** rng.uniform(-0.3, 0.3, n)
    stats = torch.zeros(api.STATS_LEN, dtype=torch.int64, device="cuda")
    lk = api.besselk(to_dev(nu), to_dev(x), result=api.RESULT_LOG, stats=stats)
    _, _, N = api.window(to_dev(nu), to_dev(x), L_window=36.0, L_quad=35.0)
    torch.cuda.synchronize()
    assert int(stats[api.STAT_ENTRIES]) == n
    assert int(stats[api.STAT_NODES]) <= 1.1 * int(N.sum()) + 2 * n
    lo = nu < 1000
    _, ref, _ = orc.besselk(nu[lo], x[lo])
    # log K = Delta - x + ...: three roundings of terms up to nu asinh(nu / x) + x
    tol = TOL_PLAIN + 4 * 2.0 ** -53 * (nu * np.arcsinh(nu / x) + x)
    assert np.all(np.abs(lk.cpu().numpy()[lo] - ref) <= tol[lo])


@pytest.mark.parametrize("n", [131071, 131072, 131585, 799999, 800000])
@pytest.mark.parametrize("L", [0.0, 600.0])
def test_plain_shapes_agree(api, n, L):
    """The launch shapes (64-, 256-, 512- and 1,024-entry workgroups) at their edges: the bits of
    calls of 4,000 with the same pairs."""
    import torch
    rng = np.random.default_rng(n)
    nu, x = rng.uniform(0.0, 20.0, n), 10 ** rng.uniform(-4, 3, n)
    odd = np.arange(0, n, 37)
    nu[odd] = np.resize([0.5, 2e4, 0.0, 3.0, np.nan, 1e-9, 3e5, 1.0, 2e6, 700.0], odd.size)
    x[odd] = np.resize([5e-13, 3e4, 1e-13, np.inf, 1.0, 2e5, 4e5, 9e7, 3e6, 650.0], odd.size)
    dn, dx = to_dev(nu), to_dev(x)
    full = api.besselk(dn, dx, result=api.RESULT_SCALED, L_window=L)
    for a in (0, n // 2 - 1000, n - 4000):
        part = api.besselk(dn[a:a + 4000], dx[a:a + 4000], result=api.RESULT_SCALED, L_window=L)
        torch.cuda.synchronize()
        assert np.array_equal(full[a:a + 4000].cpu().numpy(), part.cpu().numpy(), equal_nan=True), a


def test_plain_wide_window(api, orc):
    """x in 1e5 .. 1e8 and orders up to 1e6 by the FP32 window with both sides by products: the
    scaled result against the first terms of Hankel's series (x >= 1e5, nu <= 30: the fifth is
    below 1e-17), and log K against the uniform expansion's leading term (1 / nu) at large
    orders."""
    import torch
    rng = np.random.default_rng(33)
    nu, x = rng.uniform(0.0, 30.0, 4000), 10 ** rng.uniform(5.0, 8.0, 4000)
    got = api.besselk(to_dev(nu), to_dev(x), result=api.RESULT_SCALED).cpu().numpy()
    mu, s, t = 4 * nu.astype(np.longdouble) ** 2, np.ones(4000, np.longdouble), np.ones(4000, np.longdouble)
    for k in range(1, 7):
        t = t * (mu - (2 * k - 1) ** 2) / (8 * k * x.astype(np.longdouble))
        s = s + t
    ref = np.sqrt(np.longdouble(np.pi) / 2 / x.astype(np.longdouble)) * s
    assert rel_err(got, ref.astype(np.float64)).max() <= TOL_PLAIN
    nu = 10 ** rng.uniform(4.0, 6.0, 4000)
    x = nu * 10 ** rng.uniform(-1.0, 1.0, 4000)
    lk = api.besselk(to_dev(nu), to_dev(x), result=api.RESULT_LOG).cpu().numpy()
    z = x / nu
    eta = np.sqrt(1 + z * z) + np.log(z / (1 + np.sqrt(1 + z * z)))
    lead = 0.5 * np.log(np.pi / (2 * nu)) - nu * eta - 0.25 * np.log1p(z * z)
    assert np.all(np.abs(lk - lead) <= 1.0 / nu + 1e-12 * nu * (1 + np.abs(eta)))


def test_plain_ends_of_the_double_range(api):
    """K = 0 for the largest x (past 1e306 the window's step squared is below the double
    range), with log K at most -x: no NaN."""
    import torch
    x = np.concatenate([np.linspace(2.0, 17.0, 40) * 1e306, 10.0 ** np.arange(290, 307)])
    for nu in (0.0, 1e-9, 0.5, 40.0, 6.3e6, 1.5e14):
        v = np.full(x.shape, nu)
        k = api.besselk(to_dev(v), to_dev(x))
        lk = api.besselk(to_dev(v), to_dev(x), result=api.RESULT_LOG)
        d = api.besselk_deriv(to_dev(v), to_dev(x))
        torch.cuda.synchronize()
        assert np.all(k.cpu().numpy() == 0) and np.all(lk.cpu().numpy() <= -x), nu
        assert all(np.all(d[key].cpu().numpy() == 0) for key in ("k", "dx")), nu
    r = np.concatenate([[0.0], x[:8] * 1e-153])         # Matern distances at beta = 1e-153
    g = api.matern_grad_tiles(to_dev(r), to_dev(0 * r), 2.0, 1e-153, 0.8, r.size, 0)
    torch.cuda.synchronize()
    for key, v in g.items():
        v = v.cpu().numpy().reshape(r.size, r.size)
        assert np.all(v[~np.eye(r.size, dtype=bool)] == 0) and np.all(np.diag(v) == (2.0 if key == "c" else 0.0)), key


def test_special_values(api):
    nu = np.array([1.0, 1.0, 1.0, np.nan, 2.0, -2.5, np.inf, 3.0])
    x = np.array([0.0, -1.0, np.nan, 1.0, np.inf, 2.0, 1.0, 1e-4])
    for mode in ("plain", "mixed"):
        k = _gpu(api, nu, x, mode, 0)
        assert k[0] == np.inf and np.isnan(k[1]) and np.isnan(k[2]) and np.isnan(k[3])
        assert k[4] == 0.0 and k[6] == np.inf
        assert k[5] == _gpu(api, np.array([2.5]), np.array([2.0]), mode, 0)[0]   # K_{-nu} = K_nu
        lg = _gpu(api, nu, x, mode, 2)
        assert lg[4] == -np.inf


def test_degenerate_peak(api, orc):
    """nu^2 = x and nu^2 slightly above x: the interior peak degenerates to t = 0."""
    nu = np.array([1.0, 2.0, 3.0, 0.1, 1.0, 2.0, 3.0, 9.99])
    x = np.array([1.0, 4.0, 9.0, 0.01, 1.0 - 1e-12, 4.0 * (1 - 1e-9), 9.0 * (1 - 1e-6), 99.8])
    _, _, ks = orc.besselk(nu, x)
    assert rel_err(_gpu(api, nu, x, "plain", 1), ks).max() <= TOL_PLAIN
    assert rel_err(_gpu(api, nu, x, "mixed", 1), ks).max() <= TOL_MIXED


def test_stats_counters(api):
    import torch
    from paper_2502_00356_amd import workloads as w
    nu, x = w.small_pairs(1000, seed=3)
    stats = torch.zeros(api.STATS_LEN, dtype=torch.int64, device="cuda")
    api.besselk(to_dev(nu), to_dev(x), mode="plain", stats=stats)
    api.besselk(to_dev(nu), to_dev(x), mode="plain", stats=stats)
    torch.cuda.synchronize()
    s = stats.cpu().numpy()
    # x < 0.1 takes Temme's series (not counted as quadrature); these orders and
    # arguments are all far inside its range
    quad = 2 * int((x >= 0.1).sum())
    assert s[api.STAT_ENTRIES] == quad
    assert quad * 5 <= s[api.STAT_NODES] <= quad * 200


def test_small_x_temme_branch(api, orc):
    """Plain FP64 at x < 0.1, where it takes Temme's series with the forward
    recurrence (Sec. IV-A) unless K_nu(x) could leave the double range: K, e^x K and
    log K against the oracle's integral, including integer and half-integer orders,
    the x = 0.1 boundary, arguments down to 1e-8, and orders past the series' range
    (nu = 40..60 at x = 1e-6, where the quadrature runs instead and K overflows)."""
    rng = np.random.default_rng(21)
    nu = np.concatenate([rng.uniform(0.0, 12.0, 3000), np.arange(0, 13) * 0.5, [0.3, 2.7, 7.5, 9.99]])
    x = np.concatenate([10.0 ** rng.uniform(-8, -1, 3000), np.full(13, 0.05), [0.1, 0.0999999, 1e-8, 0.1]])
    k, lk, ks = orc.besselk(nu, x)
    got_k, got_s, got_l = (_gpu(api, nu, x, "plain", r) for r in (0, 1, 2))
    fin = np.isfinite(k) & (k >= DBL_MIN)
    assert rel_err(got_k[fin], k[fin]).max() <= TOL_PLAIN
    assert rel_err(got_s, ks).max() <= TOL_PLAIN
    assert np.all(np.abs(got_l - lk) <= TOL_PLAIN + 4 * np.finfo(float).eps * np.abs(lk))
    big_nu = np.array([40.0, 50.0, 60.0])
    big_x = np.full(3, 1e-6)
    _, lk2, _ = orc.besselk(big_nu, big_x)
    got_l2 = _gpu(api, big_nu, big_x, "plain", 2)
    assert np.all(np.isfinite(got_l2))
    assert np.all(np.abs(got_l2 - lk2) <= TOL_PLAIN + 4 * np.finfo(float).eps * np.abs(lk2))


def test_invalid_arguments(api):
    import torch
    a = torch.ones(4, dtype=torch.float64, device="cuda")
    with pytest.raises(api.BkError):
        api.besselk(a, a, mode=7)
    with pytest.raises(api.BkError):
        api.besselk(a, a, L_window=-1.0)
    with pytest.raises(api.BkError):
        api.besselk(a, a, mode="learned")          # no model


# ----------------------------------------------------------------- window export
def test_window_matches_oracle(api, orc):
    """bk_window against the oracle's bisection window at the mixed thresholds
    (L = 16, node target 15.4): t_lo and t_hi within 1e-10 (relative to max(1, t)),
    node counts equal except where (t1 - t0)/h sits within 1e-9 of an integer."""
    import torch
    from paper_2502_00356_amd import workloads as w
    nu, x = w.training_pairs(1 << 14, seed=4)
    for L, Lq in ((16.0, 15.4), (38.0, 36.5)):
        tlo, thi, N = api.window(to_dev(nu), to_dev(x), L, Lq)
        torch.cuda.synchronize()
        tlo, thi, N = tlo.cpu().numpy(), thi.cpu().numpy(), N.cpu().numpy()
        tm, gm, t0, t1 = orc.window(nu, x, L)
        assert np.all(np.abs(tlo - t0) <= 1e-10 * np.maximum(1, t0))
        assert np.all(np.abs(thi - t1) <= 1e-10 * np.maximum(1, t1))
        Nref = orc.node_count(nu, x, t0, t1, Lq)
        ratio = orc.node_count_ratio(nu, x, t0, t1, Lq)
        tie = np.abs(ratio - np.round(ratio)) < 1e-9
        mism = N != Nref
        assert np.all(~mism | (tie & (np.abs(N - Nref) <= 1))), (nu[mism][:5], x[mism][:5], N[mism][:5], Nref[mism][:5])
        print("L=%g: mean N %.2f max N %d" % (L, N.mean(), N.max()))


@pytest.mark.parametrize("mode", ["plain", "mixed", "paper"])
def test_kernel_events_bracket_the_kernel(api, mode):
    """The optional event pair is recorded around the form's main kernel: results are
    unchanged, and the pair's time is positive and within the whole call's."""
    import torch
    from paper_2502_00356_amd import workloads as w
    nu, x = w.small_pairs(4096, seed=5)
    ref = _gpu(api, nu, x, mode, 1)
    dnu, dx = to_dev(nu), to_dev(x)
    ev = (torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
    outer = (torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
    for e in ev + outer:
        e.record()
    torch.cuda.synchronize()
    outer[0].record()
    got = api.besselk(dnu, dx, mode=mode, result=1, kernel_events=ev)
    outer[1].record()
    torch.cuda.synchronize()
    np.testing.assert_array_equal(got.cpu().numpy(), ref)
    t_k, t_all = ev[0].elapsed_time(ev[1]), outer[0].elapsed_time(outer[1])
    assert 0.0 < t_k <= t_all, (t_k, t_all)


@pytest.mark.parametrize("x", [1e-300, 1e-250, 1e-100, 1e-20, 9e-13])
def test_plain_tiny_arguments(api, x):
    """Orders just below 1 at arguments below the FP32 windows' range, where the walk left of
    the peak is hundreds of units of t long: log K against its leading terms
    log(Gamma(nu) / 2) + nu log(2 / x) + log(1 + Gamma(-nu) / Gamma(nu) (x / 2)^(2 nu)) (the
    next is x^2 / (4 (1 - nu))), to 1e-13 and four roundings of log K."""
    from math import gamma, lgamma, log, log1p
    nu = np.array([0.5, 0.86, 0.9, 0.95, 0.99, 0.999])
    got = _gpu(api, nu, np.full(nu.size, x), "plain", 2)
    ref = np.array([lgamma(v) - log(2.0) + v * (log(2.0) - log(x)) +
                    log1p(gamma(-v) / gamma(v) * (x / 2) ** (2 * v)) for v in nu])
    assert np.all(np.abs(got - ref) <= TOL_PLAIN + 4 * np.finfo(float).eps * np.abs(ref))


def test_plain_left_of_the_peak(api, orc):
    """The lower end of the windowed form (x just above 0.1), where small orders walk
    furthest to the left of the reference."""
    rng = np.random.default_rng(41)
    nu = np.concatenate([10 ** rng.uniform(-4, 0.3, 4000), rng.uniform(0.3, 1.1, 4000)])
    _check_form(api, orc, nu, rng.uniform(0.1, 0.2, nu.size), "plain", TOL_PLAIN)
