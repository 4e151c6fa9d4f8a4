"""GPU test of the blocked factorisation behind the likelihood, at the edges of its
128-blocks and of the four-block steps of its trailing update, against numpy's
Cholesky of the same covariance (built by the library's own Matern tiles).

Bars: the value within 1e-9 of |z^T Sigma^-1 z| + n and every gradient component
within 1e-9 of the sum of the magnitudes of its two terms, as in the likelihood's
tests (cond(Sigma) <= 1e4 here, so both factorisations are good to ~1e-12)."""
import math

import numpy as np
import pytest

from gpu_util import to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_00356_amd import api
    return api


@pytest.mark.parametrize("n", [1, 2, 15, 17, 127, 128, 129, 255, 257, 384, 511, 512, 513, 641, 1027])
def test_loglik_block_edges(api, n):
    from paper_2502_00356_amd import workloads as w
    s2, nu = 1.2, 0.8
    beta = 0.3 / math.sqrt(n)
    side = math.isqrt(n - 1) + 1
    xy = w.jittered_grid_locations(side, seed=n)[:n]
    z = np.random.default_rng(n).standard_normal(n)
    lx, ly = to_dev(xy[:, 0]), to_dev(xy[:, 1])
    ts = max(n, 2)
    g = {k: api.unpack_tiles(v, n, ts, 0).numpy() for k, v in
         api.matern_grad_tiles(lx, ly, s2, beta, nu, ts, 0).items()}
    assert np.linalg.cond(g["c"]) <= 1e4
    L = np.linalg.cholesky(g["c"])
    a = np.linalg.solve(L.T, np.linalg.solve(L, z))
    inv = np.linalg.inv(g["c"])
    quad = z @ a
    ll = -0.5 * quad - np.log(np.diag(L)).sum() - 0.5 * n * math.log(2 * math.pi)
    terms = [(0.5 * quad / s2, 0.5 * n / s2)] + [(0.5 * a @ g[k] @ a, 0.5 * (inv * g[k]).sum()) for k in ("dbeta", "dnu")]
    got = api.matern_loglik(lx, ly, to_dev(z), s2, beta, nu)
    got_g, grad = api.matern_loglik(lx, ly, to_dev(z), s2, beta, nu, grad=True)
    assert got_g == got
    assert abs(got - ll) <= 1e-9 * (abs(quad) + n)
    for (q, t), d in zip(terms, grad):
        assert abs((q - t) - d) <= 1e-9 * (abs(q) + abs(t)) + 1e-300


@pytest.mark.parametrize("n,k", [(5, 2), (200, 150), (700, 699)])
def test_loglik_singular(api, n, k):
    """A repeated point makes two equal rows: the pivot is zero up to rounding, and where
    it is not positive the call says so instead of returning a number."""
    from paper_2502_00356_amd import workloads as w
    xy = w.jittered_grid_locations(math.isqrt(n - 1) + 1, seed=n)[:n]
    xy[k] = xy[0]
    z = np.ones(n)
    try:
        l = api.matern_loglik(to_dev(xy[:, 0]), to_dev(xy[:, 1]), to_dev(z), 1.0, 0.01, 0.5)
    except api.BkError as e:
        assert e.status == 6        # BK_ENOTPD
    else:
        assert np.isfinite(l)


@pytest.mark.parametrize("n,i,k", [(2, 0, 1), (17, 3, 16), (129, 127, 128), (200, 150, 160), (200, 5, 160), (700, 0, 699)])
def test_loglik_zero_pivot(api, n, i, k):
    """Sites so far apart that Sigma is exactly the identity, and two of them the same: the
    pivot is 1 - 1 * 1 = 0, in the first diagonal block, in a later one and through panels."""
    x = np.arange(n, dtype=np.float64)
    z = np.ones(n)
    l = api.matern_loglik(to_dev(x), to_dev(0 * x), to_dev(z), 1.0, 1e-3, 0.5)
    assert abs(l + 0.5 * n * (1 + math.log(2 * math.pi))) <= 1e-12 * n
    x[k] = x[i]
    for grad in (False, True):
        with pytest.raises(api.BkError) as e:
            api.matern_loglik(to_dev(x), to_dev(0 * x), to_dev(z), 1.0, 1e-3, 0.5, grad=grad)
        assert e.value.status == 6        # BK_ENOTPD


@pytest.mark.parametrize("s2", [5e-310, 1e-290, 1e-170, 1e-160, 1e-156, 1e-62, 1e-60, 1e60, 1e62, 1e154, 1e160, 1e300, 1.5e308])
def test_loglik_scale(api, s2):
    """Any positive sigma2: with z = sqrt(sigma2) z1 the likelihood is that of sigma2 = 1 less
    n / 2 log sigma2, its beta and nu derivatives are the same, and that in sigma2 is divided
    by sigma2. Bars as above, and z's rounding."""
    from paper_2502_00356_amd import workloads as w
    n, beta, nu = 140, 0.03, 0.8
    xy = w.jittered_grid_locations(12, seed=3)[:n]
    z = np.random.default_rng(3).standard_normal(n)
    lx, ly = to_dev(xy[:, 0]), to_dev(xy[:, 1])
    l1, g1 = api.matern_loglik(lx, ly, to_dev(z), 1.0, beta, nu, grad=True)
    assert abs(l1) <= 1e3 and max(map(abs, g1)) <= 1e3
    got = api.matern_loglik(lx, ly, to_dev(z * math.sqrt(s2)), s2, beta, nu)
    got_g, grad = api.matern_loglik(lx, ly, to_dev(z * math.sqrt(s2)), s2, beta, nu, grad=True)
    assert got_g == got
    assert abs(got - (l1 - 0.5 * n * math.log(s2))) <= 1e-9 * (1e3 + n * abs(math.log(s2)))
    # s2 * inf where 1 / s2 is not a double
    assert abs(grad[0] * s2 - g1[0]) <= 1e-9 * 1e3 or (s2 < 1e-308 and math.isinf(grad[0]))
    assert abs(grad[1] - g1[1]) <= 1e-9 * 1e4 and abs(grad[2] - g1[2]) <= 1e-9 * 1e3


@pytest.mark.parametrize("n", [4747, 4993, 5377])
def test_loglik_tile_rules(api, n):
    """Sizes around which the launches change their tiles (38 block rows for the traces, 40
    blocks for panels and columns, 1,024 tiles for the update), against torch's own
    factorisation of the same matrix on the GPU; the bars as above."""
    import torch
    from paper_2502_00356_amd import workloads as w
    s2, nu = 1.2, 0.8
    beta = 0.3 / math.sqrt(n)
    side = math.isqrt(n - 1) + 1
    xy = w.jittered_grid_locations(side, seed=n)[:n]
    z = to_dev(np.random.default_rng(n).standard_normal(n))
    lx, ly = to_dev(xy[:, 0]), to_dev(xy[:, 1])
    got = api.matern_loglik(lx, ly, z, s2, beta, nu)
    got_g, grad = api.matern_loglik(lx, ly, z, s2, beta, nu, grad=True)
    g = {k: v.view(n, n) for k, v in api.matern_grad_tiles(lx, ly, s2, beta, nu, n, 0).items()}
    L = torch.linalg.cholesky(g["c"])
    a = torch.cholesky_solve(z[:, None], L)[:, 0]
    inv = torch.cholesky_inverse(L)
    quad = float(z @ a)
    ll = -0.5 * quad - float(torch.log(torch.diagonal(L)).sum()) - 0.5 * n * math.log(2 * math.pi)
    terms = [(0.5 * quad / s2, 0.5 * n / s2)]
    terms += [(0.5 * float(a @ (g[k] @ a)), 0.5 * float((inv * g[k]).sum())) for k in ("dbeta", "dnu")]
    assert got_g == got
    assert abs(got - ll) <= 1e-9 * (abs(quad) + n)
    for (q, t), d in zip(terms, grad):
        assert abs((q - t) - d) <= 1e-9 * (abs(q) + abs(t)) + 1e-300
