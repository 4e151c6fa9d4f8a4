"""GPU tests of the window-predicting MLP: training kernels against the numpy
float64 oracle, matrix-core inference, training, and the learned evaluation form
against the CPU K_nu oracle (including forced fallbacks)."""
import os
import time

import numpy as np
import pytest

from gpu_util import TOL_MIXED, rel_err, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2502_00356_amd import api
    return api


def _rand_params(seed, scale=0.4):
    from oracle import MLP_SHAPES
    rng = np.random.default_rng(seed)
    return {k: rng.normal(0, scale, s) for k, s in MLP_SHAPES}


def _flat(p):
    from oracle import MLP_SHAPES
    return np.concatenate([p[k].ravel() for k, _ in MLP_SHAPES])


def _unflat(v):
    from oracle import MLP_SHAPES
    out, o = {}, 0
    for k, s in MLP_SHAPES:
        n = int(np.prod(s))
        out[k] = v[o:o + n].reshape(s)
        o += n
    return out


def test_gradient_kernels_match_oracle(api, orc):
    """bk_mlp_grad (FP32) against the float64 oracle: loss and every gradient entry
    within 1e-5 relative (plus 1e-6 of the largest gradient for near-zero entries)."""
    import torch
    p = _rand_params(3)
    rng = np.random.default_rng(4)
    B = 2048
    u = rng.uniform(-1, 1, (B, 2))
    tgt = rng.normal(0.5, 0.5, (B, 3))
    tau = np.array([0.1, 0.9, 0.9])
    # the GPU sees FP32-rounded parameters and data; the oracle gets the same values
    pf = _flat(p).astype(np.float32)
    uf, tf, tauf = u.astype(np.float32), tgt.astype(np.float32), tau.astype(np.float32)
    loss, grad = api.mlp_grad(to_dev(pf), to_dev(uf), to_dev(tf), to_dev(tauf))
    torch.cuda.synchronize()
    p64 = _unflat(pf.astype(np.float64))
    y, cache = orc.mlp_forward(p64, uf.astype(np.float64))
    lref = orc.mlp_loss(y, tf.astype(np.float64), tauf.astype(np.float64))
    gref = _flat(orc.mlp_backward(p64, cache, y, tf.astype(np.float64), tauf.astype(np.float64)))
    g = grad.cpu().numpy().astype(np.float64)
    assert abs(float(loss.cpu()[0]) - lref) <= 1e-5 * abs(lref)
    assert np.all(np.abs(g - gref) <= 1e-5 * np.abs(gref) + 1e-6 * np.abs(gref).max())


@pytest.mark.parametrize("B", [1, 15, 16, 17, 63, 64, 65, 129, 2047, 8192 + 33])
def test_gradient_tile_edges(api, orc, B):
    """Batches at the edges of a wave's 16 and a workgroup's 64 samples, and of the row
    sum's groups of 32 tiles: every gradient entry and the loss within 64 FP32 roundings
    (2^-24 each) of the largest term's size, for which the largest gradient of its layer
    and the loss stand; and with scratch for the tiles' rows alone, where the loss is
    summed by atomics, the same gradient bits and that loss."""
    import torch
    p = _rand_params(8)
    rng = np.random.default_rng(B)
    u = rng.uniform(-1, 1, (B, 2)).astype(np.float32)
    tgt = rng.normal(0.5, 0.5, (B, 3)).astype(np.float32)
    tau = np.array([0.1, 0.9, 0.9], np.float32)
    pf = _flat(p).astype(np.float32)
    args = [to_dev(a) for a in (pf, u, tgt, tau)]
    loss, grad = api.mlp_grad(*args)
    tiles = (B + 63) // 64
    rows = torch.empty(4 * tiles * api.MLP_NPARAM, dtype=torch.uint8, device="cuda")
    loss2, grad2 = torch.full_like(loss, 7.0), torch.empty_like(grad)
    st = api._mlp_grad(*[a.data_ptr() for a in args], B, grad2.data_ptr(), loss2.data_ptr(), rows.data_ptr(),
                       rows.numel(), 0)
    short = api._mlp_grad(*[a.data_ptr() for a in args], B, grad2.data_ptr(), loss2.data_ptr(), rows.data_ptr(),
                          rows.numel() - 1, 0)
    torch.cuda.synchronize()
    assert st == 0 and short != 0
    p64 = _unflat(pf.astype(np.float64))
    y, cache = orc.mlp_forward(p64, u.astype(np.float64))
    lref = orc.mlp_loss(y, tgt.astype(np.float64), tau.astype(np.float64))
    gref = orc.mlp_backward(p64, cache, y, tgt.astype(np.float64), tau.astype(np.float64))
    tol = 64 * 2.0 ** -24
    g = _unflat(grad.cpu().numpy().astype(np.float64))
    for k in gref:
        assert np.abs(g[k] - gref[k]).max() <= tol * np.abs(gref[k]).max(), k
    assert torch.equal(grad, grad2)
    for l in (loss, loss2):
        assert abs(float(l.cpu()[0]) - lref) <= tol * lref


def test_adam_kernel_matches_oracle(api, orc):
    import torch
    rng = np.random.default_rng(5)
    n = 4547
    p = rng.normal(0, 1, n).astype(np.float32)
    g = rng.normal(0, 1e-2, n).astype(np.float32)
    m = rng.normal(0, 1e-3, n).astype(np.float32)
    v = rng.uniform(0, 1e-4, n).astype(np.float32)
    dp, dg, dm, dv = to_dev(p), to_dev(g), to_dev(m), to_dev(v)
    api.adam_step(dp, dg, dm, dv, 7, 1e-3)
    torch.cuda.synchronize()
    P = {"a": p.astype(np.float64)}; G = {"a": g.astype(np.float64)}
    M = {"a": m.astype(np.float64)}; V = {"a": v.astype(np.float64)}
    orc.adam_step(P, G, M, V, 7, 1e-3)
    # FP32 kernel vs float64 oracle: 1 - beta2 = 1e-3 carries a relative rounding
    # error of ~1e-5 in FP32, which the new-gradient part of v inherits
    assert np.allclose(dp.cpu().numpy(), P["a"], rtol=2e-6, atol=1e-7)
    assert np.allclose(dm.cpu().numpy(), M["a"], rtol=2e-6, atol=1e-9)
    assert np.allclose(dv.cpu().numpy(), V["a"], rtol=3e-5, atol=1e-12)


def test_matrix_core_inference(api, orc):
    """bk_mlp_infer (FP16 operands, FP32 accumulation) against the float64 forward of
    the same FP32 parameters; FP16 rounding of weights and activations bounds the
    difference (here 2e-2 absolute on outputs of size ~1)."""
    import torch
    p = _rand_params(6, scale=0.25)
    m = api.Model()
    m.set_params(torch.from_numpy(_flat(p).astype(np.float32)))
    rng = np.random.default_rng(7)
    for n in (1, 63, 64, 1000, 4096):
        u = rng.uniform(-1, 1, (n, 2)).astype(np.float32)
        y = m.infer(to_dev(u))
        torch.cuda.synchronize()
        yref, _ = orc.mlp_forward(_unflat(_flat(p).astype(np.float32).astype(np.float64)), u.astype(np.float64))
        assert np.abs(y.cpu().numpy() - yref).max() <= 2e-2 * (1 + np.abs(yref).max()), n


@pytest.fixture(scope="module")
def trained(api, tmp_path_factory):
    """A model trained on the GPU on 2^18 pairs of the standalone law (seed 4)."""
    import torch
    from paper_2502_00356_amd import workloads
    nu, x = workloads.training_pairs(1 << 18, seed=4)
    m = api.Model()
    loss = m.train(to_dev(nu), to_dev(x), epochs=30, batch=4096, lr=3e-3, seed=11)
    torch.cuda.synchronize()
    assert np.isfinite(loss)
    return m


def test_prediction_cells_hold_corner_predictions(api, trained):
    """The learned K_nu form reads its window from the model's cells: each cell must
    hold the smallest t_lo and the largest t_hi and N that the network (the same
    matrix-core forward as bk_mlp_infer) predicts at the cell's four corners; the
    cells follow a change of the box."""
    import torch
    f32 = np.float32

    def check(m, ncheck, seed):
        cells = m.get_cells().numpy()
        L, Nn, _ = cells.shape
        box = m.get_box().numpy()
        norm = m.get_norm().numpy()
        rng = np.random.default_rng(seed)
        i = rng.integers(0, L, ncheck)
        j = rng.integers(0, Nn, ncheck)
        i[:2] = (0, L - 1)
        j[:2] = (0, Nn - 1)
        b = box.astype(f32)
        dl = (b[1] - b[0]) / f32(L)
        dn = (b[3] - b[2]) / f32(Nn)
        ys = []
        for a, c in ((0, 0), (1, 0), (0, 1), (1, 1)):
            lx = b[0] + (i + a).astype(f32) * dl
            nu = b[2] + (j + c).astype(f32) * dn
            u = np.stack([(lx - f32(norm[0])) * f32(1.0 / norm[1]), (nu - f32(norm[2])) * f32(1.0 / norm[3])], 1)
            ys.append(m.infer(to_dev(u.astype(f32))).cpu().numpy())
        ys = np.stack(ys)
        want = np.stack([ys[:, :, 0].min(0), ys[:, :, 1].max(0), ys[:, :, 2].max(0)], 1)
        got = cells[i, j, :3]
        # both sides round the corner inputs the same way and run the same forward
        assert np.array_equal(got, want), np.abs(got - want).max()
        assert np.all(cells[:, :, 3] == 0.0)

    check(trained, 4096, 21)
    m = api.Model()
    m.set_params(trained.get_params())
    box = trained.get_box().numpy().copy()
    box[1] -= 1.0
    box[3] *= 0.5
    m.set_box(box)
    torch.cuda.synchronize()
    check(m, 1024, 22)


def test_training_reduces_loss(api):
    import torch
    from paper_2502_00356_amd import workloads
    nu, x = workloads.training_pairs(1 << 14, seed=8)
    m1 = api.Model(); m2 = api.Model()
    l1 = m1.train(to_dev(nu), to_dev(x), epochs=1, batch=1024, seed=1)
    l2 = m2.train(to_dev(nu), to_dev(x), epochs=20, batch=1024, seed=1)
    assert l2 < 0.5 * l1


def test_learned_parity(api, orc, trained):
    """Learned form against the oracle on the standalone law: every entry within
    2e-6 (accepted entries and fallbacks alike), fallback rate reported."""
    import torch
    from paper_2502_00356_amd import workloads
    nu, x, hidx = workloads.grid_pairs(1 << 16, seed=12)
    stats = torch.zeros(api.STATS_LEN, dtype=torch.int64, device="cuda")
    out = api.besselk(to_dev(nu), to_dev(x), mode="learned", model=trained, result=api.RESULT_SCALED, stats=stats)
    torch.cuda.synchronize()
    _, _, ks = orc.besselk(nu, x)
    e = rel_err(out.cpu().numpy(), ks)
    s = stats.cpu().numpy()
    fb = s[api.STAT_FB_RANGE] + s[api.STAT_FB_TAIL] + s[api.STAT_FB_NONFINITE]
    print("learned: max rel %.3g, fallbacks %d of %d (range %d tail %d nonfinite %d), N raised %d" % (
        e.max(), fb, nu.size, s[2], s[3], s[5], s[4]))
    assert e.max() <= TOL_MIXED
    assert fb < 0.02 * nu.size


def test_learned_plan_and_per_entry_paths_agree(api, orc, trained):
    """At the default node target the kernel takes each cell's precomputed plan
    (window, node count raised to the floor at the cell's largest-x, largest-nu
    corner, walk start in FP64); at any other target it decodes the window per
    entry. Both meet the bar; the plan path only adds nodes (up to the few entries
    whose fallbacks differ)."""
    import torch
    from paper_2502_00356_amd import workloads
    nu, x, _ = workloads.grid_pairs(1 << 15, seed=14)
    _, _, ks = orc.besselk(nu, x)
    res = {}
    for lq in (0.0, 14.5000001):              # 0 selects the default 14.5: the plan path
        stats = torch.zeros(api.STATS_LEN, dtype=torch.int64, device="cuda")
        out = api.besselk(to_dev(nu), to_dev(x), mode="learned", model=trained, result=api.RESULT_SCALED,
                          L_quad=lq, stats=stats)
        torch.cuda.synchronize()
        assert rel_err(out.cpu().numpy(), ks).max() <= TOL_MIXED, lq
        res[lq] = stats.cpu().numpy()
    plan, entry = res[0.0], res[14.5000001]
    ratio = plan[api.STAT_NODES] / entry[api.STAT_NODES]
    print("plan / per-entry nodes: %.4f" % ratio)
    assert 0.999 <= ratio <= 1.03


@pytest.mark.parametrize("n", [0, 1, 63, 255, 257, 1000, 4099])
def test_learned_ragged_sizes(api, orc, trained, n):
    """Partial last blocks and tiny inputs: dead lanes take part in the block sort
    without producing output; every live entry meets the bar, at both node targets
    (cell plans and per-entry decode)."""
    import torch
    rng = np.random.default_rng(300 + n)
    nu = rng.uniform(0.01, 10, n)
    x = 10 ** rng.uniform(-4, 3, n)
    if n == 0:
        out = api.besselk(to_dev(nu), to_dev(x), mode="learned", model=trained)
        assert out.numel() == 0
        return
    _, _, ks = orc.besselk(nu, x)
    for lq in (0.0, 14.5000001):
        out = api.besselk(to_dev(nu), to_dev(x), mode="learned", model=trained, result=api.RESULT_SCALED, L_quad=lq)
        torch.cuda.synchronize()
        assert rel_err(out.cpu().numpy(), ks).max() <= TOL_MIXED, (n, lq)


@pytest.mark.parametrize("lq", [0.0, 14.5000001])
def test_learned_launch_shapes(api, trained, lq):
    """Calls on both sides of 2,000,000 pairs (one launch with the fallback in place; sorted
    blocks and a fallback queue): the same values, up to FP64 roundings of the prefactor
    (|delta| below 1e3 here: 2^10 2^-52 and a few more), and the same statistics, with
    inputs outside the box, special values and ordinary ones mixed."""
    import torch
    from paper_2502_00356_amd import workloads
    n = 2000077
    nu, x, _ = workloads.grid_pairs(1 << 21, seed=15)
    nu, x = nu[:n].copy(), x[:n].copy()
    nu[::1009] = np.resize([25.0, np.nan, 0.0, -3.0, np.inf], nu[::1009].size)
    x[::1511] = np.resize([0.0, 2e3, 1e-7, np.inf, -1.0], x[::1511].size)
    dn, dx = to_dev(nu), to_dev(x)

    def run(a, b):
        st = torch.zeros(api.STATS_LEN, dtype=torch.int64, device="cuda")
        o = api.besselk(dn[a:b], dx[a:b], mode="learned", model=trained, result=api.RESULT_SCALED, L_quad=lq, stats=st)
        torch.cuda.synchronize()
        return o, st

    full, st = run(0, n)
    parts = [run(a, min(n, a + 400000)) for a in range(0, n, 400000)]
    small = torch.cat([p[0] for p in parts])
    assert bool((torch.isnan(full) == torch.isnan(small)).all())
    assert bool((torch.isinf(full) == torch.isinf(small)).all())
    ok = torch.isfinite(full)
    assert bool(((full - small).abs()[ok] <= 4e-13 * small.abs()[ok]).all())
    tot = sum(p[1] for p in parts)
    for k in (api.STAT_ENTRIES, api.STAT_NODES, api.STAT_FB_RANGE, api.STAT_FB_TAIL, api.STAT_FB_NONFINITE,
              api.STAT_NODE_RAISED):
        assert int(st[k]) == int(tot[k]), k


@pytest.mark.parametrize("n", [4097, 2000077])
@pytest.mark.parametrize("lq", [0.0, 14.5000001])
def test_learned_in_place(api, trained, n, lq):
    """out may be x or nu, in both launch shapes: entries whose window fails the tail test
    (here by a network whose t_hi is cut short) are recomputed from their own inputs."""
    import torch
    from paper_2502_00356_amd import workloads
    m = api.Model()
    p = trained.get_params()
    p[4352 + 64:4352 + 128] *= 0.95        # W3 and b3 of t_hi
    p[4545] *= 0.95
    m.set_params(p)
    m.set_norm(trained.get_norm())
    m.set_box(trained.get_box())
    m.set_margins(0.0, 0.0, 0.1, 1.0)
    nu, x, _ = workloads.grid_pairs(1 << 21, seed=16)
    nu, x = to_dev(nu[:n]), to_dev(x[:n])
    stats = torch.zeros(api.STATS_LEN, dtype=torch.int64, device="cuda")
    ref = api.besselk(nu, x, mode="learned", model=m, L_quad=lq, stats=stats)
    assert 0.01 * n < int(stats[api.STAT_FB_TAIL]) < 0.99 * n
    for st in (None, stats):
        a, b = nu.clone(), x.clone()
        assert torch.equal(api.besselk(a, b, out=b, mode="learned", model=m, L_quad=lq, stats=st), ref)
        a, b = nu.clone(), x.clone()
        assert torch.equal(api.besselk(a, b, out=a, mode="learned", model=m, L_quad=lq, stats=st), ref)


def test_learned_out_of_range_falls_back(api, orc, trained):
    """Pairs outside the training box all take the plain-solver path and stay exact."""
    import torch
    from paper_2502_00356_amd import workloads
    nu, x = workloads.out_of_range_pairs(1 << 12, seed=6)
    stats = torch.zeros(api.STATS_LEN, dtype=torch.int64, device="cuda")
    out = api.besselk(to_dev(nu), to_dev(x), mode="learned", model=trained, result=api.RESULT_SCALED, stats=stats)
    torch.cuda.synchronize()
    _, _, ks = orc.besselk(nu, x)
    assert rel_err(out.cpu().numpy(), ks).max() <= TOL_MIXED
    assert stats.cpu().numpy()[api.STAT_FB_RANGE] == nu.size


def test_zero_weights_force_fallback(api, orc):
    """A model whose weights are all zero predicts an empty window: every entry fails
    the tail check, takes the fallback, and the result still meets the bar."""
    import torch
    from paper_2502_00356_amd import workloads
    m = api.Model()
    m.set_params(torch.zeros(api.MLP_NPARAM))
    nu, x = workloads.small_pairs(3000, seed=9)
    stats = torch.zeros(api.STATS_LEN, dtype=torch.int64, device="cuda")
    out = api.besselk(to_dev(nu), to_dev(x), mode="learned", model=m, result=api.RESULT_SCALED, stats=stats)
    torch.cuda.synchronize()
    _, _, ks = orc.besselk(nu, x)
    assert rel_err(out.cpu().numpy(), ks).max() <= TOL_MIXED
    s = stats.cpu().numpy()
    assert s[api.STAT_FB_TAIL] + s[api.STAT_FB_NONFINITE] == nu.size


def test_zero_weights_force_matern_fallback(api, orc):
    """Learned Matern tiles with an all-zero model: every off-diagonal entry is
    rejected, marked and recomputed by the fallback kernel from the model's list of
    waves (three tile rows with a ragged last one, FP64 and FP32 output)."""
    import torch
    from paper_2502_00356_amd import workloads as w
    m = api.Model()
    m.set_params(torch.zeros(api.MLP_NPARAM))
    xy = w.uniform_locations(170, seed=53)
    lx, ly = to_dev(xy[:, 0]), to_dev(xy[:, 1])
    R = orc.matern_full(xy, 1.3, 0.05, 1.7)
    for dt in (api.OUT_F64, api.OUT_F32):
        out = api.matern_tiles(lx, ly, 1.3, 0.05, 1.7, 64, 1, mode="learned", model=m, out_dtype=dt)
        torch.cuda.synchronize()
        A = api.unpack_tiles(out, 170, 64, 1).double().numpy()
        assert np.all(np.isfinite(A))
        mm = R > 1e-300
        assert rel_err(A[mm], R[mm]).max() <= TOL_MIXED + (2 ** -24 if dt == api.OUT_F32 else 0.0)


def test_halved_node_prediction_is_raised(api, orc, trained, tmp_path):
    """Halving the predicted node count (through the output scale) leaves the step
    too coarse; the strip-bound rule raises N for those entries and the bar holds."""
    import torch
    from paper_2502_00356_amd import workloads
    path = str(tmp_path / "m.bin")
    trained.save(path)
    m = api.Model(path)
    m.set_margins(0.05, 0.05, 0.0, 0.0)
    params = m.get_params()
    norm = m.get_norm().numpy().copy()
    norm[5] *= 0.5                       # halve the node-count scale: predicted N is halved
    m.set_norm(norm)
    nu, x, _ = workloads.grid_pairs(1 << 14, seed=13)
    stats = torch.zeros(api.STATS_LEN, dtype=torch.int64, device="cuda")
    out = api.besselk(to_dev(nu), to_dev(x), mode="learned", model=m, result=api.RESULT_SCALED, stats=stats)
    torch.cuda.synchronize()
    _, _, ks = orc.besselk(nu, x)
    assert rel_err(out.cpu().numpy(), ks).max() <= TOL_MIXED
    assert stats.cpu().numpy()[api.STAT_NODE_RAISED] > nu.size // 2
    assert params.shape[0] == api.MLP_NPARAM


def test_save_load_roundtrip(api, trained, tmp_path):
    import torch
    path = str(tmp_path / "w.bin")
    trained.save(path)
    m = api.Model(path)
    assert torch.equal(m.get_params(), trained.get_params())
    assert torch.equal(m.get_box(), trained.get_box())
    bad = tmp_path / "bad.bin"
    bad.write_bytes(b"not a model")
    with pytest.raises(api.BkError):
        api.Model(str(bad))


def test_learned_matern(api, orc, trained):
    """Learned Matern tiles (MLP tabulated over log10 x at the launch's nu) against
    the oracle, FP64 and FP32 output."""
    from paper_2502_00356_amd import workloads as w
    import torch
    xy = w.uniform_locations(300, seed=51)
    for nu, beta in ((0.8, 0.05), (2.3, 0.05), (3.7, 0.02)):
        lx, ly = to_dev(xy[:, 0]), to_dev(xy[:, 1])
        out = api.matern_tiles(lx, ly, 1.0, beta, nu, 128, 1, mode="learned", model=trained)
        torch.cuda.synchronize()
        A = api.unpack_tiles(out, 300, 128, 1).numpy()
        R = orc.matern_full(xy, 1.0, beta, nu)
        m = R > 1e-300
        assert rel_err(A[m], R[m]).max() <= TOL_MIXED, nu


@pytest.mark.parametrize("nu,beta", [(0.05, 0.3), (0.3, 0.002), (0.6, 1.5), (6.0, 0.01), (9.5, 0.05)])
def test_learned_matern_order_and_range_extremes(api, orc, trained, nu, beta):
    """Orders near the training box's ends and ranges that put z near both ends of
    its x span (small z: windows that start right of 0 and take the left-tail
    bound; small 2 nu h: the FP64 node factor): learned tiles against the oracle,
    FP32 and FP64 output, and the counting variant bit for bit."""
    import torch
    from paper_2502_00356_amd import workloads as w
    n, ts = 200, 128
    xy = w.uniform_locations(n, seed=54)
    lx, ly = to_dev(xy[:, 0]), to_dev(xy[:, 1])
    R = orc.matern_full(xy, 1.0, beta, nu)
    for odt, floor in ((api.OUT_F32, 1e-36), (api.OUT_F64, 1e-300)):
        out = api.matern_tiles(lx, ly, 1.0, beta, nu, ts, 1, mode="learned", model=trained, out_dtype=odt)
        st = torch.zeros(api.STATS_LEN, dtype=torch.int64, device="cuda")
        out2 = api.matern_tiles(lx, ly, 1.0, beta, nu, ts, 1, mode="learned", model=trained, out_dtype=odt,
                                stats=st)
        torch.cuda.synchronize()
        assert torch.equal(out, out2)
        A = api.unpack_tiles(out, n, ts, 1).numpy().astype(np.float64)
        m = R > floor
        assert rel_err(A[m], R[m]).max() <= TOL_MIXED, (nu, beta, odt)
        assert int(st[api.STAT_ENTRIES]) > 0


@pytest.mark.parametrize("ts,lower", [(24, 1), (64, 0), (100, 1), (129, 0), (257, 1)])
def test_learned_matern_tile_shapes(api, orc, trained, ts, lower):
    """Tile sizes that leave a workgroup's last waves idle (below 128 columns), split a
    column group or a row block, or hold the whole matrix in one tile; full and
    lower layouts. Learned tiles against the oracle (FP32 output) and bit for bit
    against the statistics variant."""
    import torch
    from paper_2502_00356_amd import workloads as w
    n, beta, nu = 257, 0.04, 1.7
    xy = w.uniform_locations(n, seed=53)
    lx, ly = to_dev(xy[:, 0]), to_dev(xy[:, 1])
    out = api.matern_tiles(lx, ly, 1.0, beta, nu, ts, lower, mode="learned", model=trained, out_dtype=api.OUT_F32)
    st = torch.zeros(api.STATS_LEN, dtype=torch.int64, device="cuda")
    out2 = api.matern_tiles(lx, ly, 1.0, beta, nu, ts, lower, mode="learned", model=trained, out_dtype=api.OUT_F32,
                            stats=st)
    torch.cuda.synchronize()
    assert torch.equal(out, out2)
    A = api.unpack_tiles(out, n, ts, lower).numpy().astype(np.float64)
    R = orc.matern_full(xy, 1.0, beta, nu)
    m = R > 1e-36
    assert rel_err(A[m], R[m]).max() <= TOL_MIXED
    assert np.all(np.diag(A) == 1.0)


def test_learned_matern_sigma2(api, orc, trained):
    """sigma^2 enters the learned Matern plans as ln sigma^2 in the exponent: the
    output matches the oracle at extreme positive sigma^2 in both output types, and
    sigma^2 = 0 or +inf (no finite logarithm) gives the constant it must."""
    import torch
    from paper_2502_00356_amd import workloads as w
    n, ts, beta, nu = 300, 128, 0.05, 2.3
    xy = w.uniform_locations(n, seed=52)
    lx, ly = to_dev(xy[:, 0]), to_dev(xy[:, 1])
    R1 = orc.matern_full(xy, 1.0, beta, nu)
    for s2, odt in ((1e-30, api.OUT_F32), (3.5, api.OUT_F32), (1e30, api.OUT_F32), (1e-200, api.OUT_F64),
                    (1e200, api.OUT_F64)):
        out = api.matern_tiles(lx, ly, s2, beta, nu, ts, 1, mode="learned", model=trained, out_dtype=odt)
        torch.cuda.synchronize()
        A = api.unpack_tiles(out, n, ts, 1).numpy().astype(np.float64)
        R = s2 * R1
        m = np.abs(R) > 1e-36 if odt == api.OUT_F32 else np.abs(R) > 1e-300
        assert m.sum() > n * n // 2, s2
        assert rel_err(A[m], R[m]).max() <= TOL_MIXED, s2
    for s2 in (0.0, float("inf")):
        for odt in (api.OUT_F32, api.OUT_F64):
            out = api.matern_tiles(lx, ly, s2, beta, nu, ts, 1, mode="learned", model=trained, out_dtype=odt)
            torch.cuda.synchronize()
            A = api.unpack_tiles(out, n, ts, 1).numpy()
            assert np.all(A == s2), (s2, odt)


def test_learned_gain_over_mixed(api, trained):
    """What the trained network buys: on 2^22 pairs of the standalone law the learned
    form is faster than the same FP32-compensated node sums behind the FP64 solve."""
    import torch
    from paper_2502_00356_amd import workloads
    nu, x, _ = workloads.grid_pairs(1 << 22, seed=2)
    dnu, dx = to_dev(nu), to_dev(x)
    out = torch.empty_like(dx)
    ws = torch.empty(api.workspace_bytes(dx.numel()), dtype=torch.uint8, device="cuda")
    times = {}
    for mode in ("mixed", "learned", "mixed", "learned"):
        api.besselk(dnu, dx, out=out, mode=mode, model=trained, workspace=ws)
        torch.cuda.synchronize()
        t0 = time.perf_counter()
        for _ in range(3):
            api.besselk(dnu, dx, out=out, mode=mode, model=trained, workspace=ws)
        torch.cuda.synchronize()
        times[mode] = (time.perf_counter() - t0) / 3
    print("2^22 pairs: mixed %.3f ms, learned %.3f ms, gain %.2fx" % (
        times["mixed"] * 1e3, times["learned"] * 1e3, times["mixed"] / times["learned"]))
    assert times["learned"] < times["mixed"]


def test_learned_kernel_events(api, trained):
    """The optional event pair brackets the learned kernel alone (the queue reset and
    the fallback launch fall outside): results unchanged, pair time within the call's."""
    import torch
    from paper_2502_00356_amd import workloads
    nu, x, _ = workloads.grid_pairs(1 << 16, seed=4)
    dnu, dx = to_dev(nu), to_dev(x)
    ref = api.besselk(dnu, dx, mode="learned", model=trained)
    ev = (torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
    outer = (torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
    for e in ev + outer:
        e.record()
    torch.cuda.synchronize()
    outer[0].record()
    got = api.besselk(dnu, dx, mode="learned", model=trained, kernel_events=ev)
    outer[1].record()
    torch.cuda.synchronize()
    np.testing.assert_array_equal(got.cpu().numpy(), ref.cpu().numpy())
    t_k, t_all = ev[0].elapsed_time(ev[1]), outer[0].elapsed_time(outer[1])
    assert 0.0 < t_k <= t_all, (t_k, t_all)


def test_two_streams_share_one_model(api, orc, trained):
    """The learned forms only read the model: Matern tiles at two orders and K_nu on
    two streams at once, each with its own workspace, give the oracle's values and
    the same bits as one call at a time."""
    import torch
    from paper_2502_00356_amd import workloads as w
    xy = w.uniform_locations(700, seed=61)
    lx, ly = to_dev(xy[:, 0]), to_dev(xy[:, 1])
    nu_s, x_s, _ = w.grid_pairs(1 << 16, seed=62)
    dnu, dx = to_dev(nu_s), to_dev(x_s)
    cases = ((0.8, 0.05), (3.7, 0.02))
    seq = [api.matern_tiles(lx, ly, 1.0, b, v, 256, 1, mode="learned", model=trained) for v, b in cases]
    kseq = api.besselk(dnu, dx, mode="learned", model=trained)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    outs = [torch.full_like(s, -1.0) for s in seq]
    kout = torch.empty_like(kseq)
    for rep in range(3):
        for o in outs:
            o.fill_(-1.0)
        kout.fill_(-1.0)
        torch.cuda.synchronize()
        for k, ((v, b), st) in enumerate(zip(cases, streams)):
            with torch.cuda.stream(st):
                api.matern_tiles(lx, ly, 1.0, b, v, 256, 1, mode="learned", model=trained, out=outs[k])
                if k == 1:
                    api.besselk(dnu, dx, mode="learned", model=trained, out=kout)
        torch.cuda.synchronize()
        for k in range(2):
            assert torch.equal(outs[k], seq[k]), (rep, k)
        assert torch.equal(kout, kseq), rep
    for (v, b), o in zip(cases, outs):
        A = api.unpack_tiles(o, 700, 256, 1).numpy()
        R = orc.matern_full(xy, 1.0, b, v)
        m = R > 1e-300
        assert rel_err(A[m], R[m]).max() <= TOL_MIXED, v


def test_learned_matern_counting_variant(api, orc, trained):
    """A call with statistics runs the counting variant of the learned Matern
    kernels: the same bits as without, and counts that add up (one quadrature per
    stored entry at nonzero distance, in range of the model)."""
    import torch
    from paper_2502_00356_amd import workloads as w
    n, ts = 333, 128                       # ragged last tile row
    xy = w.uniform_locations(n, seed=63)
    lx, ly = to_dev(xy[:, 0]), to_dev(xy[:, 1])
    ref = api.matern_tiles(lx, ly, 1.0, 0.03, 2.3, ts, 1, mode="learned", model=trained)
    stats = torch.zeros(api.STATS_LEN, dtype=torch.int64, device="cuda")
    got = api.matern_tiles(lx, ly, 1.0, 0.03, 2.3, ts, 1, mode="learned", model=trained, stats=stats)
    torch.cuda.synchronize()
    assert torch.equal(got, ref)
    st = stats.cpu().numpy()
    stored = api.matern_out_elems(n, ts, 1)
    zero_dist = n                          # the diagonal (the points are distinct)
    fb = int(st[api.STAT_FB_RANGE] + st[api.STAT_FB_TAIL] + st[api.STAT_FB_NONFINITE])
    # every nonzero-distance entry is either out of the box or walked (and some walks
    # are rejected); rejected entries are walked again by the fallback
    assert int(st[api.STAT_ENTRIES]) - fb + int(st[api.STAT_FB_RANGE]) == stored - zero_dist
    assert int(st[api.STAT_NODES]) >= 5 * int(st[api.STAT_ENTRIES])
    assert 0 <= int(st[api.STAT_FB_NODES]) <= int(st[api.STAT_NODES])
    A = api.unpack_tiles(got, n, ts, 1).numpy()
    R = orc.matern_full(xy, 1.0, 0.03, 2.3)
    m = R > 1e-300
    assert rel_err(A[m], R[m]).max() <= TOL_MIXED


def test_learned_matern_kernel_events(api, trained):
    """The optional event pair brackets the learned Matern main launches (table,
    plans, bitmap reset and fallback fall outside)."""
    import torch
    from paper_2502_00356_amd import workloads as w
    xy = w.uniform_locations(2000, seed=64)
    lx, ly = to_dev(xy[:, 0]), to_dev(xy[:, 1])
    ref = api.matern_tiles(lx, ly, 1.0, 0.05, 1.5, 512, 1, mode="learned", model=trained)
    ev = (torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
    outer = (torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True))
    for e in ev + outer:
        e.record()
    torch.cuda.synchronize()
    outer[0].record()
    got = api.matern_tiles(lx, ly, 1.0, 0.05, 1.5, 512, 1, mode="learned", model=trained, kernel_events=ev)
    outer[1].record()
    torch.cuda.synchronize()
    assert torch.equal(got, ref)
    t_k, t_all = ev[0].elapsed_time(ev[1]), outer[0].elapsed_time(outer[1])
    assert 0.0 < t_k <= t_all, (t_k, t_all)
