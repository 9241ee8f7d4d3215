"""GPU kernels at the edges of their tiles and ranges, against the oracle."""
import numpy as np
import pytest

import oracle
import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2302_05730_amd as m
    m.lib()
    return m


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float64)).cuda()


def _f32(a):
    return np.asarray(a, dtype=np.float32).astype(np.float64)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 257])
def test_bf16_sampling_at_bin_edges_of_the_identity_flow(mc, n):
    """z at the edges k/16 of the identity flow's sixteen equal bins and at both
    ends of (0, 1): whichever neighbouring bin takes an edge, x = z and q = 1,
    to the rounding of sixteen FP32 widths (16 x 2^-24) per mapped coordinate
    and layer, at most three layers deep."""
    import torch
    fl = mc.Flow(workloads.flow_init(5))
    edges = np.concatenate([np.arange(1, 16) / 16.0, [2.0 ** -33, 2.0 ** -24, 1.0 - 2.0 ** -24, 0.5 - 2.0 ** -25]])
    rng = np.random.default_rng(n)
    z = _f32(rng.choice(edges, (n, 6)))
    d_x = torch.empty(n * 6, dtype=torch.float64, device="cuda")
    d_lq = torch.empty(n, dtype=torch.float64, device="cuda")
    fl.sample(_dev(z), n, d_x, d_lq, precision=mc.MCUBES_BF16)
    assert np.abs(d_x.cpu().numpy().reshape(n, 6) - z).max() <= 3 * 16 * 2.0 ** -24
    assert np.abs(d_lq.cpu().numpy()).max() <= 12 * 16 * 2.0 ** -24


@pytest.mark.parametrize("n", [1, 63, 65, 300])
def test_bf16_sampling_of_a_partial_wave_matches_oracle(mc, n):
    """A steep flow at sample counts around one wave, within the bounds that any
    sample of the BF16 path has (ten times the 99% ones: 2e-3 in x, 2e-2 in log q)."""
    import torch
    theta = _f32(workloads.flow_random(11, out_scale=0.8))
    fl = mc.Flow(theta)
    z = _f32(np.random.default_rng(n).uniform(0.0, 1.0, (n, 6)))
    d_x = torch.empty(n * 6, dtype=torch.float64, device="cuda")
    d_lq = torch.empty(n, dtype=torch.float64, device="cuda")
    fl.sample(_dev(z), n, d_x, d_lq, precision=mc.MCUBES_BF16)
    ref = [oracle.flow_sample(theta, p, bf16=True) for p in z]
    assert np.abs(d_x.cpu().numpy().reshape(n, 6) - np.array([r[0] for r in ref])).max() <= 2e-3
    assert np.abs(d_lq.cpu().numpy() - np.array([r[1] for r in ref])).max() <= 2e-2


def _plan(mc, dim, nb, **opt):
    return mc.mcubes_plan_create(1, [5.0] * dim + [0.5] * dim, dim, 1000, 1,
                                 mc.mcubes_default_options(nbins=nb, **opt))


@pytest.mark.parametrize("nb", [2, 3, 63, 64, 65, 127, 449, 500])
@pytest.mark.parametrize("alpha", [1.5, 0.7])
def test_refinement_at_wave_edges_matches_oracle(mc, nb, alpha):
    """Bin sums around whole waves of bins: smooth, one bin only, empty stretches, no
    weight at all.  Both sides sum at most 500 values in FP64 in their own order
    (2^-53 each, relative to the total) and divide a bin by its damped weight; with
    the weights of the filled rows within 1e6 of each other the edges agree to
    500 x 2^-53 x 1e6 bins at worst, 1e-12 being the parity bound of smooth rows."""
    import torch
    rng = np.random.default_rng(nb)
    rows = [rng.uniform(0.5, 2.0, nb), np.exp(rng.uniform(-3, 3, nb)), np.zeros(nb), np.zeros(nb)]
    rows[2][nb // 2] = 3.0
    if nb >= 63:
        gap = rng.uniform(0.5, 2.0, nb)
        gap[nb // 3:nb // 2] = 0.0
        rows.append(gap)
    dim = len(rows)
    bins = np.array(rows)
    grid = np.zeros((dim, nb + 1))
    for j in range(dim):
        w = rng.gamma(2.0, size=nb) + 1e-3
        grid[j, 1:] = np.cumsum(w) / w.sum()
        grid[j, -1] = 1.0
    ref = oracle.refine(grid, bins, alpha)
    plan = _plan(mc, dim, nb, alpha=alpha)
    out = torch.empty(dim * (nb + 1), dtype=torch.float64, device="cuda")
    d_bins = _dev(bins.reshape(-1))
    mc.mcubes_refine(plan, _dev(grid.reshape(-1)), d_bins, out)
    new = out.cpu().numpy().reshape(dim, nb + 1)
    assert np.all(np.diff(new, axis=1) >= 0) and np.all(new[:, 0] == 0) and np.all(new[:, -1] == 1)
    assert np.array_equal(new[3], grid[3])
    assert np.allclose(new, ref, rtol=1e-12, atol=1e-13)
    assert np.array_equal(d_bins.cpu().numpy(), bins.reshape(-1))


@pytest.mark.parametrize("T,skip,exact", [(1, 0, ()), (2, 2, ()), (64, 0, ()), (65, 3, ()), (1024, 0, ()),
                                          (40, 0, (7, 20)), (40, 30, (7, 20))])
def test_combination_over_many_iterations_matches_oracle(mc, T, skip, exact):
    """The quotients are formed side by side and summed in iteration order, as the oracle does."""
    import torch
    rng = np.random.default_rng(T + skip)
    I, v = 1.0 + 0.01 * rng.standard_normal(T), rng.uniform(0.5e-4, 2e-4, T)
    v[list(exact)] = 0.0
    plan = _plan(mc, 2, 10, skip=skip)
    state = torch.zeros(mc.MCUBES_STATE_LEN, dtype=torch.float64, device="cuda")
    est = torch.empty(2, dtype=torch.float64, device="cuda")
    for t in range(T):
        est.copy_(torch.tensor([I[t], v[t]], dtype=torch.float64))
        mc.mcubes_combine(plan, t, est, state, 1e-3)
    got = state.cpu().numpy()
    ref = oracle.combine(I, v, skip)
    assert got[4] == T and got[6] == 0
    if T > skip:
        assert np.allclose(got[:4], [ref[0], ref[1], ref[2], ref[3]], rtol=1e-14, atol=0)
        assert got[5] == float(ref[1] <= 1e-3 * abs(ref[0]))
    else:
        assert got[0] == 0 and np.isinf(got[1]) and got[5] == 0
    assert np.array_equal(got[8:8 + 2 * T].reshape(T, 2), np.stack([I, v], axis=1))


@pytest.mark.parametrize("adapt", [True, False])
@pytest.mark.parametrize("dim,nb,ncall", [(1, 2, 10), (3, 65, 5000), (10, 500, 20000)])
def test_iteration_equals_its_parts(mc, dim, nb, ncall, adapt):
    """mcubes_iteration against the same steps one by one: the same code on the same
    values, so the results are equal but for the order of the histogram's additions."""
    import torch
    plan = mc.mcubes_plan_create(1, [5.0] * dim + [0.4] * dim, dim, ncall, 9,
                                 mc.mcubes_default_options(nbins=nb, adapt_iters=-1 if adapt else 0))
    a, b = mc.Buffers(plan), mc.Buffers(plan)
    mc.mcubes_init_grid(plan, a.grid[0])
    b.grid[0].copy_(a.grid[0])
    a.bins.fill_(7.0)  # mcubes_iteration clears it, and leaves it alone when the grid is frozen
    for t in range(3):
        mc.mcubes_iteration(plan, t, a.grid[t & 1], a.grid[1 - (t & 1)], a.bins, a.partials, a.est, a.state, 1e-3)
        g = a.grid[t & 1]
        b.bins.zero_()
        mc.mcubes_vsample(plan, t, g, b.bins if adapt else None, b.partials)
        mc.mcubes_reduce(plan, b.partials, b.est)
        mc.mcubes_combine(plan, t, b.est, b.state, 1e-3)
        assert torch.equal(a.est, b.est) and torch.equal(a.state, b.state)
        if adapt:
            assert torch.allclose(a.bins, b.bins, rtol=1e-13, atol=0)
            out = torch.empty_like(g)
            mc.mcubes_refine(plan, g, a.bins, out)
            assert torch.equal(a.grid[1 - (t & 1)], out)
        else:
            assert torch.equal(a.grid[1 - (t & 1)], g) and bool((a.bins == 7.0).all())


@pytest.mark.parametrize("entry", ["mcubes_integrate", "mcubes_integrate_noalloc"])
@pytest.mark.parametrize("itmax", [1, 3, 4, 5, 12, 13, 33, 65])
def test_runs_ended_early_equal_the_run_of_that_length(mc, entry, itmax):
    """Iterations are enqueued ahead of the stop test: a run that a tolerance ends at
    iteration T leaves the result, trace and grid of a run of T iterations, wherever T
    falls in the iterations sent ahead.  Two runs of the same samples differ by the
    order of the histogram's additions (1e-12 over these few iterations)."""
    pr = workloads.small_product_peak()
    opt = mc.mcubes_default_options(nbins=50)
    call = lambda it, tol: getattr(mc, entry)(pr.family, pr.params, 3, 20000, it, tol, 3, opt)  # noqa: E731
    full = call(itmax, 0.0)
    assert full["iterations"] == itmax and not full["converged"]
    if itmax > 1:  # a tolerance between the errors after T - 1 and T iterations
        before = call(itmax - 1, 0.0)
        tol = 0.5 * (before["error"] / abs(before["estimate"]) + full["error"] / abs(full["estimate"]))
        early = call(100, tol)
        assert early["converged"] and early["iterations"] == itmax
        for k in ("estimate", "error", "trace_I", "trace_var", "grid"):
            assert np.allclose(np.array(early[k]), np.array(full[k]), rtol=1e-10, atol=0), k
        assert early["dof"] == full["dof"]
    if entry == "mcubes_integrate":
        assert full["kernel_ms"] > 0


@pytest.mark.parametrize("itmax", [1, 4, 40])
def test_exact_and_nonfinite_iterations_end_the_run(mc, itmax):
    """Zero variance (an integrand that is 0 on the whole cube) converges at once even
    without a tolerance; an overflow is an error."""
    r = mc.mcubes_integrate(mc.MCUBES_DISCONTINUOUS, [1.0, 1.0, -1.0, -1.0], 2, 1000, itmax, 0.0, 1)
    assert r["converged"] and r["iterations"] == 1 and r["estimate"] == 0.0 and r["error"] == 0.0
    with pytest.raises(mc.MCubesError) as e:
        mc.mcubes_integrate(mc.MCUBES_DISCONTINUOUS, [800.0, 800.0, 2.0, 2.0], 2, 1000, itmax, 0.0, 1)
    assert e.value.code == mc.MCUBES_E_NONFINITE and "iteration 0 " in str(e.value)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 300])
@pytest.mark.parametrize("direction", ["density", "sample"])
def test_fp32_flow_around_one_wave_matches_oracle(mc, n, direction):
    """The FP32 flow with every product split into BF16 parts, a steep flow, points
    up to the ends of (0, 1): |dx| <= 2e-5 and |d log q| <= 2e-4, the bounds of FP32
    sums of 96 + 64 + 64 products through four layers."""
    import torch
    theta = _f32(workloads.flow_random(13, out_scale=0.8))
    fl = mc.Flow(theta)
    pts = _f32(np.random.default_rng(n).uniform(0.0, 1.0, (n, 6)))
    pts[0] = [2.0 ** -33, 1.0 - 2.0 ** -24, 0.5, 1.0 / 32, 2.0 ** -10, 0.25]
    d_out = torch.empty(n * 6, dtype=torch.float64, device="cuda")
    d_lq = torch.empty(n, dtype=torch.float64, device="cuda")
    getattr(fl, direction)(_dev(pts), n, d_out, d_lq)
    fn = oracle.flow_density if direction == "density" else oracle.flow_sample
    ref = [fn(theta, p) for p in pts]
    assert np.abs(d_out.cpu().numpy().reshape(n, 6) - np.array([r[0] for r in ref])).max() <= 2e-5
    assert np.abs(d_lq.cpu().numpy() - np.array([r[1] for r in ref])).max() <= 2e-4


def test_fp32_flow_follows_every_parameter_change(mc):
    """Density right after set_params, an Adam step and a training call, on whichever
    stream the change ran, against the flow rebuilt from its parameters (bit-equal)."""
    import torch
    theta = _f32(workloads.flow_random(3, out_scale=0.3))
    n = 200
    rng = np.random.default_rng(0)
    x, w = _dev(rng.uniform(0.05, 0.95, (n, 6))), _dev(rng.uniform(0.5, 1.5, n))
    out, lq, lq2 = (torch.empty(k, dtype=torch.float64, device="cuda") for k in (6 * n, n, n))
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    fl = mc.Flow(workloads.flow_init(5))

    def check():
        fl.density(x, n, out, lq)
        mc.Flow(fl.params()).density(x, n, out, lq2)
        assert torch.equal(lq, lq2)

    check()
    fl.set_params(theta)
    check()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        fl.loss_grad(x, w, n, None, loss)
        fl.adam_step(1e-2)
    torch.cuda.current_stream().wait_stream(side)
    check()
    for precision in (mc.MCUBES_BF16, mc.MCUBES_FP32):
        fl.train(x, w, n, 2, 64, 1e-2, precision=precision)
        check()


@pytest.mark.parametrize("n,m", [(1, 256), (31, 33), (33, 255), (255, 256), (257, 300), (300, 512)])
def test_bf16_gradient_of_a_partial_workgroup(mc, n, m):
    """n samples, a part of the waves' 32 or the workgroups' 256, against the same n among
    m whose others have weight 0: the deltas of those are zeros, every sum has the same
    terms in the same places, so gradient and loss are equal (the loss to the order of
    its additions)."""
    import torch
    fl = mc.Flow(_f32(workloads.flow_random(6, out_scale=0.4)))
    rng = np.random.default_rng(n)
    x, w = _dev(rng.uniform(0.02, 0.98, (m, 6))), _dev(rng.uniform(0.2, 2.0, m))
    w[n:] = 0.0
    out = []
    for k in (n, m):
        grad = torch.empty(mc.MCUBES_FLOW_PARAMS, dtype=torch.float64, device="cuda")
        loss = torch.zeros(1, dtype=torch.float64, device="cuda")
        fl.loss_grad(x[:k].contiguous(), w[:k].contiguous(), k, grad, loss, precision=mc.MCUBES_BF16)
        out.append((grad, loss.item()))
    assert torch.equal(out[0][0], out[1][0]) and float(out[0][0].abs().max()) > 0
    assert out[0][1] == pytest.approx(out[1][1], rel=1e-14)


def test_bf16_gradient_over_several_passes_is_the_mean_of_its_halves(mc):
    """More samples than the workgroups hold at once (256 of 256): with equal weights and
    half the count the deltas of the halves are exactly twice those of the whole, so
    only the order of the FP32 sums differs (2^-24 sqrt(n) of the terms' size; 1e-5 in
    L2 over all components)."""
    import torch
    n = 2 * 65536 + 512
    fl = mc.Flow(_f32(workloads.flow_random(6, out_scale=0.4)))
    gen = torch.Generator(device="cuda").manual_seed(1)
    x = torch.rand(n, 6, generator=gen, device="cuda", dtype=torch.float64)
    w = torch.ones(n, dtype=torch.float64, device="cuda")
    out = []
    for a, b in ((0, n), (0, n // 2), (n // 2, n)):
        grad = torch.empty(mc.MCUBES_FLOW_PARAMS, dtype=torch.float64, device="cuda")
        loss = torch.zeros(1, dtype=torch.float64, device="cuda")
        fl.loss_grad(x[a:b].contiguous(), w[a:b].contiguous(), b - a, grad, loss, precision=mc.MCUBES_BF16)
        out.append((grad, loss.item()))
    mean = 0.5 * (out[1][0] + out[2][0])
    assert (out[0][0] - mean).norm() <= 1e-5 * mean.norm()
    assert abs(out[0][1] - 0.5 * (out[1][1] + out[2][1])) <= 1e-6 * abs(out[0][1])


@pytest.mark.parametrize("itmax", [2, 40])  # 3 x 4 and 3 x 80 trace values against 3 x 2 x 2 bin sums
def test_batch_results_and_traces(mc, itmax):
    """Results and traces read through the bin sums' place and past it: the
    first iteration is that of a single-iteration call bit for bit, and the
    estimate is the weighted mean of the trace (sums of itmax terms: 1e-13)."""
    items = [(workloads.PRODUCT_PEAK, 2, 20_000, [3.0, 4.0, 0.3, 0.6]), (workloads.GAUSSIAN, 2, 5_000, [2.0, 3.0, 0.5, 0.4]),
             (workloads.CORNER_PEAK, 2, 30_011, [1.0, 2.0, 0.0, 0.0])]
    b = mc.Batch(items, 7, mc.mcubes_default_options(nbins=2))
    _, once = b.integrate(1, 0.0, traces=True)
    _, res = b.integrate(itmax, 0.0, traces=True)
    for r, o in zip(res, once):
        I, var = np.asarray(r["trace_I"]), np.asarray(r["trace_var"])
        assert I.shape == var.shape == (itmax,) and r["iterations"] == itmax
        assert (I[0], var[0]) == (o["trace_I"][0], o["trace_var"][0])
        mean = (I / var).sum() / (1.0 / var).sum()
        assert abs(r["estimate"] - mean) <= 1e-13 * abs(mean)
        assert abs(r["error"] - (1.0 / var).sum() ** -0.5) <= 1e-13 * r["error"]


@pytest.mark.parametrize("n", [1, 2, 300])
def test_batch_iterations_equal_single_runs(mc, n):
    """One integrand and more than there are CUs: every iteration of every one
    as in a run of its own (the samples are the same, the sums differ in their
    order: 1e-12 of the first estimate and variance, 1e-9 once the grids, refined
    from bin sums in another order, have drifted apart)."""
    items = [(workloads.PRODUCT_PEAK, 2, 2000 + 37 * i, [3.0, 4.0, 0.3, 0.6]) for i in range(n)]
    b = mc.Batch(items, 11, mc.mcubes_default_options(nbins=20))
    for graph in (True, False):
        _, res = b.integrate(3, 0.0, use_graph=graph, grids=True, traces=True)
        for i in sorted({0, n // 2, n - 1}):
            opt = mc.mcubes_default_options(nbins=20, stream_id=i)
            one = mc.mcubes_integrate(*items[i][:1], items[i][3], 2, items[i][2], 3, 0.0, 11, opt)
            r = res[i]
            assert (r["iterations"], r["dof"]) == (one["iterations"], one["dof"])
            for t in range(3):
                tol = 1e-12 if t == 0 else 1e-9
                assert r["trace_I"][t] == pytest.approx(one["trace_I"][t], rel=tol)
                assert r["trace_var"][t] == pytest.approx(one["trace_var"][t], rel=tol)
            assert np.abs(np.asarray(r["grid"]) - np.asarray(one["grid"])).max() <= 1e-9


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("dim", range(1, 11))
def test_batch_of_all_families_equals_single_runs(mc, dim, precision):
    """Every family, with p = 2 and p > 2, in one launch of a dimension: one
    iteration of each as in a run of its own (the same samples in another order
    of summation: 1e-12 of the sums' size)."""
    rng = np.random.default_rng(dim)
    sizes = {}
    for n in range(3, 40_000):  # the first budgets past 1000, else below, of two and of more samples per cube
        g = max(1, int((n / 2) ** (1.0 / dim) + 1e-9))
        two = n // g ** dim == 2
        if two not in sizes or (sizes[two] < 1000 <= n):
            sizes[two] = n
    probs = [workloads.random_problem(rng, f, dim, n, 30) for f in range(8) for n in sizes.values()
             if not (f == workloads.MIXTURE and dim == 1)]
    kw = dict(nbins=30, precision=mc.MCUBES_FP32 if precision == "fp32" else mc.MCUBES_FP64)
    b = mc.Batch([(q.family, q.dim, q.ncall, q.params) for q in probs], 5, mc.mcubes_default_options(**kw))
    _, res = b.integrate(1, 0.0, grids=True, traces=True)
    for i, (q, r) in enumerate(zip(probs, res)):
        one = mc.mcubes_integrate(q.family, q.params, dim, q.ncall, 1, 0.0, 5,
                                  mc.mcubes_default_options(stream_id=i, **kw))
        assert r["samples_per_cube"] == one["samples_per_cube"], q.name
        size = abs(one["estimate"]) + np.sqrt(one["samples_per_iter"]) * one["error"]
        assert abs(r["estimate"] - one["estimate"]) <= 1e-12 * size, q.name
        assert abs(r["error"] - one["error"]) <= 1e-12 * size, q.name
        assert np.abs(np.asarray(r["grid"]) - np.asarray(one["grid"])).max() <= 1e-9, q.name


@pytest.mark.parametrize("itmax", [1, 2, 5])
@pytest.mark.parametrize("adapt", [-1, 0, 1, 4])
def test_batch_graph_of_later_iterations(mc, adapt, itmax):
    """The replayed iterations, with and without refinement, against launches
    one by one (the bin sums' order differs from run to run: 1e-9), three times."""
    items = [(workloads.GAUSSIAN, 3, 20_000 + i, [5.0, 6.0, 7.0, 0.4, 0.5, 0.6]) for i in range(5)]
    b = mc.Batch(items, 3, mc.mcubes_default_options(nbins=50, adapt_iters=adapt))
    _, want = b.integrate(itmax, 0.0, use_graph=False, grids=True, traces=True)
    for _ in range(3):
        _, got = b.integrate(itmax, 0.0, use_graph=True, grids=True, traces=True)
        for g, w in zip(got, want):
            assert g["iterations"] == w["iterations"] == itmax
            np.testing.assert_allclose(g["trace_I"], w["trace_I"], rtol=1e-9)
            np.testing.assert_allclose(g["trace_var"], w["trace_var"], rtol=1e-9)
            np.testing.assert_allclose(g["grid"], w["grid"], atol=1e-9, rtol=0)


@pytest.mark.parametrize("n,m", [(1, 64), (15, 17), (63, 64), (65, 128), (200, 512)])
def test_fp32_gradient_of_a_partial_workgroup(mc, n, m):
    """n samples, a part of the products' 16 or the workgroups' 64, against the
    same n among m whose others have weight 0: every sum has the same terms in
    the same order and zeros behind them, so gradient and loss are equal (the
    loss to the order of its additions)."""
    import torch
    fl = mc.Flow(_f32(workloads.flow_random(6, out_scale=0.4)))
    rng = np.random.default_rng(n)
    x, w = _dev(rng.uniform(0.02, 0.98, (m, 6))), _dev(rng.uniform(0.2, 2.0, m))
    w[n:] = 0.0
    out = []
    for k in (n, m):
        grad = torch.empty(mc.MCUBES_FLOW_PARAMS, dtype=torch.float64, device="cuda")
        loss = torch.zeros(1, dtype=torch.float64, device="cuda")
        fl.loss_grad(x[:k].contiguous(), w[:k].contiguous(), k, grad, loss, precision=mc.MCUBES_FP32)
        out.append((grad, loss.item()))
    assert torch.equal(out[0][0], out[1][0]) and float(out[0][0].abs().max()) > 0
    assert out[0][1] == pytest.approx(out[1][1], rel=1e-14)
