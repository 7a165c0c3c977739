"""GPU parity where the call chain changes form: counts of rows that the
float64 fix-ups take (their partner segments, the 64-row chunks in which they
are merged, none and all), and the sizes either side of the float64 passes'
step groups.  Oracle, metrics and tolerances of tests/gpu_util.py."""
import numpy as np
import pytest

from paper_2010_02994_amd import workloads as W
from tests.gpu_util import check, oracle_ref, run_gpu, say

pytestmark = pytest.mark.gpu


def isolated_case(seed, core, far, spacing):
    """`core` events within half a bandwidth of the origin (the first and last
    events among them, so that the float32 origin sits there) and `far` events
    on a square grid around them, each `spacing` bandwidths from its nearest
    neighbour: their rates are about exp(-spacing^2 / 2)."""
    rng = np.random.default_rng(seed)
    m = int(np.ceil(np.sqrt(far))) + 3
    g = np.stack(np.meshgrid(*[np.arange(-m, m + 1)] * 2), axis=-1).reshape(-1, 2).astype(float)
    g = g[np.abs(g).max(axis=1) >= 1]
    g = g[np.argsort((g**2).sum(axis=1), kind="stable")][:far] * spacing
    x = np.concatenate([0.1 * rng.standard_normal((core, 2)), g])
    x = x[rng.permutation(len(x))]
    at = np.flatnonzero(np.abs(x).max(axis=1) < spacing / 2)
    if core >= 2:   # core events first and last
        for end, j in ((0, at[0]), (len(x) - 1, at[-1])):
            x[[end, j]] = x[[j, end]]
    t = np.sort(rng.uniform(0.0, 2.0, size=len(x)))
    return x, t, np.array([0.5, 1.0, 10.0, 0.4, 0.2, 1.0])


@pytest.mark.parametrize("prec,spacing", [("mixed", 20.0), ("fp64", 37.0)])
@pytest.mark.parametrize("core,far", [(200, 1), (190, 63), (130, 65), (200, 130), (70, 520), (40, 1100)])
def test_flagged_row_counts(prec, spacing, core, far):
    import torch

    from paper_2010_02994_amd import api
    x, t, p = isolated_case(core + far, core, far, spacing)
    say(f"case flagged rows core={core} far={far} prec={prec}")
    got = run_gpu(x, t, p, prec)
    info, flags = api.diagnostics(torch.tensor(x, device="cuda:0"), torch.tensor(t, device="cuda:0"), p, prec=prec)
    # the core's own rows stand far above the window, the isolated ones below
    assert info["flagged_rows"] == far
    assert np.array_equal(flags != 0, np.abs(x).max(axis=1) > spacing / 2)
    check(prec, got, oracle_ref(x, t, p), p, label=f"far{far}")


@pytest.mark.parametrize("prec,spacing", [("mixed", 17.0), ("fp64", 37.0)])
def test_every_row_flagged(prec, spacing):
    """No event within reach of another: every row takes the fix-ups."""
    import torch

    from paper_2010_02994_amd import api
    x, t, p = isolated_case(5, 0, 96, spacing)
    say(f"case every row flagged prec={prec}")
    got = run_gpu(x, t, p, prec)
    info, _ = api.diagnostics(torch.tensor(x, device="cuda:0"), torch.tensor(t, device="cuda:0"), p, prec=prec)
    assert info["flagged_rows"] == len(t)
    check(prec, got, oracle_ref(x, t, p), p, label="all")


@pytest.mark.parametrize("seed,n,d,ties", [(31, 70, 1, 3), (32, 577, 4, 0), (33, 1100, 3, 40), (34, 6144, 2, 5),
                                           (35, 6145, 2, 5), (36, 900, 5, 2)])
def test_float64_step_groups(seed, n, d, ties):
    """Float64 calls with two step groups per tile (up to 700 tiles, d <= 4) and
    just outside: gradient, and the rate pass alone (loglik)."""
    import torch

    from paper_2010_02994_amd import api
    w = W.random_case(seed, n, d, ties=ties, t_span=max(3.0, n / 40))
    say(f"case step groups n={n} d={d} ties={ties}")
    ref = oracle_ref(w.x, w.t, w.params)
    got = run_gpu(w.x, w.t, w.params, "fp64")
    check("fp64", got, ref, w.params, label=w.name)
    ll = api.loglik(torch.tensor(w.x, device="cuda:0"), torch.tensor(w.t, device="cuda:0"), w.params, prec="fp64")
    assert abs(ll - ref.ll) <= 1e-10 * abs(ref.ll)


@pytest.mark.parametrize("prec", ["mixed", "fp64"])
@pytest.mark.parametrize("tau,omega", [(0.05, 0.5), (40.0, 300.0), (0.05, 300.0), (2.0, 40.0)])
@pytest.mark.parametrize("n,d", [(1500, 2), (1100, 6), (6200, 1)])
def test_culled_terms_are_bitwise_identical(prec, tau, omega, n, d):
    """Far tiles that keep only the excitation term (short background
    bandwidth), only the background term (fast decay), neither, and a mixture:
    every output equals the all-pairs run's bit for bit, with and without the
    gradient."""
    import torch

    from paper_2010_02994_amd import api
    w = W.random_case(41, n, d, ties=3, t_span=400.0)
    p = w.params.copy()
    p[2], p[4] = tau, omega
    say(f"case culled terms n={n} d={d} tau={tau} omega={omega} prec={prec}")
    a = run_gpu(w.x, w.t, p, prec)
    b = run_gpu(w.x, w.t, p, prec + "+cull")
    assert a[0] == b[0] and np.array_equal(a[1], b[1]) and np.array_equal(a[2], b[2])
    x, t = torch.tensor(w.x, device="cuda:0"), torch.tensor(w.t, device="cuda:0")
    assert api.loglik(x, t, p, prec=prec) == api.loglik(x, t, p, prec=prec + "+cull")


@pytest.mark.parametrize("params,scale", [((0.5, 1.0, 1e20, 0.0, 1e20, 1.0), 1.0), ((0.5, 1.0, 1e20, 0.3, 1e20, 1.0), 1.0),
                                          ((0.5, 1.0, 1.0, 0.0, 1.0, 1e-20), 1.0)])
@pytest.mark.parametrize("n,d", [(70, 1), (700, 2), (700, 6)])
@pytest.mark.parametrize("cull", ["", "+cull"])
def test_mixed_scales_beyond_float32(params, scale, n, d, cull):
    """omega tau_t, or (tau_x / h)^2, beyond float32's range: the excitation of
    every pair is zero in float32 and next to nothing in fact (its weight is
    zero, or its exponent below -1e17), the background as usual, and pairs
    that do not interact (an event with itself among them) add nothing."""
    rng = np.random.default_rng(n + d)
    x = scale * rng.normal(size=(n, d))
    t = np.sort(rng.uniform(0.0, 10.0, n))
    p = np.array(params)
    say(f"case scales n={n} d={d} params={params} cull={cull}")
    got = run_gpu(x, t, p, "mixed" + cull)
    ref = oracle_ref(x, t, p)
    ll, gx, gp = got
    assert abs(ll - ref.ll) <= 1e-5 * abs(ref.ll)
    assert np.all(np.isfinite(gp))
    d_row = np.linalg.norm(gx - ref.gx, axis=1)
    assert np.all(d_row <= 3e-4 * ref.row_scale)


@pytest.mark.parametrize("prec,spacing", [("mixed", 20.0), ("fp64", 37.0)])
@pytest.mark.parametrize("core,far", [(200, 1), (130, 65), (40, 1100), (0, 96), (4200, 1), (9000, 130), (18000, 700), (33000, 3)])
def test_flagged_rows_without_a_gradient(prec, spacing, core, far):
    """Log-likelihood and per-event terms of calls whose flagged rows are split
    into partner segments (one up to 4,095 events, then two, four, eight and,
    with few rows, 16): the log-likelihood at the precision's tolerance, and
    the flagged rows' terms, which are float64 sums in both precisions, at
    float64's."""
    import oracle
    import torch

    from paper_2010_02994_amd import api
    x, t, p = isolated_case(core + far, core, far, spacing)
    xd, td = torch.tensor(x, device="cuda:0"), torch.tensor(t, device="cuda:0")
    say(f"case flagged rows without a gradient core={core} far={far} prec={prec}")
    terms, ll = api.event_terms(xd, td, p, prec=prec)
    info, flags = api.diagnostics(xd, td, p, prec=prec)
    assert info["flagged_rows"] == far and np.array_equal(flags != 0, np.abs(x).max(axis=1) > spacing / 2)
    _, ref, _, _ = oracle.loglik_grad(x, t, p, threads=True, want_grad_x=False)
    tol = {"mixed": 1e-5, "fp64": 1e-10}[prec]
    assert abs(ll - ref) <= tol * abs(ref)
    assert api.loglik(xd, td, p, prec=prec) == ll
    rows = np.flatnonzero(flags)
    got, want = terms.cpu().numpy()[rows], oracle.event_terms(x, t, p, rows=rows)
    assert np.all(np.abs(got[:, 2:] - want[:, 2:]) <= 1e-10 * np.maximum(1.0, np.abs(want[:, 2:])))
    # rates of exp(-spacing^2 / 2), down to 1e-297: the exponent's rounding, up to
    # 700 ulp(1), is the value's relative error
    assert np.all(np.abs(got[:, :2] - want[:, :2]) <= 1e-10 * np.abs(want[:, :2]))


def test_one_flagged_row_costs_little_without_a_gradient():
    """At N = 50,000 the exact recomputation of one row, split over the chip,
    adds under 5 % to a log-likelihood (one workgroup took 180 us, 11 %)."""
    import torch

    from paper_2010_02994_amd import api
    w = W.config2(seed=3, n=50000, same_density=True)
    td, xs = torch.tensor(w.t, device="cuda:0"), []
    for far in (0, 1):
        x = w.x.copy()
        if far:
            x[20000] = x.max(axis=0) + 60.0 * max(w.params[1], w.params[5])
        xs.append(torch.tensor(x, device="cuda:0"))
    us = ([], [])
    for _ in range(40):   # in turn; the medians of the later half
        for far in (0, 1):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            api.loglik(xs[far], td, w.params, prec="fp64")
            b.record()
            b.synchronize()
            us[far].append(a.elapsed_time(b) * 1e3)
            info, _ = api.diagnostics(xs[far], td, w.params, prec="fp64")
            assert info["flagged_rows"] == far
    without, with_one = (float(np.median(v[20:])) for v in us)
    say(f"  us: {without:.0f} and with one flagged row {with_one:.0f}")
    assert with_one <= 1.05 * without


def test_one_flagged_row_beside_a_short_gradient_pass():
    """Culling with a short background bandwidth and fast decay leaves a
    gradient pass shorter than a flagged row's recomputation beside it was:
    the row adds under 13 % to the call (16 % before its partners were read a
    step ahead)."""
    import torch

    from paper_2010_02994_amd import api
    w = W.config2(seed=3, n=50000, same_density=True)
    p = w.params.copy()
    p[[1, 2, 4, 5]] = 40.0, 2.0, 2.0, 5.0
    td, xs, us = torch.tensor(w.t, device="cuda:0"), [], ([], [])
    for far in (0, 1):
        x = w.x.copy()
        if far:
            x[20000] = x.max(axis=0) + 700.0
        xs.append(torch.tensor(x, device="cuda:0"))
    say("case one flagged row beside a short gradient pass")
    for _ in range(60):   # in turn; the medians of the later half
        for far in (0, 1):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            api.grad(xs[far], td, p, prec="mixed+cull")
            b.record()
            b.synchronize()
            us[far].append(a.elapsed_time(b) * 1e3)
            info, _ = api.diagnostics(xs[far], td, p, prec="mixed+cull")
            assert info["flagged_rows"] == far
    without, with_one = (float(np.median(v[30:])) for v in us)
    say(f"  us: {without:.0f} and with one flagged row {with_one:.0f}")
    assert with_one <= 1.13 * without
