"""GPU parity of the Bayesian MDS log-likelihood and gradients against the
CPU oracle (Sec. 2.2.3)."""
import numpy as np
import pytest

import oracle
from paper_2010_02994_amd import workloads as W
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

TOL = {"fp64": {"ll": 1e-12, "ds": 1e-11, "gx": 1e-11}, "mixed": {"ll": 1e-5, "ds": 1e-4, "gx": 1e-4}}


def _gpu(c, prec):
    import torch
    from paper_2010_02994_amd import api
    x = torch.tensor(c.x, device="cuda:0")
    dl = torch.tensor(c.delta, device="cuda:0")
    out4, gx = api.bmds(x, dl, c.sigma, prec=prec)
    torch.cuda.synchronize()
    return out4.cpu().numpy(), gx.cpu().numpy()


def _check(c, prec, label):
    st, ll, ds, M, gx_ref = oracle.bmds(c.x, c.delta, c.sigma)
    assert st == 0
    o, gx = _gpu(c, prec)
    e_ll = abs(o[0] - ll) / abs(ll)
    e_ds = abs(o[1] - ds) / max(abs(ds), M / c.sigma)
    e_gx = np.linalg.norm(gx - gx_ref) / np.linalg.norm(gx_ref)
    say(f"  bmds {label} {prec}: ll {o[0]:.15g} ref {ll:.15g} | err ll {e_ll:.2e} dsigma {e_ds:.2e} gx {e_gx:.2e}")
    t = TOL[prec]
    assert o[3] == 0 and o[2] == M
    assert e_ll <= t["ll"] and e_ds <= t["ds"] and e_gx <= t["gx"]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("seed,n,d,missing,groups", [(1, 1000, 2, 0.1, 0), (2, 700, 6, 0.0, 40), (3, 2, 3, 0.0, 0),
                                                      (4, 65, 2, 0.0, 0), (5, 257, 4, 0.5, 0), (6, 1500, 8, 0.0, 0)])
def test_bmds_matches_oracle(prec, seed, n, d, missing, groups):
    c = W.bmds_case(seed, n, d, missing=missing, groups=groups)
    say(f"case bmds n={n} d={d} missing={missing} groups={groups} prec={prec}")
    _check(c, prec, c.name)


def test_bmds_invalid_delta_is_reported():
    import torch
    c = W.bmds_case(7, 300, 2)
    c.delta[200, 17] = -1.0
    say("case bmds invalid delta")
    o, gx = _gpu(c, "fp64")
    assert o[3] == -3 and np.isnan(o[0]) and np.all(np.isnan(gx))


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("row", [0, 63, 64, 299])
def test_bmds_nonfinite_coordinate_is_reported(prec, row):
    """A non-finite coordinate in any row band (first and last rows of a
    band, the last event) makes the call report a data error."""
    c = W.bmds_case(7, 300, 2)
    c.x[row, 1] = np.inf if row % 2 else np.nan
    say(f"case bmds non-finite x row={row} prec={prec}")
    o, gx = _gpu(c, prec)
    assert o[3] == -3 and np.isnan(o[0]) and np.isnan(o[1]) and np.all(np.isnan(gx))


def test_bmds_deterministic():
    c = W.bmds_case(8, 900, 3, missing=0.2)
    say("case bmds determinism")
    a = _gpu(c, "mixed")
    b = _gpu(c, "mixed")
    assert np.array_equal(a[0], b[0]) and np.array_equal(a[1], b[1])


_big = {}


def _check_device_case(key, seed, n, d, prec):
    """Device-drawn case of size n (5 % unobserved), the oracle's result
    cached per (n, d) across the precisions."""
    import torch
    from paper_2010_02994_amd import api
    if _big.get("key") != key:
        _big.clear()
        x, dl, sigma = W.bmds_case_device(seed, n, d, missing=0.05)
        _big.update(key=key, case=(x, dl, sigma), ref=oracle.bmds(x.cpu().numpy(), dl.cpu().numpy(), sigma))
    x, dl, sigma = _big["case"]
    st, ll, ds, M, gx_ref = _big["ref"]
    assert st == 0
    say(f"case bmds n={n} d={d} prec={prec}")
    out4, gxd = api.bmds(x, dl, sigma, prec=prec)
    torch.cuda.synchronize()
    o, gx = out4.cpu().numpy(), gxd.cpu().numpy()
    e_ll = abs(o[0] - ll) / abs(ll)
    e_ds = abs(o[1] - ds) / max(abs(ds), M / sigma)
    e_gx = np.linalg.norm(gx - gx_ref) / np.linalg.norm(gx_ref)
    say(f"  err ll {e_ll:.2e} dsigma {e_ds:.2e} gx {e_gx:.2e}")
    t = TOL[prec]
    assert o[3] == 0 and o[2] == M
    assert e_ll <= t["ll"] and e_ds <= t["ds"] and e_gx <= t["gx"]


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("d", [6, 2])
def test_bmds_many_tiles_matches_oracle(prec, d):
    """N = 12,000 (over 4,096 tiles, so several columns per lane)."""
    _check_device_case(("many", d), 9 + d, 12000, d, prec)


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("n", [11456, 11457])
def test_bmds_tile_count_boundary(prec, n):
    """Either side of the 4,096-tile switch: N = 11,456 is the largest with
    fewer tiles (179 bands, 4,095 tiles: one workgroup per tile for float64
    pairs, single-band strips of one column per lane for float32 pairs), and
    N = 11,457 the smallest with more (the wide strips)."""
    _check_device_case(("edge", n), 30 + n % 7, n, 3, prec)


@pytest.mark.parametrize("spread", [0.1, 0.6, 2.0])
@pytest.mark.parametrize("n,d", [(2, 1), (3, 2), (66, 5), (67, 4), (255, 8), (259, 2)])
def test_bmds_near_pairs_and_row_groups(n, d, spread):
    """Float64 pairs at small z (the tail's fitted forms, coincident events,
    waves that hold near and far pairs) at counts that end a row band within a
    group of rows.  Each pair's terms carry some tens of roundings and a sum
    over a row up to N more, so the errors stay below 1e-13 of the sums of the
    terms' magnitudes."""
    rng = np.random.default_rng(n + d)
    sigma = 0.8
    x = rng.normal(size=(n, d)) * spread * sigma
    if n > 4:
        x[4] = x[1]
        x[n // 2:] *= 4.0
    dist = np.sqrt(((x[:, None] - x[None]) ** 2).sum(-1))
    delta = np.abs(dist + sigma * rng.normal(size=(n, n)))
    say(f"case bmds near pairs n={n} d={d} spread={spread}")
    st, ll, ds, M, gx_ref = oracle.bmds(x, delta, sigma)
    assert st == 0
    o, gx = _gpu(_Case(x, delta, sigma), "fp64")
    low = np.tril(np.ones((n, n), bool), -1)
    size = (delta + dist) / sigma ** 2 + 1.0 / sigma   # bounds |delta - d|/sigma^2 + rho/sigma (rho <= 0.8)
    size = np.where(low, size, 0.0)
    row = size.sum(1) + size.sum(0)
    s_ll = np.where(low, (delta - dist) ** 2 / (2 * sigma ** 2) + abs(np.log(sigma)) + 0.7, 0.0).sum()
    s_ds = np.where(low, (delta - dist) ** 2 / sigma ** 3 + (delta + dist) * dist / sigma ** 3 + 2.0 / sigma, 0.0).sum()
    assert o[3] == 0 and o[2] == M
    assert abs(o[0] - ll) <= 1e-13 * s_ll
    assert abs(o[1] - ds) <= 1e-13 * s_ds
    assert np.all(np.abs(gx - gx_ref) <= 1e-13 * row[:, None])


class _Case:
    def __init__(self, x, delta, sigma):
        self.x, self.delta, self.sigma = x, delta, sigma


@pytest.mark.parametrize("far,near", [(37, 5), (66, 64), (1, 0)])
def test_bmds_overflowing_pair_stays_in_its_rows(far, near):
    """One event so far away that its distance overflows, observed from one
    other event only: those two events' gradients are not finite, and every
    other event's is what it is without that pair."""
    c = W.bmds_case(9, 70, 3)
    c.x[far] = 1e200
    c.delta[far, :] = c.delta[:, far] = np.nan
    say(f"case bmds overflow far={far} near={near}")
    o0, g0 = _gpu(c, "fp64")
    assert o0[3] == 0 and np.all(np.isfinite(g0))
    c.delta[far, near] = c.delta[near, far] = 1.0
    o, g = _gpu(c, "fp64")
    rest = np.setdiff1d(np.arange(70), [far, near])
    assert not np.isfinite(o[0]) and not np.any(np.isfinite(g[[far, near]]))
    assert np.all(np.abs(g[rest] - g0[rest]) <= 1e-14 * np.abs(g0).max())


@pytest.mark.parametrize("value", [-1.0, np.inf])
@pytest.mark.parametrize("row,col", [(1, 0), (64, 63), (299, 298), (299, 0)])
def test_bmds_strips_report_an_invalid_delta(row, col, value):
    """Float32 pairs (strips): an invalid dissimilarity in the first and last
    rows and in the corners of a band reaches the totals and every gradient
    row, and the next call with valid data does not see it."""
    c = W.bmds_case(7, 300, 2)
    keep = c.delta[row, col]
    c.delta[row, col] = value
    say(f"case bmds strips invalid delta row={row} col={col}")
    o, gx = _gpu(c, "mixed")
    assert o[3] == -3 and np.isnan(o[0]) and np.isnan(o[1]) and np.all(np.isnan(gx))
    c.delta[row, col] = keep
    _check(c, "mixed", c.name)


@pytest.mark.parametrize("sigma", [1.0, 1e-6, 1e-10, 1e-15])
@pytest.mark.parametrize("n,d,apart", [(2, 3, 0.0), (2, 1, 1e-20), (70, 2, 0.0), (11457, 2, 0.0)])
def test_bmds_coincident_float32_pairs_add_no_direction(n, d, apart, sigma):
    """Float32 pairs (narrow strips, and the wide ones from 11,457 events on) of
    events at one place, whose residuals over sigma^2 reach 1e30: their
    distances are exactly zero (or so small that their squares are subnormal),
    so every gradient entry is zero.  The scalars follow
    from d = 0: each pair adds delta^2/(2 sigma^2) + log Phi(0), and
    delta^2/sigma^3 (float32 terms: 1e-5)."""
    import torch
    from paper_2010_02994_amd import api
    x = torch.zeros((n, d), dtype=torch.float64, device="cuda:0")
    x[1:] += apart
    dl = torch.ones((n, n), dtype=torch.float64, device="cuda:0")
    say(f"case bmds coincident n={n} d={d} apart={apart} sigma={sigma}")
    out4, gx = api.bmds(x, dl, sigma, prec="mixed")
    o = out4.cpu().numpy()
    m = n * (n - 1) // 2
    assert o[3] == 0 and o[2] == m
    assert not torch.any(gx).item()   # all zero (a NaN would count as nonzero)
    assert o[0] == pytest.approx(-m * (np.log(sigma) + 0.5 / sigma**2 + np.log(0.5)), rel=1e-5)
    assert o[1] == pytest.approx(m * (1.0 / sigma**3 - 1.0 / sigma), rel=1e-5, abs=1e-5 * m / sigma)
