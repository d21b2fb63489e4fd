"""The nonlinear combination (blend_c, blend_vjp) with linear weights far from the usual
ones, against the oracle: the kernels form its denominator g0 e0 + g1 e1 + g2 e2 as
e0 + g1 (e1 - e0) + g2 (e2 - e0), which would cancel if e0 could exceed e1 and e2 by much.
It cannot, since the high-degree indicator is never far below the others, so every weight
that the problem accepts is as accurate as the scheme itself.

Bounds.  The scheme divides p0 - g1 p1 - g2 p2 by g0 before it multiplies by w0, and
w0 / g0 = e0 / sum is at most 1.25: the candidates' roundings (some ten of the data's
size each, and as many from the indicators) stay a few dozen in all, 1e-13 in FP64 and 1e-5
in FP32, where the oracle divides by g0 in 64 bits: with g0 = 1e-6 its own 64 bits leave 1e-9,
which FP64 is then held to instead."""
import numpy as np
import pytest
import torch

from oracle import hweno_ref as o
from tests import test_host_math as M

WEIGHTS = [(1.0 / 3, 1.0 / 3, 1.0 / 3), (1e-2, 0.495, 0.495), (1e-6, 1.0 - 2e-6, 1e-6),
           (1e-6, 1e-6, 1.0 - 2e-6), (1e-6, 0.5, 0.499999)]


def _ids(w):
    return "%g,%g,%g" % w


def _rows(seed, prec):
    rows = M._data(seed) if prec == "d" else M._data(seed, **M.FP32_RANGE)
    g = np.random.default_rng(seed + 1)
    # stencils on which the quintic's (rows 0, 1, 2 mod 4) or quartic's (3) indicator is as
    # small as it gets beside the others
    n = len(rows) // 4
    u1 = 10.0 ** g.uniform(-2, 2, n)
    u2 = -0.8 * u1 * (1 + 0.05 * g.standard_normal(n))
    f0, H0 = g.standard_normal(n), 1e-3 * g.standard_normal(n)
    lap, t = u1 - u2, u1 + u2
    Hd, Hs = -6.067488135033763 / 3.012679250059034 * lap, 2 * H0 - 45.165651404159786 / 15.029579351881592 * t
    rows[::4] = np.stack([f0 + u1 - H0, f0, f0 + H0 - u2, (Hs + Hd) / 2, H0, (Hs - Hd) / 2], 1)
    return rows


@pytest.fixture
def weights(request, monkeypatch):
    monkeypatch.setattr(M, "LIN", request.param)
    monkeypatch.setattr(M, "LIM", request.param)
    return request.param


@pytest.mark.parametrize("weights", WEIGHTS, indirect=True, ids=_ids)
@pytest.mark.parametrize("prec", ["d", "f"])
def test_reconstruction_and_limiter_take_any_weights(prec, weights):
    rows = _rows(51, prec)
    tol = 1e-5 if prec == "f" else (1e-9 if weights[0] < 1e-3 else 1e-13)
    if prec == "f":
        rows = rows.astype(np.float32).astype(np.float64)
    t = torch.as_tensor(rows, dtype=torch.float64)
    got = M._run("r", prec, rows)
    ref = o.hweno_plus(*[t[:, c] for c in range(6)], weights, M.EPS).numpy()
    err = np.abs(got - ref) / M._scale(rows)
    assert np.isfinite(got).all() and err.max() <= tol, (err.max(), rows[err.argmax()])

    lim = rows.copy()
    n = len(lim[::4])
    g = np.random.default_rng(52)
    h = lim[:, 5] = 2.0 ** -g.integers(3, 10, len(lim)).astype(float)
    d1 = 10.0 ** g.uniform(-2, 2, n)
    d2 = 0.629 * d1 * (1 + 0.05 * g.standard_normal(n))
    D, lap = d1 + d2, d2 - d1
    e = D * (0.5 * 3.0 / 16.0) / (2.440625 + 9.0 / 256.0)
    Vs, Vd = D + e, -12.554318802466193 / 6.254843361443233 * lap
    u0 = g.standard_normal(n)
    lim[::4, :5] = np.stack([u0 - d1, u0, u0 + d2, (Vs + Vd) / (2 * h[::4]), (Vs - Vd) / (2 * h[::4])], 1)
    if prec == "f":
        lim = lim.astype(np.float32).astype(np.float64)
    t = torch.as_tensor(lim, dtype=torch.float64)
    got = M._run("l", prec, lim)
    ref = o.limit_derivative(*[t[:, c] for c in range(6)], weights, M.EPS).numpy()
    scale = np.maximum(np.abs(lim[:, :3]).max(1) / lim[:, 5], np.abs(lim[:, 3:5]).max(1))
    err = np.abs(got - ref) / scale
    assert np.isfinite(got).all() and err.max() <= tol, (err.max(), lim[err.argmax()])


def test_high_degree_indicators_are_never_far_below_the_others():
    """min over all data of c0 / c1 and c0 / c2 without eps (which only brings the ratios
    nearer to one): a ratio of quadratic forms, the smallest generalised eigenvalue."""
    E = np.eye(5)
    # (u1, u2, H0, Hs, Hd) as in hw_blend
    u1, u2, H0, Hs, Hd = E
    lap, t = u1 - u2, u1 + u2
    sq = lambda v: np.outer(v, v)
    c0 = (3 / 13) * sq(H0) + sq(6.067488135033763 * lap + 3.012679250059034 * Hd) \
        + sq(15.029579351881592 * (Hs - 2 * H0) + 45.165651404159786 * t) \
        + 2.2469689522048239 * sq(t) + 0.24822509386187025 * sq(lap)
    for u in (u1, u2):
        c = (3 / 13) * sq(H0) + sq(u)
        # c <= c0 / 0.89 for all data: c0 - 0.89 c is positive semidefinite
        assert np.linalg.eigvalsh(c0 - 0.89 * c).min() > -1e-9
    # (d1, d2, Vs, Vd) as in limit_blend
    d1, d2, Vs, Vd = np.eye(4)
    D, lap = d1 + d2, d2 - d1
    e = Vs - D
    c0 = 1.0813413108057222 * sq(lap) + 2.440625 * sq(e) \
        + sq(12.554318802466193 * lap + 6.254843361443233 * Vd) + sq(0.5 * D - 3 / 16 * e)
    for d in (d1, d2):
        assert np.linalg.eigvalsh(c0 - 0.80 * sq(d)).min() > -1e-9
