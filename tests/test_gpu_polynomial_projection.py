"""Projection, its adjoint and the sky gradient from polynomials per stencil base
against the oracle, where its runs can go wrong: one link sample, one more or
less than a run or a workgroup of them, both kinds of coefficient tables,
positions further apart than the light times or moving through many samples.

The polynomials replace the weights up to rounding (what they drop is below
2.5e-17 of the largest sample), so the bars are those of the other parity
tests: 1e-11 forward, 1e-10 for the transpose, 1e-6 for the gradient against Richardson
extrapolated differences.
"""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2204_06633_amd import inputs
from tests import cases

pytestmark = pytest.mark.gpu
T0 = 2e6


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch


def _orbits(kind):
    """Coarse orbit samples over [2e6, 2.1e6] s."""
    s = inputs.make_orbit_samples("keplerian", T0, T0 + 1e5)
    t = s.t0 + s.dt * np.arange(s.n)
    x = s.x.copy()
    if kind == "spread":                 # positions three times as far apart as the light times
        m = x.mean(axis=1, keepdims=True)
        x = m + 3.0 * (x - m)
    elif kind == "fast":                 # hundreds of integer parts in 256 link samples
        x = x + (0.3 * inputs.C_LIGHT) * (t - T0 - 1000.0)[:, None, None] * np.array([0.6, 0.8, 0.0])
    return dataclasses.replace(s, x=x)


SIZES = [(n, 25, 10.0, "keplerian") for n in (1, 252, 253, 256, 504, 505, 1100)]
SIZES += [(505, o, 10.0, "keplerian") for o in (1, 3, 13, 15, 17, 31)]
SIZES += [(700, 25, dt, "keplerian") for dt in (0.28, 0.5, 1.5)]
SIZES += [(600, o, 10.0, k) for k in ("spread", "fast") for o in (7, 25)]


@pytest.mark.parametrize("n_y,order,dt,kind", SIZES)
def test_polynomial_projection_adjoint(torch_cuda, n_y, order, dt, kind):
    from paper_2204_06633_amd import native
    torch = torch_cuda
    s = _orbits(kind)
    orb, ref = native.Orbits.from_samples(s), oracle.Orbits.from_samples(s)
    f, b = orb.projection_padding(order, dt)
    t0_h, n_h, start = T0 + 1000.0 - f * dt, f + n_y + b + 3, f + 1
    q = np.arange(start, start + n_y)
    rng = np.random.default_rng(n_y + order)
    g_y = rng.standard_normal((6, n_y))
    th = dt * np.arange(n_h)             # smooth over the stencils, so that orders agree
    hp, hc = np.cos(0.31 / dt * th + 0.4), np.sin(0.23 / dt * th + 1.0)
    lam, beta = 1.1, -0.4
    dev = lambda a: torch.tensor(a, dtype=torch.float64, device="cuda")
    ghp, ghc, g_sky = native.project_adjoint(orb, t0_h, dt, n_h, dev(hp), dev(hc),
                                             dev([lam, beta]), order, start, dev(g_y))
    only_p, only_c, _ = native.project_adjoint(orb, t0_h, dt, n_h, None, None, dev([lam, beta]),
                                               order, start, dev(g_y), want_sky=False)
    got = [a.cpu().numpy() for a in (ghp, ghc, only_p, only_c, g_sky)]
    want = np.stack(oracle.project_adjoint(ref, t0_h, dt, n_h, lam, beta, order, q, g_y))
    cases.check(np.stack(got[:2]), want, 1e-10)
    cases.check(np.stack(got[2:4]), want, 1e-10)

    def value(lam, beta):
        return np.sum(g_y * oracle.project_links(ref, t0_h, dt, hp, hc, lam, beta, order, q))

    def slope(i, step):
        d = [0.0, 0.0]
        d[i] = step
        return (value(lam + d[0], beta + d[1]) - value(lam - d[0], beta - d[1])) / (2.0 * step)

    # an interpolant of low order has kinks where a position crosses a sample
    if order >= 13:
        # in samples, so that the differences see the same phases at every dt
        step = 2e-3 * dt / (500.0 if kind != "fast" else 1e4)
        fd = [(4.0 * slope(i, step / 2) - slope(i, step)) / 3.0 for i in range(2)]
        cases.check(got[4], np.array(fd), 1e-6)


# 0.2 s: fewer link samples than bases; 0.05 s: every stencil from h
@pytest.mark.parametrize("n_y,order,dt,kind", SIZES + [(700, 25, 0.2, "keplerian"),
                                                       (300, 9, 0.05, "keplerian"),
                                                       (300, 25, 0.05, "keplerian")])
def test_polynomial_projection(torch_cuda, n_y, order, dt, kind):
    from paper_2204_06633_amd import native
    torch = torch_cuda
    s = _orbits(kind)
    orb, ref = native.Orbits.from_samples(s), oracle.Orbits.from_samples(s)
    f, b = orb.projection_padding(order, dt)
    t0_h, n_h, start = T0 + 1000.0 - f * dt, f + n_y + b + 3, f + 1
    h = np.random.default_rng(n_y + order).standard_normal((2, n_h))
    h[:, :2] = h[:, -2:] = np.nan        # padding that no stencil reaches
    lam, beta = 1.1, -0.4
    dev = lambda a: torch.tensor(a, dtype=torch.float64, device="cuda")
    y = native.project_links(orb, t0_h, dt, dev(h[0]), dev(h[1]), dev([lam, beta]), order, start,
                             n_y).cpu().numpy()
    ref = oracle.project_links(ref, t0_h, dt, h[0], h[1], lam, beta, order,
                               np.arange(start, start + n_y))
    assert np.array_equal(np.isfinite(ref), np.isfinite(y))
    ok = np.isfinite(ref)
    cases.check(y[ok], ref[ok], 1e-11)
