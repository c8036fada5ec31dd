"""TDI as filters with slowly varying taps (forward and transpose) against the
oracle, where its intervals can go wrong: tile edges, delays that cross an
integer or sit on one, light times too fast or too rough for one interval per
tile, and non-finite samples.

The filters replace the interpolations up to rounding (a cubic in time whose
error is below 1e-16 of the series), so the bars are those of the other
parity tests: 1e-11 forward, 1e-10 transpose.
"""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2204_06633_amd import inputs
from tests import cases

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch


def _orbits(kind):
    """Coarse orbit samples over [2e6, 2.1e6] s."""
    s = inputs.make_orbit_samples("keplerian", 2e6, 2.1e6)
    t = s.t0 + s.dt * np.arange(s.n)
    ltt = s.ltt.copy()
    if kind == "integer":                       # every delay a whole number of samples
        ltt[:] = 10.0
    elif kind == "crossing":                    # 2 L and 4 L cross integers near 2.004e6 s
        ltt = 10.0 + 2e-8 * (t - 2.004e6)[:, None] * np.array([1.0, -1.0, 0.5, 2.0, -0.7, 0.0])
    elif kind == "fast":                        # tens of pieces in a tile
        ltt = 8.3 + 1e-6 * (t - 2e6)[:, None] * np.array([1.0, -1.0, 0.5, 2.0, -0.7, 0.3])
    elif kind == "rough":                       # knots that one cubic cannot pass
        ltt = ltt + 1e-7 * np.random.default_rng(3).standard_normal(ltt.shape)
    return dataclasses.replace(s, ltt=ltt)


def _setup(torch, kind, gen, order, n_out, dt):
    from paper_2204_06633_amd import native
    s = _orbits(kind)
    orb = native.Orbits.from_samples(s)
    ft, bt = orb.tdi_padding(order, gen, dt)
    return s, orb, ft + 1, ft + n_out + bt + 4, 2e6 + 1000.0


CASES = [("keplerian", g, o, n, dt) for g in (1, 2) for o in (1, 7, 25, 31)
         for n, dt in ((1, 10.0), (512, 10.0), (1537, 5.0))]
CASES += [(k, 2, o, 1400, 10.0) for k in ("integer", "crossing", "fast", "rough") for o in (3, 25)]
CASES += [("crossing", 1, 25, 700, 10.0), ("keplerian", 2, 25, 513, 1.5)]


@pytest.mark.parametrize("kind,gen,order,n_out,dt", CASES)
def test_filters_match_oracle(torch_cuda, kind, gen, order, n_out, dt):
    from paper_2204_06633_amd import native
    torch = torch_cuda
    s, orb, start, n_y, t0 = _setup(torch, kind, gen, order, n_out, dt)
    rng = np.random.default_rng(order + n_out)
    y, g = rng.standard_normal((6, n_y)), rng.standard_normal((3, n_out))
    dev = lambda a: torch.tensor(a, dtype=torch.float64, device="cuda")
    out = native.tdi_combine(orb, t0, dt, dev(y), gen, order, "XYZ", start, n_out)
    g_y = native.tdi_adjoint(orb, t0, dt, n_y, gen, order, "XYZ", start, dev(g))
    torch.cuda.synchronize()
    o = oracle.Orbits.from_samples(s)
    p = np.arange(start, start + n_out)
    cases.check(out.cpu().numpy(), oracle.tdi_xyz(o, t0, dt, y, gen, order, p), 1e-11)
    cases.check(g_y.cpu().numpy(), oracle.tdi_adjoint(o, t0, dt, n_y, gen, order, p, g), 1e-10)


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_a_non_finite_sample_stays_in_its_stencils(torch_cuda, value):
    from paper_2204_06633_amd import native
    torch = torch_cuda
    gen, order, n_out, dt = 2, 25, 1100, 10.0
    s, orb, start, n_y, t0 = _setup(torch, "keplerian", gen, order, n_out, dt)
    rng = np.random.default_rng(5)
    y, g = rng.standard_normal((6, n_y)), rng.standard_normal((3, n_out))
    y[4, start + 200] = y[0, start + 900] = value
    g[1, 300] = value
    dev = lambda a: torch.tensor(a, dtype=torch.float64, device="cuda")
    out = native.tdi_combine(orb, t0, dt, dev(y), gen, order, "XYZ", start, n_out).cpu().numpy()
    g_y = native.tdi_adjoint(orb, t0, dt, n_y, gen, order, "XYZ", start, dev(g)).cpu().numpy()
    o = oracle.Orbits.from_samples(s)
    p = np.arange(start, start + n_out)
    for got, ref, tol in ((out, oracle.tdi_xyz(o, t0, dt, y, gen, order, p), 1e-11),
                          (g_y, oracle.tdi_adjoint(o, t0, dt, n_y, gen, order, p, g), 1e-10)):
        ok = np.isfinite(ref)
        assert np.array_equal(ok, np.isfinite(got)) and not ok.all()
        cases.check(got[ok], ref[ok], tol)
