"""How smooth an orbit handle's light times are, and what the batch plan makes of
it (CPU only): the filters with slowly varying taps follow light times that stay
within rounding of one cubic over a tile, and leave the others to the kernels that
interpolate delay by delay.  Whether a plan holds filters shows in its workspace,
which has room for their tables."""
import ctypes
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2204_06633_amd import inputs, native

T0 = 1e6


def _samples(kind, spacing):
    s = inputs.make_orbit_samples("keplerian", T0, T0 + 1e6, dt_orbit=spacing)
    t = s.t0 + s.dt * np.arange(s.n)
    ltt = s.ltt
    if kind == "fast":
        ltt = 8.3 + 1e-6 * (t - T0)[:, None] * np.array([1.0, -1.0, 0.5, 2.0, -0.7, 0.3]) / 10.0
    elif kind == "rough":
        ltt = ltt + 1e-9 * np.random.default_rng(3).standard_normal(ltt.shape)
    return dataclasses.replace(s, ltt=ltt)


@pytest.mark.parametrize("kind,spacing", [("keplerian", 1e4), ("keplerian", 1e3), ("fast", 1e4),
                                          ("rough", 1e4)])
def test_rate_and_jump_bound_the_splines(kind, spacing):
    s = _samples(kind, spacing)
    b = native.OrbitBounds.from_samples(s).c
    c = oracle.Orbits.from_samples(s).coef[9:15]           # [6][segment][4]
    u = np.linspace(0.0, s.dt, 33)
    rate = np.abs(c[..., 1:2] + u * (2.0 * c[..., 2:3] + 3.0 * u * c[..., 3:4])).max()
    assert rate <= b.L_rate <= 3.0 * rate
    # from coefficients whose own rounding is that of light times of 8 s
    jump = np.abs(np.diff(c[..., 3], axis=1)).max()
    assert abs(b.L_jump - jump) <= 64.0 * 2e-15 / s.dt ** 3


@pytest.mark.parametrize("kind", ["keplerian", "rigid"])
def test_distance_and_speed_bound_the_splines(kind):
    s = inputs.make_orbit_samples(kind, T0, T0 + 1e6)
    b = native.OrbitBounds.from_samples(s).c
    c = oracle.Orbits.from_samples(s).coef[:9].reshape(3, 3, -1, 4)    # [spacecraft][xyz]
    u = np.linspace(0.0, s.dt, 33)
    x = c[..., 0:1] + u * (c[..., 1:2] + u * (c[..., 2:3] + u * c[..., 3:4]))
    v = c[..., 1:2] + u * (2.0 * c[..., 2:3] + 3.0 * u * c[..., 3:4])
    apart = max(np.linalg.norm(x[i] - x[(i + 1) % 3], axis=0).max() for i in range(3))
    speed = np.linalg.norm(v, axis=1).max()
    assert apart <= b.D_max <= 1.05 * apart
    assert speed <= b.V_max <= 1.5 * speed


ROUTES = [("keplerian", 1e4, 5.0, True), ("keplerian", 1e4, 10.0, True),
          ("keplerian", 1e4, 15.0, True), ("keplerian", 3e3, 2.5, True),
          ("keplerian", 3e3, 10.0, False), ("keplerian", 1e3, 5.0, False),
          ("keplerian", 1e3, 10.0, False), ("keplerian", 1e2, 10.0, False),
          ("fast", 1e4, 10.0, False), ("rough", 1e4, 10.0, False)]


@pytest.mark.parametrize("kind,spacing,dt,filters", ROUTES)
def test_filters_only_for_smooth_light_times(kind, spacing, dt, filters):
    L = native._batch_lib()
    o = native.OrbitBounds.from_samples(_samples(kind, spacing))

    def ws(n_out):
        t = (native.lr_template * 1)(native.lr_template(0, n_out + 2000, 1000, n_out, 0))
        return L.lr_batch_workspace(t, 1, ctypes.byref(o.c), dt, 25, 2, native.CHANNELS["AET"],
                                    2, 512, 0, 0)

    per_output = (ws(512 * 400) - ws(512 * 200)) / (512 * 200)
    assert (per_output > 20.0) == filters and (filters or per_output < 2.0), per_output
