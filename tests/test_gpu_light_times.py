"""TDI calls over light times of every smoothness against the oracle: orbits sampled
so densely that rounding shows at the splines' knots, fast and rough ones (which
filters with slowly varying taps do not follow), and delays that cross an integer
number of samples, at many outputs of one tile and close together.

Forward 1e-11, transpose 1e-10: the bars of the other parity tests, since which
kernel serves a call changes a result by rounding alone.
"""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2204_06633_amd import inputs, workloads
from tests import cases

pytestmark = pytest.mark.gpu
T0, DT, ORDER = 2e6, 10.0, 25


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch


def _light_times(s, kind, t_mark):
    """Orbit samples with light times of a kind; t_mark: a time among the outputs."""
    t = s.t0 + s.dt * np.arange(s.n)
    per_link = np.array([1.0, -1.0, 0.5, 2.0, -0.7, 0.3])
    ltt = s.ltt.copy()
    if kind.startswith("crossing"):             # links cross 10 s this many outputs apart
        apart = float(kind[8:])
        at = t_mark + DT * (0.5 + apart * np.arange(6))
        ltt = 10.0 + 2e-8 * (t[:, None] - at) * np.sign(per_link)
    elif kind == "fast":
        ltt = 8.3 + 1e-6 * (t - T0)[:, None] * per_link
    elif kind == "rough":
        ltt = ltt + 1e-7 * np.random.default_rng(3).standard_normal(ltt.shape)
    return dataclasses.replace(s, ltt=ltt)


KINDS = [(kind, 1e4) for kind in ("crossing0", "crossing1.3", "crossing3.7", "crossing90", "fast",
                                  "rough")] + [("keplerian", h) for h in (100.0, 1000.0, 3000.0)]


@pytest.mark.parametrize("gen", [1, 2])
@pytest.mark.parametrize("kind,spacing", KINDS)
def test_tdi_and_its_transpose(torch_cuda, kind, spacing, gen):
    from paper_2204_06633_amd import native
    torch = torch_cuda
    n_out, t0 = 1400, T0 + 1000.0
    s = inputs.make_orbit_samples("keplerian", T0, T0 + 3e4, dt_orbit=spacing)
    start = 60
    s = _light_times(s, kind, t0 + DT * (start + 200))
    orb, ref = native.Orbits.from_samples(s), oracle.Orbits.from_samples(s)
    front, back = orb.tdi_padding(ORDER, gen, DT)
    assert front <= start
    n_y = start + n_out + back + 4
    rng = np.random.default_rng(gen)
    y, g = rng.standard_normal((6, n_y)), rng.standard_normal((3, n_out))
    dev = lambda a: torch.tensor(a, dtype=torch.float64, device="cuda")
    out = native.tdi_combine(orb, t0, DT, dev(y), gen, ORDER, "XYZ", start, n_out)
    g_y = native.tdi_adjoint(orb, t0, DT, n_y, gen, ORDER, "XYZ", start, dev(g))
    again = native.tdi_adjoint(orb, t0, DT, n_y, gen, ORDER, "XYZ", start, dev(g))
    assert torch.equal(g_y, again)
    p = np.arange(start, start + n_out)
    cases.check(out.cpu().numpy(), oracle.tdi_xyz(ref, t0, DT, y, gen, ORDER, p), 1e-11)
    cases.check(g_y.cpu().numpy(), oracle.tdi_adjoint(ref, t0, DT, n_y, gen, ORDER, p, g), 1e-10)


# pairs of templates by duration: (1400, 1023), (513, 512), (31, nothing); the second
# of a pair ends within a tile, and within a piece of one
SIZES = [512, 1400, 31, 0, 1023, 513]


@pytest.mark.parametrize("bad", [None, float("nan"), float("inf")])
@pytest.mark.parametrize("kind,spacing", [k for k in KINDS if k[1] != 100.0])
def test_batched_transpose(torch_cuda, kind, spacing, bad):
    """lr_response_adjoint of uneven pairs; a gradient that is not finite stays
    within its template's stencils."""
    from paper_2204_06633_amd import native
    torch = torch_cuda
    grids, params, _, _ = workloads.make_batch(len(SIZES), "keplerian", SIZES, DT, ORDER, 2, 7)
    for g in grids:                             # light times of up to 10.2 s
        g.front_tdi += 16
        g.back_tdi += 16
    t_start = grids[0].t_start
    lo = min(g.t0_h for g in grids)
    sp = inputs.make_orbit_samples("keplerian", lo, lo + DT * max(g.n_h for g in grids))
    st = inputs.make_orbit_samples("keplerian", t_start, t_start + 3e4, dt_orbit=spacing)
    st = _light_times(st, kind, t_start + DT * 200)
    lay = workloads.batch_layout(grids, 3)
    gp, gt = native.Orbits.from_samples(sp), native.Orbits.from_samples(st)
    op, ot = oracle.Orbits.from_samples(sp), oracle.Orbits.from_samples(st)
    b = native.Batch(lay.templates(), gp, gt, t_start, DT, ORDER, 2, "XYZ", adjoint=True)
    g_out = np.random.default_rng(5).standard_normal(b.out_extent)
    if bad is not None:                         # in the longest template, which has a partner
        k = SIZES.index(1400)
        g_out[lay.out_offsets[k] + 1400 + 300] = bad
    dev = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    sky = dev(params[:, 6:8])
    ghp, ghc, _ = b.adjoint(None, None, sky, dev(g_out), want_sky=False)
    got = np.stack([ghp.cpu().numpy(), ghc.cpu().numpy()])
    for k, (g, n, ho, oo) in enumerate(zip(grids, SIZES, lay.h_offsets, lay.out_offsets)):
        if n == 0:
            continue
        ref = np.stack(oracle.response_adjoint(op, ot, g, params[k][6], params[k][7], ORDER, 2,
                                               g_out[oo:oo + 3 * n].reshape(3, n), "XYZ"))
        mine = got[:, ho:ho + g.n_h]
        ok = np.isfinite(ref)
        assert np.array_equal(ok, np.isfinite(mine)), (k, n)
        assert ok.all() == (bad is None or n != 1400)
        cases.check(mine[ok], ref[ok], 1e-10, "template %d" % k)


@pytest.mark.parametrize("apart", [1.3, 40.0])
def test_crossings_cost_little(torch_cuda, apart):
    """A short template in which delays cross integers takes a few times as long as
    one in which none does, at most: it is one tile's work in some more pieces."""
    from paper_2204_06633_amd import native
    torch = torch_cuda
    n_out, t0, start = 1400, T0 + 1000.0, 60
    s = inputs.make_orbit_samples("keplerian", T0, T0 + 3e4)
    times = []
    for sample in (s, _light_times(s, "crossing%g" % apart, t0 + DT * (start + 200))):
        orb = native.Orbits.from_samples(sample)
        n_y = start + n_out + orb.tdi_padding(ORDER, 2, DT)[1] + 4
        y = torch.zeros((6, n_y), dtype=torch.float64, device="cuda")
        out = torch.zeros((3, n_out), dtype=torch.float64, device="cuda")
        best = [1e9, 1e9]
        for _ in range(12):
            for i, call in enumerate((
                    lambda: native.tdi_combine(orb, t0, DT, y, 2, ORDER, "XYZ", start, n_out, out=out),
                    lambda: native.tdi_adjoint(orb, t0, DT, n_y, 2, ORDER, "XYZ", start, out, g_y=y))):
                a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
                a.record()
                call()
                b.record()
                b.synchronize()
                best[i] = min(best[i], a.elapsed_time(b))
        times.append(best)
    assert times[1][0] < 12.0 * times[0][0] and times[1][1] < 12.0 * times[0][1], times
