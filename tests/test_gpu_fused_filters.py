"""The fused batched forward's TDI filters against the oracle, where the
choice between a work item's shared filters and one-by-one delays can go
wrong: tile and interval edges, light times that cross or sit on an integer
number of samples or are too fast or too rough for one cubic per interval, and
non-finite samples.  How a batch is cut must not change a bit.

The bar is the forward's, 1e-11: a filter differs from the interpolations it
sums up by rounding alone.
"""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2204_06633_amd import inputs, workloads
from tests import cases

pytestmark = pytest.mark.gpu
T0, DT = 1e6, 10.0
SIZES = [1, 512, 0, 513, 1400, 31, 1023]


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch


def _batch(kind, order, gen):
    """Grids, parameters and orbit samples; the TDI light times are ``kind``."""
    grids, params, sp, st = workloads.make_batch(len(SIZES), "keplerian", SIZES, DT, order, gen, 7)
    t = st.t0 + st.dt * np.arange(st.n)
    per_link = np.array([1.0, -1.0, 0.5, 2.0, -0.7, 0.3])
    ltt = st.ltt.copy()
    if kind == "integer":
        ltt[:] = 10.0
    elif kind == "crossing":                    # 2 L and 4 L cross integers near 1.006e6 s
        ltt = 10.0 + 2e-8 * (t - T0 - 6e3)[:, None] * per_link
    elif kind == "fast":
        ltt = 8.3 + 1e-6 * (t - T0)[:, None] * per_link
    elif kind == "rough":                       # knots that one cubic cannot pass
        ltt = ltt + 1e-7 * np.random.default_rng(3).standard_normal(ltt.shape)
    for g in grids:                             # light times of up to 10.2 s
        g.front_tdi += 16
        g.back_tdi += 16
    return grids, params, sp, dataclasses.replace(st, ltt=ltt)


CASES = [("keplerian", g, o, None) for g in (1, 2) for o in (1, 7, 25, 31)]
CASES += [(k, 2, o, None) for k in ("integer", "crossing", "fast", "rough") for o in (3, 25)]
CASES += [("keplerian", 2, 25, float("nan")), ("crossing", 2, 25, float("inf"))]


@pytest.mark.parametrize("kind,gen,order,bad", CASES)
def test_fused_filters_match_oracle(torch_cuda, kind, gen, order, bad):
    from paper_2204_06633_amd import native
    torch = torch_cuda
    grids, params, sp, st = _batch(kind, order, gen)
    lay = workloads.batch_layout(grids, 3)
    h = np.zeros((2, lay.n_h_total))
    for g, ho, p in zip(grids, lay.h_offsets, params):
        h[:, ho:ho + g.n_h] = inputs.gb_polarizations(p, g.waveform_times())
    if bad is not None:                         # within the longest template, and near the end of another
        h[0, lay.h_offsets[4] + grids[4].n_h // 2] = bad
        h[1, lay.h_offsets[3] + grids[3].n_h - 60] = bad
    dev = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    gp, gt = native.Orbits.from_samples(sp), native.Orbits.from_samples(st)
    outs = []
    for group, segment in ((1, 0), (2, 0), (2, 2), (4, 0)):
        b = native.Batch(lay.templates(), gp, gt, T0, DT, order, gen, "XYZ", group=group,
                         segment=segment)
        out = b.response(dev(h[0]), dev(h[1]), dev(params[:, 6:8]))
        outs.append([b.output_block(out, k).cpu().numpy() for k in range(len(SIZES))])
    op, ot = oracle.Orbits.from_samples(sp), oracle.Orbits.from_samples(st)
    finite = True
    for k, (g, ho, p) in enumerate(zip(grids, lay.h_offsets, params)):
        if g.n_out == 0:
            continue
        ref = oracle.response(op, ot, g, h[0, ho:ho + g.n_h], h[1, ho:ho + g.n_h], p[6], p[7],
                              order, gen, "XYZ")
        ok = np.isfinite(ref)
        finite &= ok.all()
        for o in outs:
            assert np.array_equal(ok, np.isfinite(o[k])), (k, g.n_out)
            cases.check(o[k][ok], ref[ok], 1e-11, "template %d" % k)
            if bad is None:
                assert np.array_equal(o[k], outs[0][k]), (k, g.n_out)
    assert finite == (bad is None)


@pytest.mark.parametrize("tile", [256, 512])
@pytest.mark.parametrize("dt,order", [(0.4, 25), (0.7, 7), (1.0, 25), (1.5, 25), (2.5, 25)])
def test_fused_tiles_at_small_dt(torch_cuda, dt, order, tile):
    """Runs and tiles where the positions' spread and the TDI halo eat into them."""
    from paper_2204_06633_amd import native
    torch = torch_cuda
    n_out = [1, 700, 333]
    grids, params, sp, _ = workloads.make_batch(3, "keplerian", n_out, dt, order, 2, 11)
    lay = workloads.batch_layout(grids, 3)
    h = np.zeros((2, lay.n_h_total))
    for g, ho, p in zip(grids, lay.h_offsets, params):
        h[:, ho:ho + g.n_h] = inputs.gb_polarizations(p, g.waveform_times())
    dev = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    orb, ref = native.Orbits.from_samples(sp), oracle.Orbits.from_samples(sp)
    b = native.Batch(lay.templates(), orb, orb, grids[0].t_start, dt, order, 2, "XYZ", tile=tile)
    out = b.response(dev(h[0]), dev(h[1]), dev(params[:, 6:8]))
    for k, (g, ho, p) in enumerate(zip(grids, lay.h_offsets, params)):
        want = oracle.response(ref, ref, g, h[0, ho:ho + g.n_h], h[1, ho:ho + g.n_h], p[6], p[7],
                               order, 2, "XYZ")
        cases.check(b.output_block(out, k).cpu().numpy(), want, 1e-11, "template %d" % k)
