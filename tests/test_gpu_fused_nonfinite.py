"""Non-finite samples in the fused batched forward and in the TDI filters: they
reach the outputs whose stencils read them, and change no bit elsewhere, however
the batch is cut into groups, tiles and segments."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2204_06633_amd import inputs, workloads

pytestmark = pytest.mark.gpu
DT = 10.0
SIZES = [1400, 600, 1023, 31, 2050]


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch


@pytest.mark.parametrize("gen,order", [(1, 25), (2, 3), (2, 25), (2, 31)])
@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_other_outputs_keep_their_bits(torch_cuda, gen, order, value):
    from paper_2204_06633_amd import native
    torch = torch_cuda
    grids, params, sp, st = workloads.make_batch(len(SIZES), "keplerian", SIZES, DT, order, gen, 7)
    lay = workloads.batch_layout(grids, 3)
    h = np.zeros((2, lay.n_h_total))
    for g, ho, p in zip(grids, lay.h_offsets, params):
        h[:, ho:ho + g.n_h] = inputs.gb_polarizations(p, g.waveform_times())
    bad = h.copy()
    hit = SIZES.index(2050)
    bad[0, lay.h_offsets[hit] + grids[hit].n_h // 2] = value
    dev = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    gp, gt = native.Orbits.from_samples(sp), native.Orbits.from_samples(st)
    sky = dev(params[:, 6:8])

    def run(h, **cut):
        b = native.Batch(lay.templates(), gp, gt, grids[0].t_start, DT, order, gen, "XYZ", **cut)
        out = b.response(dev(h[0]), dev(h[1]), sky)
        return [b.output_block(out, k).cpu().numpy() for k in range(len(SIZES))]

    clean = run(h)
    op, ot = oracle.Orbits.from_samples(sp), oracle.Orbits.from_samples(st)
    g, ho, p = grids[hit], lay.h_offsets[hit], params[hit]
    ok = np.isfinite(oracle.response(op, ot, g, bad[0, ho:ho + g.n_h], bad[1, ho:ho + g.n_h],
                                     p[6], p[7], order, gen, "XYZ"))
    assert 0 < (~ok).sum() < ok.size // 2
    for cut in ({}, dict(group=1), dict(group=4), dict(segment=3), dict(tile=256), dict(tile=1024),
                dict(group=1, tile=256, segment=2)):
        got = run(bad, **cut)
        for k in range(len(SIZES)):
            keep = ok if k == hit else np.ones_like(clean[k], dtype=bool)
            assert np.array_equal(np.isfinite(got[k]), keep), (cut, SIZES[k])
            assert np.array_equal(got[k][keep], clean[k][keep]), (cut, SIZES[k])


def test_whole_number_delays_read_their_whole_stencils(torch_cuda):
    """Where every delay is a whole number of samples, all weights but one are
    exactly zero: a non-finite sample still reaches every output whose stencil
    holds it, in TDI, its transpose and the fused batch.  Rounding decides on which
    side of the whole number a stencil lies; what both sides agree on is compared."""
    from paper_2204_06633_amd import native
    torch = torch_cuda
    order, gen, n_out, t0 = 7, 2, 700, 2e6 + 1000.0
    s = inputs.make_orbit_samples("keplerian", 2e6, 2.03e6)
    s = dataclasses.replace(s, ltt=np.full_like(s.ltt, 10.0))
    sides = [oracle.Orbits.from_samples(dataclasses.replace(s, ltt=s.ltt * (1.0 + e)))
             for e in (-1e-9, 1e-9)]
    orb = native.Orbits.from_samples(s)
    front, back = orb.tdi_padding(order, gen, DT)
    start, n_y = front + 1, front + 1 + n_out + back
    rng = np.random.default_rng(1)
    y, g = rng.standard_normal((6, n_y)), rng.standard_normal((3, n_out))
    y[2, start + 300] = np.nan
    g[1, 350] = np.inf
    dev = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    out = native.tdi_combine(orb, t0, DT, dev(y), gen, order, "XYZ", start, n_out).cpu().numpy()
    g_y = native.tdi_adjoint(orb, t0, DT, n_y, gen, order, "XYZ", start, dev(g)).cpu().numpy()
    p = np.arange(start, start + n_out)

    def agrees(got, oracles):
        a, b = [np.isfinite(o) for o in oracles]
        same = a == b
        assert (~a).any() and (~a & same).sum() > (~same).sum()
        assert np.array_equal(np.isfinite(got)[same], a[same])

    agrees(out, [oracle.tdi_xyz(o, t0, DT, y, gen, order, p) for o in sides])
    agrees(g_y, [oracle.tdi_adjoint(o, t0, DT, n_y, gen, order, p, g) for o in sides])

    grids, params, sp, _ = workloads.make_batch(2, "keplerian", [700, 333], DT, order, gen, 7,
                                                t_start=t0)
    for gr in grids:
        gr.front_tdi += 16
    lay = workloads.batch_layout(grids, 3)
    h = rng.standard_normal((2, lay.n_h_total))
    gr, ho, q = grids[0], lay.h_offsets[0], params[0]
    h[0, ho + gr.n_h // 2] = np.nan
    b = native.Batch(lay.templates(), native.Orbits.from_samples(sp), orb, t0, DT, order, gen, "XYZ")
    got = b.response(dev(h[0]), dev(h[1]), dev(params[:, 6:8]))
    op = oracle.Orbits.from_samples(sp)
    agrees(b.output_block(got, 0).cpu().numpy(),
           [oracle.response(op, o, gr, h[0, ho:ho + gr.n_h], h[1, ho:ho + gr.n_h], q[6], q[7],
                            order, gen, "XYZ") for o in sides])
    assert np.isfinite(b.output_block(got, 1).cpu().numpy()).all()
