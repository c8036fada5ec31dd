"""The fused batched forward over orbits whose positions lie further apart, or move
faster, than light times say: runs of the projection that the workgroup's stencil
bases do not cover.  Against the oracle, and the same bits however the batch is cut
(short runs at a tile's or a template's end are covered where full ones are not)."""
import dataclasses

import numpy as np
import pytest

import oracle
from paper_2204_06633_amd import inputs, workloads
from tests import cases

pytestmark = pytest.mark.gpu
SIZES = [1400, 31, 1023]


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch


@pytest.mark.parametrize("order,dt", [(7, 5.0), (25, 2.0), (25, 10.0), (31, 2.0)])
@pytest.mark.parametrize("kind", ["spread", "fast"])
def test_any_cut_gives_the_same_bits(torch_cuda, kind, order, dt):
    from paper_2204_06633_amd import native
    torch = torch_cuda
    grids, params, sp, st = workloads.make_batch(len(SIZES), "keplerian", SIZES, dt, order, 2, 7)
    t = sp.t0 + sp.dt * np.arange(sp.n)
    if kind == "spread":                 # positions four times as far apart as the light times
        m = sp.x.mean(axis=1, keepdims=True)
        x = m + 4.0 * (sp.x - m)
        more = int(60.0 / dt) + 4
    else:                                # hundreds of integer parts in a run
        x = sp.x + (0.3 * inputs.C_LIGHT) * (t - t[0])[:, None, None] * np.array([0.6, 0.8, 0.0])
        more = int(0.3 * (t[-1] - t[0]) / dt) + 64
    sp = dataclasses.replace(sp, x=x)
    for g in grids:
        g.front_proj += more
        g.back_proj += more
    lay = workloads.batch_layout(grids, 3)
    h = np.random.default_rng(order).standard_normal((2, lay.n_h_total))
    dev = lambda a: torch.tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")
    gp, gt = native.Orbits.from_samples(sp), native.Orbits.from_samples(st)
    outs = []
    for cut in ({}, dict(group=1), dict(group=4), dict(segment=3), dict(tile=256), dict(tile=1024)):
        b = native.Batch(lay.templates(), gp, gt, grids[0].t_start, dt, order, 2, "XYZ", **cut)
        out = b.response(dev(h[0]), dev(h[1]), dev(params[:, 6:8]))
        outs.append([b.output_block(out, k).cpu().numpy() for k in range(len(SIZES))])
        for k in range(len(SIZES)):
            assert np.array_equal(outs[-1][k], outs[0][k]), (cut, SIZES[k])
    op, ot = oracle.Orbits.from_samples(sp), oracle.Orbits.from_samples(st)
    for k, (g, ho, p) in enumerate(zip(grids, lay.h_offsets, params)):
        ref = oracle.response(op, ot, g, h[0, ho:ho + g.n_h], h[1, ho:ho + g.n_h], p[6], p[7],
                              order, 2, "XYZ")
        cases.check(outs[0][k], ref, 1e-11, "template %d" % k)
