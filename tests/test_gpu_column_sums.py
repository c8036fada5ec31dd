"""Sums of the waveform adjoint's partial rows: one row, lanes without a row, more
rows than lanes, against the oracle and bitwise the same again.

The bar is the waveform adjoint's, 1e-8 per component."""
import numpy as np
import pytest

from oracle import waveform
from paper_2204_06633_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 1024, 1025, 64 * 1024, 65 * 1024 + 3, 600_000])
def test_parameter_gradient_at_row_counts(n):
    import torch
    from paper_2204_06633_amd import native
    rng = np.random.default_rng(n)
    params = inputs.draw_gb_params(rng, 2)
    g = rng.standard_normal((2, 2, n))
    dev = lambda a: torch.tensor(a, dtype=torch.float64, device="cuda")
    run = lambda: native.gb_polarizations_adjoint(dev(params), 0, 10.0, dev(g[0]), dev(g[1]))
    got, again = run(), run()
    assert torch.equal(got, again)
    for k in range(2):
        t = 10.0 * np.arange(n)
        want = waveform.polarizations_vjp(params[k], t, g[0, k], g[1, k])
        close = np.abs(got[k].cpu().numpy() - want) <= 1e-8 * np.abs(want)
        assert close.all(), (k, got[k], want)
