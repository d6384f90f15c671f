"""The eigenvalue solver of the stability analysis takes matrices of any size whose products do not overflow: its shifts are
formed from values scaled to order one.  The growth rates of the discrete-velocity Boltzmann equation are homogeneous in
the wave number and the inverse relaxation time, so scaling both by a power of two scales the rates by it, within the
backward error of the solver (1e-12 of the largest rate)."""
import pytest
import torch

from paper_2002_05265_amd import lsa

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("power", [-400, -250, 250, 400])
def test_growth_scales(gpu, power):
    s = 2.0 ** power
    kx, ky = lsa.k_grid(12, gpu)
    pts = [lsa.point("BGK", 0.0, ma, 0.3, "SRT", order, omega=[1.0] * 5) for ma in (0.1, 0.5) for order in (2, 3, 4)]
    ref = lsa.dvbe_growth(pts, kx, ky, 1.0)
    got = lsa.dvbe_growth(pts, kx * s, ky * s, 1.0 / s) / s
    assert torch.isfinite(ref).all() and torch.isfinite(got).all()
    assert (got - ref).abs().max() <= 1e-12 * max(1.0, ref.abs().max().item())
