"""The scheme is homogeneous of degree one in the populations, and a factor that is a power of two changes no rounding: FP64
runs from densities near both ends of the range (two steps of Newton on the hardware's reciprocal there, as
anywhere) are the run from density one times the factor, bit for bit.  Products of two deviations (K) leave a
smaller range of factors."""
import pytest
import torch

from paper_2002_05265_amd import inputs
from paper_2002_05265_amd.sim import Sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [40, 300, 1100])
@pytest.mark.parametrize("power", [-900, -300, 300, 900])
def test_scaled_density(gpu, n, power):
    rho, ux, uy = (torch.tensor(a, device=gpu) for a in inputs.vortex_fields(n, n, 0.3))
    s = 2.0 ** power
    for model in inputs.MODEL_NAMES:
        if model == "K" and abs(power) > 400:
            continue
        a, b = Sim(rho, ux, uy, device=gpu), Sim(rho * s, ux, uy, device=gpu)
        for n_steps in (1, 9):
            a.step(model, inputs.rates(1e-3, "REG"), n_steps)
            b.step(model, inputs.rates(1e-3, "REG"), n_steps)
        assert torch.equal(a.state() * s, b.state()), model
        assert a.status() == b.status() == (10, -1)
        a.close()
        b.close()
