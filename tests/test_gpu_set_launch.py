"""An explicit launch shape takes the model's steps, as it did before there were walking and tile launches: lbm_set_launch
turns these off for its model and leaves the other models' and the fused setting alone."""
import pytest
import torch

from paper_2002_05265_amd import inputs
from paper_2002_05265_amd.sim import Sim

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,n,kind", [("f64", 64, "tile"), ("f32", 600, "tile"), ("f64", 1100, "walk")])
def test_shape_takes_the_steps(gpu, prec, n, kind):
    fields = [torch.tensor(a, device=gpu) for a in inputs.vortex_fields(n, n, 0.2)]
    a, b = (Sim(*fields, prec=prec, device=gpu) for _ in range(2))
    first = getattr(a, kind)("RR")
    assert first[0] > 0
    fused = a.fusion("RR"), a.fusion_depth("RR")
    for rows, xcd in ((2, 1), (1, 0)):
        a.set_launch("RR", rows, xcd)
        assert a.walk("RR") == a.tile("RR") == (0, 0)
        assert (a.fusion("RR"), a.fusion_depth("RR")) == fused
        assert getattr(a, kind)("K") == first
        for s in (a, b):
            s.step("RR", inputs.rates(1e-2, "REG"), 7)
        assert torch.equal(a.state(), b.state())
    a.close()
    b.close()
