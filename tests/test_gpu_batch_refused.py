"""A run that is refused advances nothing: single steps left over by walking passes need the residency probe, which cannot
run inside a capture, and are asked for before the first pass is recorded."""
import pytest
import torch

from paper_2002_05265_amd import binding, inputs
from paper_2002_05265_amd.batch import Batch

pytestmark = pytest.mark.gpu


def test_walking_run_refused_under_capture(gpu):
    insts = [{"nx": 64, "ny": 64, "model": m, "eq_order": 4, "rho0": 1.0, "ux0": 0.0, "uy0": 0.0,
              "omega": list(inputs.rates(1e-2, "SRT"))} for m in ("K", "RR", "BGK")]
    stream = torch.cuda.Stream(gpu)
    b = Batch(insts, [inputs.vortex_fields(64, 64, 0.2)] * 3, device=gpu, stream=stream)
    b.set_pass(1)
    mark = torch.zeros(1, device=gpu)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        with pytest.raises(binding.LbmError) as e:
            b.run(4)  # a walking pass of three steps and a single step
        mark.fill_(1.0)
    assert e.value.code == -4 and b.status()[0] == 0
    before = b.state(0)
    g.replay()
    torch.cuda.synchronize()
    assert mark.item() == 1.0 and b.status()[0] == 0 and torch.equal(b.state(0), before)
    b.run(4)  # probed now
    assert b.status()[0] == 4
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=stream):
        b.run(4)
    for r in range(3):
        g.replay()
        torch.cuda.synchronize()
        assert b.status()[0] == 8 + 4 * r
    b.close()
