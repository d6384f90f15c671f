"""Batch.state called on a stream that is not the batch's: the result's memory may still be in use by work queued on the
caller's stream, which the copy out has to follow, and the caller may read the result at once."""
import pytest
import torch

from paper_2002_05265_amd import inputs
from paper_2002_05265_amd.batch import Batch

pytestmark = pytest.mark.gpu


def test_state_on_another_stream(gpu):
    insts = [{"nx": 256, "ny": 200, "model": m, "eq_order": 4, "rho0": 1.0, "ux0": 0.0, "uy0": 0.0,
              "omega": list(inputs.rates(1e-2, "SRT"))} for m in ("K", "RR")]
    own = torch.cuda.Stream(gpu)
    b = Batch(insts, [inputs.vortex_fields(256, 200, 0.2)] * 2, device=gpu, stream=own)
    b.run(6)
    own.synchronize()
    with torch.cuda.stream(own):
        want = [b.state(j).clone() for j in range(2)]
    own.synchronize()
    for turn in range(6):
        j = turn % 2
        busy = torch.empty((9, 200, 256), dtype=torch.float64, device=gpu)
        for k in range(400):  # some milliseconds of writes to the memory that the result will get
            busy.fill_(float(k))
        del busy
        f = b.state(j)
        assert torch.equal(f, want[j]), turn
        del f
    b.close()
