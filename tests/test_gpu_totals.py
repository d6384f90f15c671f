"""The totals of lbm_moments come from a slot of host memory per context, and from a copy for the contexts
past the last slot: both give the same values, also after slots were given back and taken again."""
import numpy as np
import pytest

from paper_2002_05265_amd.sim import Sim

pytestmark = pytest.mark.gpu


def test_more_contexts_than_slots(gpu):
    one, zero = np.ones((6, 8)), np.zeros((6, 8))
    sims = [Sim(one * (1.0 + 0.01 * k), zero + 0.001 * k, zero, device=gpu) for k in range(70)]
    for turn in range(2):
        for k, s in enumerate(sims):
            tot = s.totals()
            rho, u = 1.0 + 0.01 * k, 0.001 * k
            np.testing.assert_allclose(tot[:5], [48 * rho, 48 * rho * u, 0.0, 24 * rho * u * u, u * u], rtol=1e-12, atol=1e-13)
        for k in range(5, 60):
            sims[k].close()
            sims[k] = Sim(one * (1.0 + 0.01 * k), zero + 0.001 * k, zero, device=gpu)
