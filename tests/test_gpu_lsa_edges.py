"""The eigenvalue solver of the stability analysis where its rotations and convergence test degenerate: wave
numbers at which M(k) is real or has zero columns, rates that make moments vanish or leave them alone, a
resting flow, entries far apart in size.  Each returned eigenvalue must be one of a matrix close to M (backward
error): the smallest singular value of M - lambda is at most that of about 120 rotations (28 for the Hessenberg
form, and some 90 in two to three sweeps per eigenvalue) of three rounding errors each on both sides,
120 * 6 * 2.2e-16 = 1.6e-13 of the norm; and the eigenvalues add up to the trace within nine times that."""
import math

import numpy as np
import pytest
import torch

from paper_2002_05265_amd import inputs, lsa

pytestmark = pytest.mark.gpu

CX, CY = (0, 1, 0, -1, 0, 1, -1, -1, 1), (0, 0, 1, 0, -1, 1, 1, -1, -1)
K = np.array([0.0, math.pi, -math.pi, math.pi / 2, -math.pi / 2, 1e-9, 1e-160, 0.7, -2.9, 3.0])


@pytest.mark.parametrize("mach,phi", [(0.0, 0.0), (0.4, 0.0), (0.4, math.pi / 4), (1e-9, 1.0)])
@pytest.mark.parametrize("rates", [[0.0] * 5, [1.0] * 5, [2.0] * 5, [2.0, 1.0, 0.0, 1e-12, 1.0], [1.9, 1.9, 1.0, 1.0, 1.0]])
def test_backward_error(gpu, mach, phi, rates):
    kx, ky = (a.ravel() for a in np.meshgrid(K, K))
    phase = np.exp(-1j * (np.outer(kx, CX) + np.outer(ky, CY)))
    for model in inputs.MODEL_NAMES:
        pt = lsa.point(model, 0.0, mach, phi, omega=rates)
        J = lsa.jacobian(pt, gpu).cpu().numpy()
        M = phase[:, :, None] * J[None]
        x, y = (torch.from_numpy(a).to(gpu) for a in (kx, ky))
        lam = lsa.eigenvalues(pt, x, y).cpu().numpy()
        norm = np.linalg.norm(J)
        assert np.isfinite(lam).all(), model
        least = np.linalg.svd(M[:, None] - lam[:, :, None, None] * np.eye(9), compute_uv=False)[..., -1]
        assert least.max() <= 1.6e-13 * norm, (model, least.max() / norm)
        trace = np.abs(lam.sum(axis=1) - np.trace(M, axis1=1, axis2=2)).max()
        assert trace <= 9 * 1.6e-13 * norm, (model, trace / norm)
        r = lsa.radius([pt], x, y).cpu().numpy()[0]
        np.testing.assert_allclose(r, np.abs(lam).max(axis=1), rtol=4.5e-16)

