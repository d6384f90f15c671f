"""Reverse steps on small grids, whose strips run all their rows side by side: two per launch against one per
launch, adjoint and rate gradients bit for bit, on grids below a strip, of one strip, of partial strips in
both directions and of the most strips that take this kernel, and just above."""
import numpy as np
import pytest
import torch

from paper_2002_05265_amd import binding as B
from paper_2002_05265_amd import inputs
from paper_2002_05265_amd.sim import Sim

pytestmark = pytest.mark.gpu

GRIDS = [(2, 2), (5, 3), (64, 8), (65, 9), (63, 17), (130, 70), (256, 256), (257, 330), (512, 512), (520, 512)]


@pytest.mark.parametrize("prec", ["f64", "f32", "f16"])
@pytest.mark.parametrize("nx,ny", GRIDS)
def test_pairs_equal_singles(gpu, prec, nx, ny):
    g = torch.Generator(device=gpu).manual_seed(nx + ny)
    rough = [a + 0.01 * torch.randn((ny, nx), generator=g, device=gpu, dtype=torch.float64)
             for a in (torch.ones((ny, nx), device=gpu, dtype=torch.float64), torch.zeros((ny, nx), device=gpu),
                       torch.zeros((ny, nx), device=gpu))]
    s = Sim(*rough, prec=prec, device=gpu, ref_velocity=(0.05, 0.01))
    kind = torch.float64 if prec == "f64" else torch.float32
    start = torch.randn(B.lbm_adjoint_bytes(s.ctx) // (8 if prec == "f64" else 4), generator=g, device=gpu, dtype=kind)
    n = 5
    states = [torch.empty(B.lbm_state_bytes(s.ctx), dtype=torch.uint8, device=gpu) for _ in range(n + 1)]
    B.lbm_save_state(s.ctx, states[0].data_ptr())
    ptr = [b.data_ptr() for b in states]
    for model in inputs.MODEL_NAMES if nx * ny < 20000 else inputs.MODEL_NAMES[nx % 3::3]:
        code, omega = inputs.MODEL_CODES[model], [1.9, 1.6, 1.3, 1.1, 0.9]
        B.lbm_step_raw_many(s.ctx, code, omega, ptr[:n], ptr[1:], 0)
        got = []
        for depth in (1, 2):
            B.lbm_set_adjoint_depth(s.ctx, depth)
            lam = [start.clone(), torch.zeros_like(start), torch.zeros_like(start)]
            dw = torch.zeros(5, dtype=torch.float64, device=gpu)
            print(f"reverse {prec} {model} {nx}x{ny} depth {depth}", flush=True)
            B.lbm_adjoint_many(s.ctx, code, omega, ptr[n - 1::-1], [lam[k % 3].data_ptr() for k in range(n + 1)],
                               dw.data_ptr())
            torch.cuda.synchronize()
            plane = start.numel() // 9
            got.append((lam[n % 3].view(9, plane)[:, :nx * ny], dw))
        assert torch.isfinite(got[0][0]).all() and torch.equal(got[0][0], got[1][0]), model
        assert torch.equal(got[0][1], got[1][1]), model
    s.close()
