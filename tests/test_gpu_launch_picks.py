"""Where walking and tile launches lose against strip launches a new context does not take them: low and wide grids
in FP32 and FP16 (their waves or patches fill the device badly), and runs of two or three steps that one strip launch
takes in even rounds.  States are bit-identical to single steps whichever launches run; the picks are compared with
the strips' time (set_fusion_depth turns the others off), at most 12% slower where the launches left out were
20-38% slower and runs differ by 2%."""
import pytest
import torch

from paper_2002_05265_amd import inputs
from paper_2002_05265_amd.sim import Sim

pytestmark = pytest.mark.gpu


def sim(gpu, prec, nx, ny, model):
    g = torch.Generator(device=gpu).manual_seed(nx + ny)
    f = [0.02 * torch.randn((ny, nx), generator=g, device=gpu, dtype=torch.float64) for _ in range(3)]
    return Sim(1.0 + f[0], 0.05 + f[1], f[2], prec=prec, device=gpu, ref_velocity=(0.05, 0.0))


def us(s, model, n):
    omega = inputs.rates(1e-2, "SRT")
    best = float("inf")
    for _ in range(8):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        for _ in range(20):
            s.step(model, omega, n)
        e1.record()
        e1.synchronize()
        best = min(best, e0.elapsed_time(e1) * 50.0)
    return best


@pytest.mark.parametrize("prec,nx,ny,n", [("f32", 125000, 32, 12), ("f16", 125000, 32, 12), ("f16", 160000, 24, 12),
                                          ("f16", 160000, 20, 12), ("f32", 2048, 128, 2), ("f32", 2048, 128, 3),
                                          ("f64", 2048, 128, 2), ("f32", 768, 512, 3)])
def test_no_slower_than_strips(gpu, prec, nx, ny, n):
    s, t = sim(gpu, prec, nx, ny, "K"), sim(gpu, prec, nx, ny, "K")
    t.set_fusion("K", 0)
    s.step("K", inputs.rates(1e-2, "SRT"), n)
    t.step("K", inputs.rates(1e-2, "SRT"), n)
    assert torch.equal(s.state(), t.state()) and s.status() == t.status() == (n, -1)
    t.close()
    now = us(s, "K", n)
    s.set_fusion_depth("K", s.fusion_depth("K"))
    strips = us(s, "K", n)
    print(f"picks {prec} {nx}x{ny} {n} steps: {now:.1f} us, strips {strips:.1f}", flush=True)
    assert now < 1.12 * strips
    s.close()


@pytest.mark.parametrize("prec,nx,ny,model", [("f32", 16, 200000, "K"), ("f16", 32, 120000, "K"), ("f32", 60000, 16, "K"),
                                              ("f16", 60000, 16, "BGK"), ("f32", 83333, 48, "K"), ("f32", 125000, 32, "BGK"),
                                              ("f16", 160000, 20, "BGK"), ("f64", 120000, 32, "K")])
def test_taken_where_they_gain(gpu, prec, nx, ny, model):
    s = sim(gpu, prec, nx, ny, model)
    assert s.walk(model)[0] + s.tile(model)[0] > 0
    s.close()
