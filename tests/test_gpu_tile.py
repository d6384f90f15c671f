"""Tile launches (several steps of a patch in LDS, lbm_get_tile) against single steps: the same arithmetic
per node on values of the stored type, so states, step counters and blow-up steps are bit-identical.
Grids from four nodes to the largest with each patch, smaller than a patch, than a tile and than a halo, with
sides that are no multiple of a tile; step counts below, at and above a launch's; blow-ups in each step of a
launch, on tile edges; captured runs that are replayed."""
import numpy as np
import pytest
import torch

import oracle
from paper_2002_05265_amd import inputs
from paper_2002_05265_amd.sim import Sim

pytestmark = pytest.mark.gpu

MODELS = list(inputs.MODEL_NAMES) + ["STREAM_ONLY"]
GRIDS = [(2, 2), (2, 9), (7, 2), (5, 3), (33, 17), (64, 64), (150, 77), (400, 15), (333, 290), (511, 385),
         (640, 770), (1450, 40), (1000, 900)]


def rough(nx, ny, seed, device):
    """A vortex on a mean flow with 1% noise on every node."""
    rho, ux, uy = (torch.tensor(a, device=device) for a in inputs.vortex_fields(max(nx, 2), max(ny, 2), 0.2))
    g = torch.Generator(device=device).manual_seed(seed)
    return [(a + 0.01 * torch.randn(a.shape, generator=g, device=device, dtype=torch.float64))[:ny, :nx].contiguous()
            for a in (rho, ux, uy)]


@pytest.mark.parametrize("prec", ["f64", "f32", "f16"])
@pytest.mark.parametrize("nx,ny", GRIDS)
def test_tile_bit_identical(gpu, prec, nx, ny):
    rng = np.random.default_rng(nx + ny)
    fields = rough(nx, ny, nx + ny, gpu)
    ref = (0.2 * inputs.CS, 0.01)
    for k, model in enumerate(MODELS if nx * ny < 20000 else MODELS[(nx + ny) % 3::3]):
        omega = inputs.rates(1e-2, "REG") if k % 2 else np.array([1.8, *rng.uniform(0.6, 1.8, 4)])
        order = 2 + k % 3 if model in ("BGK", "RM", "HM", "PR", "RR") else 4
        a, b = (Sim(*fields, prec=prec, eq_order=order, device=gpu, ref_velocity=ref) for _ in range(2))
        a.set_fusion(model, 0)
        most, patch = b.tile(model)
        assert a.tile(model) == (0, 0) and b.walk(model) == (0, 0)
        assert patch in (22, 32, 44) and 3 <= most and patch - 2 * (most - 1) >= 4
        print(f"tile {prec} {model} {nx}x{ny} order {order} patch {patch} steps {most}", flush=True)
        total = 0
        for n in (2, most, 1, most + 1, 3 * most - 1):
            a.step(model, omega, n)
            b.step(model, omega, n)
            total += n
            assert a.status() == b.status() == (total, -1)
            assert torch.equal(a.state(), b.state()), n
        a.close()
        b.close()


@pytest.mark.parametrize("prec,nx,ny", [("f64", 64, 64), ("f32", 150, 77), ("f16", 90, 130), ("f64", 600, 520)])
def test_tile_blowup_step(gpu, prec, nx, ny):
    # zero rates: populations only stream.  f_3 = f_1 = -0.6 planted d nodes right and left of a node
    # meet there d steps later and make its density negative; nowhere before
    one, zero = np.ones((ny, nx)), np.zeros((ny, nx))
    f = torch.from_numpy(oracle.init_eq(4, one, zero, zero)).to(gpu)
    s = Sim(one, zero, zero, prec=prec, device=gpu)
    most, patch = s.tile("BGK")
    tw = patch - 2 * (most - 1)
    for ax, ay in ((0, 0), (nx - 1, ny - 1), (tw, tw - 1), (tw - 1, 2 * tw)):
        for d in range(1, most + 3):
            g = f.clone()
            g[3, ay, (ax + d) % nx] = g[1, ay, (ax - d) % nx] = -0.6
            s = Sim(one, zero, zero, prec=prec, device=gpu)
            s.set_state(g, 10)
            s.step("BGK", [0.0] * 5, 2 * most)
            assert s.status() == (10 + 2 * most, 10 + d), (ax, ay, d)
            s.close()


@pytest.mark.parametrize("prec,nx,ny,n", [("f64", 64, 64, 2), ("f64", 64, 64, 10), ("f32", 150, 77, 4),
                                          ("f32", 512, 512, 12), ("f16", 300, 300, 24)])
def test_tile_captured_run(gpu, prec, nx, ny, n):
    # an even number of strip launches: the captured run ends in the copy it starts from and can be
    # replayed to go on, with eager work between the replays
    omega = inputs.rates(1e-2, "REG")
    stream = torch.cuda.Stream(gpu)
    with torch.cuda.stream(stream):
        fields = rough(nx, ny, 5, gpu)
        a, b = (Sim(*fields, prec=prec, device=gpu) for _ in range(2))
        print(f"tile {prec} {nx}x{ny} captured run of {n}", flush=True)
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            b.step("K", omega, n)
        for r in range(4):
            a.step("K", omega, n)
            g.replay()
            assert torch.equal(a.state(), b.state()), r
    a.close()
    b.close()


def test_tile_settings(gpu):
    one, zero = np.ones((256, 256)), np.zeros((256, 256))
    s = Sim(one, zero, zero, prec="f64", device=gpu)
    first = s.tile("K")
    s.set_fusion("K", 8, 16)
    s.set_fusion_depth("RR", 3)
    assert s.tile("K") == s.tile("RR") == (0, 0) and s.tile("CM") == first
    s.autotune("K", inputs.rates(1e-2), 2)
    assert s.tile("K") in ((0, 0), first)
    s.close()
    # walking launches, too many nodes, too low for more than a patch per CU
    for prec, nx, ny in (("f64", 1030, 1030), ("f32", 2048, 2048), ("f64", 100, 50000), ("f32", 30000, 15)):
        t = Sim(np.ones((ny, nx)), np.zeros((ny, nx)), np.zeros((ny, nx)), prec=prec, device=gpu)
        assert t.tile("BGK") == (0, 0), (prec, nx, ny)
        t.close()
