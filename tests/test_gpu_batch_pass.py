"""Walking and resident passes of a batch (lbm_batch_set_pass) against persistent single-step passes: states,
step counters, blow-up steps and the means of |u|^2 are bit-identical for every live instance.  Widths that
are no multiple of a strip or of a lane's columns, below a strip and just above one, heights from the lowest
a walking pass takes, node counts at the edges of each resident size; step counts that take every split of a
run; instances that blow up, that are retired, tables dealt anew, and captured runs that are replayed."""
import numpy as np
import pytest
import torch

from paper_2002_05265_amd import binding, inputs
from paper_2002_05265_amd.batch import Batch

pytestmark = pytest.mark.gpu

WALK = [(64, 64), (2, 9), (128, 33), (129, 40), (225, 31), (112, 130), (34, 8), (300, 270), (448, 100), (96, 300)]
SMALL = [(32, 32), (31, 33), (2, 2), (3, 7), (16, 64), (5, 200), (1024 // 8, 8), (27, 27), (29, 30)]


def batch(gpu, sizes, prec, stable=True, seed=3, **kw):
    rng = np.random.default_rng(seed)
    insts, fields = [], []
    for k, (nx, ny) in enumerate(sizes):
        model = inputs.MODEL_NAMES[(k + seed) % 8]
        nu = 1e-2 if stable else 10 ** rng.uniform(-6, -3)
        mach = float(rng.uniform(0.1, 0.3) if stable else rng.uniform(0.4, 0.8))
        insts.append({"nx": nx, "ny": ny, "model": model, "eq_order": 4, "rho0": 1.0,
                      "ux0": 0.1 if prec != "f64" else 0.0, "uy0": 0.0,
                      "omega": list(inputs.rates(nu, "REG" if k % 2 else "SRT"))})
        fields.append(inputs.fourier_mode_fields(nx, ny, mach, np.random.default_rng(seed * 100 + k)))
    b = Batch(insts, fields, prec=prec, device=gpu, **kw)
    small = max(nx * ny for nx, ny in sizes) <= (2496 if prec == "f64" else 4096)
    assert b.passes() == (2 if small else 0, 0)
    b.set_pass(0)
    return b


def same(a, b, blown_too=False):
    (na, ba), (nb, bb) = a.status(), b.status()
    assert na == nb and ba == bb
    ua, ub = a.mean_u2(), b.mean_u2()
    for j in range(a.n):
        if ba[j] < 0 or blown_too:
            assert torch.equal(a.state(j).nan_to_num(9.0), b.state(j).nan_to_num(9.0)), (j, a.shapes[j])
        if ba[j] < 0:
            assert ua[j] == ub[j], j
    return sum(v >= 0 for v in ba)


@pytest.mark.parametrize("prec", ["f64", "f32", "f16"])
@pytest.mark.parametrize("seed", range(8))
def test_walking_passes(gpu, prec, seed):
    a, b = (batch(gpu, WALK, prec, seed=seed) for _ in range(2))
    b.set_pass(1)
    assert b.passes() == (1, 5 if prec == "f16" else 7)
    for n in (7, 5, 3, 23, 1, 2, 4, 8, 11):
        print(f"walking {prec} seed {seed}: {n} steps", flush=True)
        a.run(n)
        b.run(n)
        assert same(a, b) == 0


@pytest.mark.parametrize("prec,sizes", [(p, SMALL) for p in ("f64", "f32", "f16")] +
                         [(p, SMALL + [(45, 45), (64, 32)]) for p in ("f64", "f32", "f16")] +
                         [("f64", SMALL + [(48, 52), (40, 60)]), ("f32", SMALL + [(64, 64), (4, 1000)]),
                          ("f16", SMALL + [(64, 64), (2, 1500)])])
def test_resident_passes(gpu, prec, sizes):
    for seed in range(8):
        a, b = (batch(gpu, sizes, prec, seed=seed) for _ in range(2))
        b.set_pass(2)
        assert b.passes() == (2, 0)
        for n in (1, 2, 3, 12):
            print(f"resident {prec} seed {seed}: {n} steps", flush=True)
            a.run(n)
            b.run(n)
            assert same(a, b) == 0


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("kind", [1, 2])
def test_blow_up_and_retire(gpu, prec, kind):
    sizes = [(32, 32), (24, 40), (30, 34), (32, 20)] * 6
    a, b = (batch(gpu, sizes, prec, stable=False, seed=5) for _ in range(2))
    b.set_pass(kind)
    flags = torch.ones(a.n, dtype=torch.int32, device=gpu)
    flags[::5] = 0
    for k, n in enumerate((30, 61, 100, 200, 400)):
        for x in (a, b):
            x.run(n)
            if k == 1:
                x.set_active(flags)
            if k == 2:
                x.rebalance()
        blown = same(a, b, blown_too=kind == 2)
        print(f"kind {kind} {prec}: {blown} of {a.n} blown up", flush=True)
    assert 0 < blown < a.n


@pytest.mark.parametrize("kind,n", [(1, 14), (1, 8), (2, 9), (2, 10)])
def test_captured_passes(gpu, kind, n):
    sizes = [(32, 32), (64, 24), (40, 48)] * 5
    s = torch.cuda.Stream()
    a, b = batch(gpu, sizes, "f64"), batch(gpu, sizes, "f64", stream=s)
    b.set_pass(kind)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        b.run(n)
    assert b.status()[0] == 0  # capturing ran nothing
    for r in range(4):
        g.replay()
        a.run(n)
        s.synchronize()
        assert same(a, b) == 0
        if r == 1:
            b.rebalance()
    b.set_pass(0)
    a.run(3)
    b.run(3)
    assert same(a, b) == 0


def test_pass_settings(gpu):
    b = batch(gpu, [(32, 32), (40, 40)], "f64")
    for back in (lambda: b.set_fusion(0), lambda: b.set_fusion_depth(2), lambda: b.set_launch(2)):
        b.set_pass(2)
        back()
        assert b.passes() == (0, 0)
    b.autotune(2)
    assert b.passes()[0] in (0, 1, 2)
    with pytest.raises(binding.LbmError):
        b.set_pass(3)
    for sizes, kind in (([(32, 32), (111, 20)], 1), ([(127, 20)], 1), ([(32, 7)], 1), ([(50, 50)], 2)):
        c = batch(gpu, sizes, "f64")
        with pytest.raises(binding.LbmError):
            c.set_pass(kind)
        c.run(5)
        assert c.passes() == (0, 0) and c.status()[0] == 5
