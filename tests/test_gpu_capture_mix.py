"""A graph captured on a context names the copy that held the state then.  Eager runs of the same context between
the replays must leave the state where the graph looks for it, as runs by strip launches always did: the number of
launches of a run has the parity that its strip launches would have."""
import pytest
import torch

import paper_2002_05265_amd.binding as B
from paper_2002_05265_amd import inputs
from paper_2002_05265_amd.sim import Sim

pytestmark = pytest.mark.gpu

OMEGA = inputs.rates(1e-2, "REG")
# (precision, nx, ny): walking launches, tile launches of every patch, strips alone
GRIDS = [("f32", 2130, 1900), ("f64", 1230, 1200), ("f16", 2131, 1901), ("f32", 512, 512), ("f64", 64, 64),
         ("f16", 300, 300)]


def pair(prec, nx, ny, gpu, stream):
    fields = [torch.tensor(a, device=gpu) for a in inputs.vortex_fields(nx, ny, 0.2)]
    return [Sim(*fields, prec=prec, device=gpu, stream=stream, ref_velocity=(0.1, 0.0)) for _ in range(2)]


def strip_launches(sim, model, n):
    ring, depth = sim.fusion(model)[0], sim.fusion_depth(model)
    per = 1 if not ring else (3 if ring in (4, 8) and depth == 3 else 2)
    return -(-n // per)


@pytest.mark.parametrize("prec,nx,ny", GRIDS)
def test_eager_runs_between_replays_of_a_run(gpu, prec, nx, ny):
    stream = torch.cuda.Stream(gpu)
    with torch.cuda.stream(stream):
        a, b = pair(prec, nx, ny, gpu, stream)
        for x in (a, b):
            x.step("K", OMEGA, 7)  # before the capture: any launches
        runs = [n for n in range(2, 24) if strip_launches(b, "K", n) % 2 == 0]
        n = runs[1]
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            b.step("K", OMEGA, n)
        for k in runs:
            g.replay()
            b.step("K", OMEGA, k)
            a.step("K", OMEGA, n)
            a.step("K", OMEGA, k)
            print(f"mix {prec} {nx}x{ny} captured {n}, then {k}", flush=True)
            g.replay()
            a.step("K", OMEGA, n)
            assert torch.equal(a.state(), b.state()), k
    a.close()
    b.close()


@pytest.mark.parametrize("prec,nx,ny", GRIDS[:1] + GRIDS[3:5])
@pytest.mark.parametrize("what", ["moments", "state", "save"])
def test_eager_runs_between_replays_of_a_read(gpu, prec, nx, ny, what):
    stream = torch.cuda.Stream(gpu)
    with torch.cuda.stream(stream):
        a, b = pair(prec, nx, ny, gpu, stream)
        runs = [n for n in range(2, 14) if strip_launches(b, "CM", n) % 2 == 0]
        if what == "moments":
            out = torch.zeros((3, ny, nx), dtype=torch.float64, device=gpu)
            read = lambda s: B.lbm_moments(s.ctx, *(t.data_ptr() for t in out), want_totals=False)
        elif what == "state":
            out = torch.zeros((9, ny, nx), dtype=torch.float64, device=gpu)
            read = lambda s: B.lbm_get_state(s.ctx, out.data_ptr())
        else:
            out = torch.zeros(B.lbm_state_bytes(b.ctx), dtype=torch.uint8, device=gpu)
            read = lambda s: B.lbm_save_state(s.ctx, out.data_ptr())
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=stream):
            read(b)
        for k in runs:
            a.step("CM", OMEGA, k)
            b.step("CM", OMEGA, k)
            print(f"mix {what} {prec} {nx}x{ny} after {k}", flush=True)
            g.replay()
            got = out.clone()
            read(a)
            assert torch.equal(got, out), k
    a.close()
    b.close()
