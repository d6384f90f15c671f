"""Chains of raw steps by tile and walking launches (lbm_step_raw_chain) against single raw steps, bit for bit,
whatever of the states is kept: none, all, one at each step of a launch, runs of three and four between kept
ones; and the gradients of all checkpoint schedules against the same run with one step per launch."""
import numpy as np
import pytest
import torch

from paper_2002_05265_amd import binding as B
from paper_2002_05265_amd import inputs
from paper_2002_05265_amd.adjoint import _Run
from paper_2002_05265_amd.sim import Sim

pytestmark = pytest.mark.gpu


def state(sim, buf):
    B.lbm_load_state(sim.ctx, buf.data_ptr(), 0)
    return sim.state()


@pytest.mark.parametrize("prec,nx,ny,kind", [("f64", 37, 50, "tile"), ("f32", 300, 200, "tile"), ("f16", 512, 500, "tile"),
                                             ("f64", 700, 640, "tile"), ("f64", 1100, 1000, "walk"),
                                             ("f32", 2131, 1901, "walk"), ("f16", 2131, 1901, "walk")])
def test_chain(gpu, prec, nx, ny, kind):
    fields = [torch.tensor(a, device=gpu) for a in inputs.vortex_fields(nx, ny, 0.2)]
    s = Sim(*fields, prec=prec, device=gpu, ref_velocity=(0.1, 0.0))
    code, omega = inputs.MODEL_CODES["CHM"], inputs.rates(1e-2, "REG")
    assert (s.tile(code)[0] > 0) == (kind == "tile") and (s.walk(code)[0] > 0) == (kind == "walk")
    n = 23
    bufs = [torch.empty(B.lbm_state_bytes(s.ctx), dtype=torch.uint8, device=gpu) for _ in range(n + 1)]
    B.lbm_save_state(s.ctx, bufs[0].data_ptr())
    ptr = [b.data_ptr() for b in bufs]
    B.lbm_step_raw_many(s.ctx, code, omega, ptr[:n], ptr[1:], 0)
    ref = [state(s, b) for b in bufs]
    out = [torch.empty_like(b) for b in bufs[1:]]
    hold = [torch.empty_like(bufs[0]) for _ in range(2)]
    tmp = [b.data_ptr() for b in hold]
    for kept in ([n - 1], list(range(n)), [0, n - 1], [1, 2, 9, n - 1], [3, 6, 10, 14, 19, n - 1], [9, 19, n - 1], [0]):
        count = kept[-1] + 1
        for b in out:
            b.fill_(255)
        dst = [out[k].data_ptr() if k in kept else None for k in range(count)]
        print(f"chain {prec} {nx}x{ny} kept {kept}", flush=True)
        moved = B.lbm_step_raw_chain(s.ctx, code, omega, ptr[0], dst, tmp if len(kept) < count else None, 0)
        assert len(kept) + 1 <= moved <= 3 * count
        for k in kept:
            assert torch.equal(state(s, out[k]), ref[k + 1]), (kept, k)
    assert B.lbm_step_raw_chain(s.ctx, code, omega, ptr[0], [], None, 0) == 0
    for dst, scratch in (([ptr[1], None], tmp), ([None, ptr[2]], None), ([None, ptr[0]], tmp), ([ptr[1], ptr[1]], tmp),
                         ([None, tmp[0]], tmp)):
        with pytest.raises(B.LbmError):
            B.lbm_step_raw_chain(s.ctx, code, omega, ptr[0], dst, scratch, 0)
    s.set_fusion("CHM", 0)
    with pytest.raises(B.LbmError):
        B.lbm_step_raw_chain(s.ctx, code, omega, ptr[0], [ptr[1]], None, 0)
    s.close()


@pytest.mark.parametrize("prec,n,steps", [("f64", 40, 31), ("f32", 200, 50)])
def test_gradients_of_chains(gpu, prec, n, steps):
    rho, ux, uy = inputs.vortex_fields(n, n, 0.2)
    _, tx, ty = inputs.vortex_fields(n, n, 0.1)
    u0, target = (torch.tensor(np.stack(a), device=gpu) for a in ((ux, uy), (tx, ty)))
    got = {}
    for schedule, slots in (("sqrt", 0), ("store_all", 0), ("revolve", 3), ("revolve", 1)):
        for single in (False, True):
            run = _Run(u0, [1.99, 1.7, 1.3, 1.1, 0.9], torch.tensor(rho, device=gpu), target, "K", steps, prec, 4, schedule,
                       slots, (0.1, 0.0))
            if single:
                B.lbm_set_fusion(run.ctx, inputs.MODEL_CODES["K"], 0, 0)
            assert run._long() == (not single)
            print(f"gradient {prec} {schedule} {slots} single {single}", flush=True)
            loss = run.forward()
            got[schedule, slots, single] = (loss, *run.backward())
            run.close()
    ref = got["sqrt", 0, True]
    for key, val in got.items():
        assert val[0] == ref[0] and torch.equal(val[1], ref[1]) and torch.equal(val[2], ref[2]), key
