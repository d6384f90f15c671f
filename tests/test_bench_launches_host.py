"""The bench names the kernel that a context's launches are of, and what a tuned batch runs."""
import pytest

import bench


class Sim:
    def __init__(self, walk=(0, 0), tile=(0, 0), fusion=(0, 0), depth=2):
        self.settings = {"walk": walk, "tile": tile, "fusion": fusion, "fusion_depth": depth}

    def __getattr__(self, name):
        return lambda model: self.settings[name]


@pytest.mark.parametrize("sim,prec,steps,name", [
    (Sim(walk=(8, 76), fusion=(8, 32), depth=3), "f32", 8, "k_walk8"), (Sim(walk=(6, 12)), "f64", 6, "k_walk6"),
    (Sim(tile=(7, 44), fusion=(8, 8), depth=3), "f32", 7, "k_tile"), (Sim(tile=(3, 44)), "f16", 3, "k_tile"),
    (Sim(fusion=(8, 32), depth=3), "f32", 3, "k_step3"), (Sim(fusion=(8, 32), depth=3), "f64", 3, "k_step3n"),
    (Sim(fusion=(16, 16), depth=3), "f32", 2, "k_step2"), (Sim(fusion=(8, 40)), "f16", 2, "k_step2"),
    (Sim(), "f32", 1, "k_step")])
def test_kernel_names(sim, prec, steps, name):
    assert bench.launch_steps(sim, "K") == steps
    assert bench.step_kernel_name(sim, "K", prec) == name


class Batch:
    def __init__(self, passes, fusion=0, depth=2):
        self.passes, self.fusion, self.fusion_depth = (lambda: passes), (lambda: fusion), (lambda: depth)


@pytest.mark.parametrize("batch,name,npt,steps,rows", [
    (Batch((0, 0)), "persistent", 4, 1, 0), (Batch((0, 0), 64, 3), "persistent", 4, 3, 64),
    (Batch((1, 7), 64, 3), "walking", None, 7, None), (Batch((2, 0), 64, 3), "resident", None, None, None)])
def test_batch_launches(batch, name, npt, steps, rows):
    got = bench.batch_launches(batch, (4, 2, 11.0))
    assert (got["pass"], got["nodes_per_thread"], got["steps_per_pass"], got["strip_rows"]) == (name, npt, steps, rows)
