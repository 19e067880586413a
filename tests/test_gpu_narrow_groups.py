"""Groups of 256 threads, five a compute unit: both sides of the line where
many replications take them, equal to 1024-thread groups; and a burn whose
frontier is wider than their queues in LDS, equal to the oracle."""
import numpy as np
import pytest
import torch

from paper_1905_09317_amd import Request, Simulator

from _helpers import assert_same_outputs, oracle_run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sim():
    s = Simulator(0)
    yield s
    s.close()


def _landscape(rows, cols, seed):
    rng = np.random.default_rng(seed)
    fuel = rng.integers(0, 19, (rows, cols)).astype(np.uint8)
    elev = rng.integers(0, 120, (rows, cols)).astype(np.int16)
    wx = rng.uniform([90, 50, 5, 0], [96, 120, 45, 360], (2, 6, 4)).astype(np.float32)
    return fuel, elev, wx


@pytest.mark.parametrize("precision", [0, 1])
@pytest.mark.parametrize("shape,more,block", [((128, 128), 0, 256), ((129, 128), 0, 512), ((129, 128), 1, 256),
                                              ((512, 512), 1, 256), ((513, 512), 1, 512)])
def test_rule_for_many_replications(sim, shape, more, block, precision):
    fuel, elev, wx = _landscape(*shape, seed=shape[0])
    reps = 5 * torch.cuda.get_device_properties(0).multi_processor_count + more
    kw = dict(n_periods=6, reps=reps, seed=3, sigma=0.2, rounding=1, precision=precision,
              ignition_mode=1, scenario_mode=1, outputs=("scar", "burn_count", "burned_cells", "ignition_cell"))
    print(f"many replications: {shape}, {reps}, precision {precision}", flush=True)
    land, w = sim.load_landscape(fuel, elev), sim.set_weather(wx, period_min=60)
    try:
        a = sim.simulate(Request(landscape=land, weather=w, **kw))
        assert sim.stats()["block_threads"] == block
        sim.set_tuning(1024)
        b = sim.simulate(Request(landscape=land, weather=w, **kw))
        assert_same_outputs(a, b, where=f"{shape} {kw}")
    finally:
        sim.set_tuning(0)
        sim.unload_landscape(land)
        sim.unset_weather(w)


@pytest.mark.parametrize("shape,precision,block", [((64, 64), 0, 512), ((300, 200), 0, 1024), ((512, 513), 1, 1024),
                                                   ((1024, 1025), 0, 1024)])
def test_groups_held_back_by_scratch_are_wide(sim, shape, precision, block):
    fuel, elev, wx = _landscape(*shape, seed=shape[1])
    reps = 6 * torch.cuda.get_device_properties(0).multi_processor_count
    kw = dict(n_periods=3, reps=reps, seed=8, sigma=0.1, rounding=1, precision=precision, ignition_mode=1,
              scenario_mode=1, outputs=("burn_count", "burned_cells", "ignition_cell"), device_out=True)
    print(f"held back: {shape}, {reps}, precision {precision}", flush=True)
    land, w = sim.load_landscape(fuel, elev), sim.set_weather(wx, period_min=60)
    try:
        a = sim.simulate_noalloc(Request(landscape=land, weather=w, **kw))
        st = sim.stats()
        assert st["grid_blocks"] < reps and st["block_threads"] == block
        b = sim.simulate(Request(landscape=land, weather=w, **kw))
        torch.cuda.synchronize()
        for k in kw["outputs"]:
            assert torch.equal(a[k].cpu(), b[k].cpu()), k
    finally:
        sim.unload_landscape(land)
        sim.unset_weather(w)


@pytest.mark.parametrize("shape,reps,block", [((1024, 1024), 1, 1024), ((2047, 2048), 1, 1024), ((2048, 2048), 1, 512),
                                              ((2048, 2049), 2, 1024)])
def test_width_of_few_fp64_fires(sim, shape, reps, block):
    fuel, elev, wx = _landscape(*shape, seed=shape[1])
    kw = dict(n_periods=4, reps=reps, seed=11, sigma=0.1, rounding=1, ignition_mode=1)
    print(f"few fires: {shape}, {reps}", flush=True)
    land, w = sim.load_landscape(fuel, elev), sim.set_weather(wx, period_min=60)
    try:
        a = sim.simulate(Request(landscape=land, weather=w, **kw))
        assert sim.stats()["block_threads"] == block
        sim.set_tuning(1536 - block)   # the other width
        b = sim.simulate(Request(landscape=land, weather=w, **kw))
        assert_same_outputs(a, b, where=f"{shape} {reps}")
    finally:
        sim.set_tuning(0)
        sim.unload_landscape(land)
        sim.unset_weather(w)


@pytest.mark.parametrize("reps", [1, 256, 3000])
def test_launch_counters_sum_the_replications(sim, reps):
    fuel, elev, wx = _landscape(9, 8, seed=2)
    kw = dict(n_periods=4, reps=reps, seed=6, sigma=0.1, ignition_mode=1, scenario_mode=1)
    print(f"counters: {reps}", flush=True)
    land, w = sim.load_landscape(fuel, elev), sim.set_weather(wx, period_min=60)
    try:
        for _ in range(2):   # nothing is carried into the next launch
            r = sim.simulate(Request(landscape=land, weather=w, **kw))
            st = sim.stats()
            assert st["ignitions"] == int(np.asarray(r["burned_cells"]).sum())
            assert st["entries"] >= st["ignitions"] > 0 and st["continuations"] > 0 and st["rate_evals"] > 0
    finally:
        sim.unload_landscape(land)
        sim.unset_weather(w)


def test_frontier_wider_than_the_queue(sim):
    fuel = np.full((96, 96), 15, np.uint8)
    wx = np.tile(np.float32([96, 120, 30, 45]), (1, 4, 1))
    kw = dict(n_periods=4, reps=2, seed=5, ignition_mode=1)
    land, w = sim.load_landscape(fuel, None, cell_m=2), sim.set_weather(wx, period_min=60)
    sim.set_tuning(256)
    try:
        print(f"wide frontier: {kw}", flush=True)
        g = sim.simulate(Request(landscape=land, weather=w, **kw))
        assert np.asarray(g["burned_cells"]).max() > 4096
        assert_same_outputs(g, oracle_run(fuel, None, wx, period_min=60, cell_m=2, **kw))
    finally:
        sim.set_tuning(0)
        sim.unload_landscape(land)
        sim.unset_weather(w)
