"""Four lanes a cell: the propagation where chunks of 16 cells are partly
filled, at every block size and with every option that reads all axes of a
cell, against the oracle (bit-exact); and the quad's FP32 rates against one
thread's, bit for bit."""
import sys

import numpy as np
import pytest

from paper_1905_09317_amd import Request, Simulator, inputs

from _helpers import assert_same_outputs, oracle_run

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def sim():
    s = Simulator(0)
    yield s
    s.close()


@pytest.mark.parametrize("block", [64, 256, 512, 1024])
@pytest.mark.parametrize("shape", [(1, 1), (1, 17), (4, 4), (16, 3), (13, 5), (65, 31)])
def test_partly_filled_chunks_equal_the_oracle(sim, shape, block):
    rows, cols = shape
    rng = np.random.default_rng(100 * rows + cols)
    fuel = rng.integers(0 if rows * cols > 40 else 1, 19, shape).astype(np.uint8)
    elev = rng.integers(0, 120, shape).astype(np.int16)
    wx = rng.uniform([88, 40, 5, 0], [96, 120, 45, 360], (2, 9, 4)).astype(np.float32)
    land, w = sim.load_landscape(fuel, elev), sim.set_weather(wx, period_min=30)
    sim.set_tuning(block)
    try:
        for sigma, rounding, threshold, burnout, hfi in ((0.0, 0, 0.0, 0.0, 0.0), (0.3, 1, 0.0, 0.0, 300.0),
                                                         (0.15, 0, 2.0, 3.0, 0.0)):
            kw = dict(n_periods=9, reps=3, seed=17, sigma=sigma, rounding=rounding, threshold=threshold,
                      burnout=burnout, hfi_min=hfi, ignition_mode=1, scenario_mode=1)
            _say(f"quads: {rows}x{cols}, block {block}, {kw}")
            g = sim.simulate(Request(landscape=land, weather=w, **kw))
            assert_same_outputs(g, oracle_run(fuel, elev, wx, period_min=30, **kw), where=f"{shape} {block} {kw}")
    finally:
        sim.set_tuning(0)
        sim.unload_landscape(land)
        sim.unset_weather(w)


@pytest.mark.parametrize("n", [1, 63, 64, 65, 70001])
def test_quad_rates_equal_one_thread_rates_in_fp32(sim, n):
    """Rounding 0: q = floor(x + 1/2) in FP32 of the rates the same call reports."""
    rng = np.random.default_rng(n)
    fuel = rng.integers(1, 19, (1, n)).astype(np.uint8)
    elev = inputs.elevation_grid(1, n, 3, elev_max=900.0) if n > 1 else None
    land = sim.load_landscape(fuel, elev, cell_m=60, pc=30.0, curing=65.0)
    sim.set_landscape_fbp(land, fmc=110.0, pdf=35.0)
    wx = np.array([[[90, 60, 12, 10], [96, 140, 40, 200], [86, 20, 0.9, 300], [98, 200, 70, 120]]], np.float32)
    w = sim.set_weather(wx)
    for p in range(4):
        for sigma in (0.0, 0.3):
            _say(f"quad rates: {n} cells, period {p}, sigma {sigma}")
            o = sim.eval_ros(land, w, period=p, rep=5, seed=11, sigma=sigma, precision=1)
            want = np.floor(o["x8"].astype(np.float32) + np.float32(0.5)).astype(np.int64)
            assert np.array_equal(o["q8"], want), (n, p, sigma)
    sim.unload_landscape(land)
    sim.unset_weather(w)
