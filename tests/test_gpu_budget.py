"""Device memory kept for the next launch is given back when an input or an
output needs it: under a budget that holds either, a landscape and a weather
table load after a launch of many replications, and a call with large outputs
runs after it."""
import numpy as np
import pytest

from paper_1905_09317_amd import Request, Simulator

from _helpers import assert_same_outputs

pytestmark = pytest.mark.gpu

MB = 1 << 20


def _many(sim):
    """A launch of 1500 small fires and its request."""
    fuel = np.random.default_rng(3).integers(1, 19, (64, 64)).astype(np.uint8)
    wx = np.tile(np.float32([92, 80, 20, 100]), (1, 6, 1))
    req = Request(landscape=sim.load_landscape(fuel), weather=sim.set_weather(wx), n_periods=6, reps=1500, seed=2,
                  ignition_mode=1, outputs=("burn_count", "burned_cells"))
    return req, sim.simulate(req)


@pytest.mark.parametrize("what", ["landscape", "weather", "outputs", "rates"])
def test_kept_buffers_make_room(what):
    with Simulator(0, hbm_budget_bytes=1000 * MB) as sim:
        req, first = _many(sim)
        held = sim.memory()[0]
        print(f"budget: {what}, {held >> 20} MB held", flush=True)
        assert held < 1000 * MB
        if what == "landscape":
            sim.load_landscape(np.full((3000, 3000), 2, np.uint8), np.zeros((3000, 3000), np.int16))
        elif what == "weather":
            sim.set_weather(np.tile(np.float32([92, 80, 20, 100]), (1000, 500, 1)))
        elif what == "outputs":
            fuel = np.random.default_rng(4).integers(1, 19, (200, 200)).astype(np.uint8)
            kw = dict(n_periods=2, reps=700, seed=5, ignition_mode=1,
                      outputs=("scar", "arrival_minute", "arrival_period", "burn_count"))
            out = sim.simulate(Request(landscape=sim.load_landscape(fuel), weather=req.weather, **kw))
            with Simulator(0) as other:
                wx = other.set_weather(np.tile(np.float32([92, 80, 20, 100]), (1, 6, 1)))
                ref = other.simulate(Request(landscape=other.load_landscape(fuel), weather=wx, **kw))
            assert_same_outputs(out, ref, names=kw["outputs"], where=what)
        else:
            big = sim.load_landscape(np.full((1200, 1200), 2, np.uint8))
            sim.eval_ros(big, req.weather)
        assert sim.memory()[0] <= 1000 * MB
        assert_same_outputs(sim.simulate(req), first, names=req.outputs, where=what)
