"""A list capacity learnt from an overflow is remembered without the width of
the launch that overflowed: one held to few groups by the serving limit leaves
the width of an unrestricted call of the same shape, and the one written to the
tuning file, as the rule has them."""
import numpy as np
import pytest

from paper_1905_09317_amd import Request, Simulator

from _helpers import assert_same_outputs

pytestmark = pytest.mark.gpu

SIDE, REPS = 512, 600   # more replications than two a compute unit: 512 threads, 1024 in few groups


def _inputs(sim):
    # every cell burns within the first period: more queue entries than the
    # default capacity of so many replications holds
    fuel = np.full((SIDE, SIDE), 15, np.uint8)
    wx = np.tile(np.float32([96, 120, 30, 45]), (1, 1, 1))
    return sim.load_landscape(fuel, None, cell_m=1), sim.set_weather(wx, period_min=600)


def test_overflow_of_a_limited_launch_leaves_the_width(tmp_path):
    kw = dict(n_periods=1, reps=REPS, seed=3, ignition_mode=1, outputs=("burn_count", "burned_cells"))
    path = str(tmp_path / "tuning.txt")
    with Simulator(0) as sim:
        land, w = _inputs(sim)
        # another number of replications of the same class: the rule's width
        sim.simulate(Request(landscape=land, weather=w, **dict(kw, reps=REPS + 1)))
        want = sim.stats()["block_threads"]
        sim.set_serving(lanes=1, max_batch_grid=8)
        print(f"learnt width: {want} wanted, limited launch", flush=True)
        ticket, _ = sim.submit(Request(landscape=land, weather=w, **kw))
        a = sim.wait(ticket)
        sim.save_tuning(path)
        entry = [line.split() for line in open(path) if line.startswith(f"{SIDE * SIDE} {REPS} 0 ")]
        assert len(entry) == 1 and int(entry[0][4]) > 1 << 16, entry   # it overflowed and was remembered
        assert int(entry[0][3]) == want, entry
        print("learnt width: unrestricted call", flush=True)
        b = sim.simulate(Request(landscape=land, weather=w, **kw))
        st = sim.stats()
        assert st["relaunches"] == 0 and st["block_threads"] == want, st
        assert_same_outputs(a, b, names=kw["outputs"])
