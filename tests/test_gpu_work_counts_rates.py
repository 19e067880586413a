"""c2f_count_work where an FP32 rate would round to another integer than the
FP64 one (grass on a steep slope against the wind, a rate next to 17.5 m/min
that decides whether a neighbour 1415 m away is reached within 80 minutes):
the counts equal the oracle's."""
import numpy as np
import pytest

from paper_1905_09317_amd import Request, Simulator

from _helpers import assert_same_outputs, oracle_run

pytestmark = pytest.mark.gpu


def test_counts_take_fp64_rates():
    fuel = np.full((3, 3), 14, np.uint8)
    elev = np.zeros((3, 3), np.int16)
    elev[1, 2], elev[0, 1] = 2306, 1737
    kw = dict(n_periods=1, ignition_mode=0, ignition_cell=4)
    seen = set()
    with Simulator(0) as sim:
        land = sim.load_landscape(fuel, elev, cell_m=1000, curing=100.0)
        for ffmc in np.linspace(94.0425, 94.0445, 33).astype(np.float32):
            wx = np.float32([[[ffmc, 74.7782, 112.274, 412.4949]]])
            w = sim.set_weather(wx, period_min=80)
            req = Request(landscape=land, weather=w, outputs=("arrival_minute", "burned_cells"), device_out=True, **kw)
            g = sim.simulate(req)
            print(f"counts: {ffmc!r}", flush=True)
            got = sim.count_work(req, g["arrival_minute"])
            r = oracle_run(fuel, elev, wx, period_min=80, cell_m=1000, curing=100.0, **kw)
            assert_same_outputs({k: v.cpu().numpy() for k, v in g.items()}, r, ("arrival_minute", "burned_cells"))
            assert got == {"ignitions": int(r["stats"][0]), "burning_cell_periods": int(r["stats"][3]),
                           "axis_reaches": int(r["stats"][4])}, ffmc
            seen.add(got["axis_reaches"])
            sim.unset_weather(w)
    assert len(seen) > 1   # the rate decides
