"""Work lists of a no-allocation call grow into all of the scratch that one
slot leaves: fires whose lists need more than a quarter step but whose next full
step does not fit beside the plane."""
import numpy as np
import pytest
import torch

from paper_1905_09317_amd import Request, Simulator

pytestmark = pytest.mark.gpu


def test_lists_take_the_room_that_is_left():
    side = 5700   # a plane of 130 MB in the 128 MiB scratch
    with Simulator(0) as sim:
        land = sim.load_landscape(np.full((side, side), 2, np.uint8), None, cell_m=10)
        for minutes in (150, 160, 175):
            print(f"noalloc room: one period of {minutes} minutes", flush=True)
            w = sim.set_weather(np.float32([[[92, 80, 8, 60]]]), period_min=minutes)
            req = Request(landscape=land, weather=w, n_periods=1, ignition_mode=2,
                          outputs=("burn_count", "burned_cells"), device_out=True)
            a = sim.simulate_noalloc(req)
            assert sim.stats()["list_capacity"] > 4096
            b = sim.simulate(req)
            torch.cuda.synchronize()
            assert int(a["burned_cells"][0]) > 15000
            for k in req.outputs:
                assert torch.equal(a[k], b[k]), (minutes, k)
            sim.unset_weather(w)
