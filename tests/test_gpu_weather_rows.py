"""Weather tables on either side of the line between a wave and a lane a row,
long ones whose last wave is not full, and the largest there is: the rates of
rows at both ends and in between against the oracle's."""
import numpy as np
import pytest

import oracle
from paper_1905_09317_amd import Simulator

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_rows", [1024, 1025, (1 << 20) - 1, (1 << 20) + 1, 1 << 26])
def test_rates_of_long_weather_tables(n_rows):
    fuel = np.array([[2, 15, 6, 11, 18]], np.uint8)
    i = np.arange(n_rows, dtype=np.uint32)
    wx = np.empty((n_rows, 1, 4), np.float32)
    wx[:, 0, 0] = 80.0 + (i % 19).astype(np.float32)
    wx[:, 0, 1] = 20.0 + (i % 101).astype(np.float32)
    wx[:, 0, 2] = 3.0 + (i % 37).astype(np.float32)
    wx[:, 0, 3] = (i % 359).astype(np.float32)
    del i
    print(f"weather rows: {n_rows}", flush=True)
    with Simulator(0) as sim:
        land, w = sim.load_landscape(fuel), sim.set_weather(wx)
        for k in sorted({0, 1, 63, 64, n_rows // 2, n_rows - 2, n_rows - 1}):
            one = wx[k:k + 1]
            for precision in (0, 1):
                g = sim.eval_ros(land, w, scenario=k, precision=precision)
                o = oracle.eval_ros(fuel, None, one)
                tol = 1e-11 if precision == 0 else 1e-5
                assert np.allclose(g["x8"], o["x8"], rtol=tol, atol=1e-9), (k, precision)
