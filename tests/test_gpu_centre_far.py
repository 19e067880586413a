"""The burnable cell nearest the centre where it lies 65536 cells or more away
(its squared distance leaves 32 bits), in every direction, tied and across the
edges of the search's tiles, against a direct search."""
import numpy as np
import pytest

from paper_1905_09317_amd import Request, Simulator

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sim():
    s = Simulator(0)
    yield s
    s.close()


# (rows, cols), burnable cells as row-major indices (negative ones from the end)
CASES = [
    ((140000, 1), [0]), ((140000, 1), [-1]), ((140000, 1), [0, -1]),
    ((1, 140000), [0]), ((1, 140000), [-1]),
    ((200000, 3), [0]), ((200000, 3), [-1]), ((200000, 3), [2, 0, -1, -3]),
    ((3, 200000), [0]), ((3, 200000), [-1]), ((3, 200000), [0, 400000, 199999, -1]),
    # 2^16 away, where the low 32 bits of the squared distance are 0, and nearer
    ((140000, 1), [70000 + 65536, 70000 - 60000]), ((140000, 1), [70000 - 65536, 70000 + 65535]),
    ((1, 262145), [131072 - 65536, 131072 + 65536, 131072 - 65537]),
    # 25 cells away in many directions: the lowest index
    ((60, 60), [30 * 60 + 55, 5 * 60 + 30, 10 * 60 + 15, 10 * 60 + 45, 55 * 60 + 30]),
    ((64, 64), [63, 4032]), ((127, 129), [0, -1, 128]), ((4097, 1), [0, 4095, 4096]), ((5000, 5000), [0, -1]),
]


@pytest.mark.parametrize("k", range(len(CASES)))
def test_far_centre_cell(sim, k):
    (rows, cols), at = CASES[k]
    fuel = np.zeros((rows, cols), np.uint8)
    fuel.reshape(-1)[at] = 2
    i = np.flatnonzero(fuel).astype(np.int64)
    d2 = (i // cols - rows // 2) ** 2 + (i % cols - cols // 2) ** 2
    print(f"far centre cell: {rows}x{cols}, {at}", flush=True)
    land = sim.load_landscape(fuel)
    wx = sim.set_weather(np.array([[[90.0, 60.0, 10.0, 0.0]]], np.float32))
    out = sim.simulate(Request(landscape=land, weather=wx, n_periods=1, ignition_mode=2, outputs=("ignition_cell",)))
    assert int(out["ignition_cell"][0]) == int(i[d2 == d2.min()][0])
    sim.unload_landscape(land)
    sim.unset_weather(wx)
