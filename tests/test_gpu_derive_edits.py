"""Edits of a derived landscape, several of one cell among them: the last one
given stands, for fewer and for more edits than cells.  Compared as the burn of
a landscape loaded with the edited fuel; and the refusal of a bad fuel code
names its cell wherever it lies."""
import numpy as np
import pytest

from paper_1905_09317_amd import Request, Simulator

from _helpers import assert_same_outputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sim():
    s = Simulator(0)
    yield s
    s.close()


@pytest.mark.parametrize("shape,n_edits", [((1, 2), 1), ((1, 2), 900), ((40, 33), 255), ((40, 33), 1320),
                                           ((40, 33), 1321), ((40, 33), 20000), ((300, 257), 257),
                                           ((300, 257), 70001)])
def test_last_edit_of_a_cell_stands(sim, shape, n_edits):
    rng = np.random.default_rng(n_edits)
    fuel = rng.integers(1, 19, shape).astype(np.uint8)
    elev = rng.integers(0, 90, shape).astype(np.int16)
    wx = rng.uniform([90, 50, 5, 0], [96, 120, 45, 360], (1, 6, 4)).astype(np.float32)
    spots = rng.integers(0, fuel.size, max(1, n_edits // 3))   # three edits of a cell and more
    cells = rng.choice(spots, n_edits).astype(np.int32)
    codes = rng.integers(0, 19, n_edits).astype(np.uint8)
    edited = fuel.copy().reshape(-1)
    for c, f in zip(cells, codes):
        edited[c] = f
    print(f"edits: {shape}, {n_edits}", flush=True)
    base = sim.load_landscape(fuel, elev)
    der = sim.derive_landscape(base, cells, codes)
    whole = sim.load_landscape(edited.reshape(shape), elev)
    w = sim.set_weather(wx)
    kw = dict(weather=w, n_periods=6, reps=8, seed=4, ignition_mode=1, sigma=0.1)
    try:
        if edited.any():
            assert_same_outputs(sim.simulate(Request(landscape=der, **kw)),
                                sim.simulate(Request(landscape=whole, **kw)), where=f"{shape} {n_edits}")
    finally:
        for lid in (der, whole, base):
            sim.unload_landscape(lid)
        sim.unset_weather(w)


@pytest.mark.parametrize("at", [0, 4095, 4096, 8200, 9999])
def test_bad_fuel_code_is_refused_with_its_cell(sim, at):
    fuel = np.ones((100, 100), np.uint8)
    fuel.reshape(-1)[at] = 19
    if at < 9999:
        fuel.reshape(-1)[9999] = 77
    with pytest.raises(Exception, match=f"fuel code 19 at cell {at} "):
        sim.load_landscape(fuel)
