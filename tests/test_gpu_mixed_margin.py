"""FP64 results at the inputs where an FP32 evaluation strays furthest from
FP64 (found by a search over weather, slope and fuel): steep slopes against the
wind in grass, C-6 that starts to crown in dry foliage, surface fuel
consumption from nearly equal terms.  One weather value is stepped through the
floats around every point where a rate crosses a rounding boundary, and the
burn-out intensity through values around the cell's own; integer rates equal
the floor of the same call's FP64 rates, fires equal the oracle's."""
import numpy as np
import pytest

from paper_1905_09317_amd import Request, Simulator

from _helpers import assert_same_outputs, oracle_run

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sim():
    s = Simulator(0)
    yield s
    s.close()


def _elevation(gx, gn):
    """A 3 x 3 grid whose middle cell has the (even) Horn numerators gx, gn."""
    z = np.zeros((3, 3), np.int16)
    z[1, 2 if gx > 0 else 0] = abs(gx) // 2
    z[0 if gn > 0 else 2, 1] = abs(gn) // 2
    return z


# fuel, (FFMC, BUI, wind km/h, direction), (gx, gn) on cells of 1 km, (percent
# conifer, curing, foliar moisture, percent dead fir), column stepped, range
RATES = {
    "grass, wind and slope cancel": (15, (95.0997, 118.6166, 112.2551, 442.5186), (5562, 780), (50, 100, 97, 50), 0,
                                     (94.0, 98.5)),
    "grass, the same turned": (14, (95.5266, 74.7782, 112.274, 412.4949), (4612, 3474), (50, 100, 97, 50), 0,
                               (94.0, 98.5)),
    "C-6 in dry foliage": (6, (72.2998, 25.5049, 59.8705, 170.6723), (2546, 2726), (100, 20, 1, 100), 1,
                           (24.0, 27.0)),
    "C-6 in dry foliage, light wind": (6, (81.6206, 24.2976, 22.7541, 108.0061), (-4804, -976), (100, 20, 1, 100), 1,
                                       (23.0, 26.0)),
    "C-6 in dry foliage, gale": (6, (81.6134, 24.2775, 102.7857, 108.0123), (-4794, -800), (100, 20, 1, 100), 0,
                                 (80.0, 83.0)),
}


def _wrong_at_boundaries(sim, land, row, col, lo, hi, cell, what, **kw):
    """(rates looked at, those that are not the floor of the FP64 rate) of one
    cell, the weather value `col` stepped through the floats around every
    rounding boundary between lo and hi."""
    def rates(values):
        wx = np.tile(np.float32(row), (len(values), 1))
        wx[:, col] = values
        w = sim.set_weather(wx[:, None, :])
        out = [sim.eval_ros(land, w, scenario=k, precision=0, **kw) for k in range(len(values))]
        sim.unset_weather(w)
        return np.array([o["x8"][cell] for o in out]), np.array([o["q8"][cell] for o in out])

    grid = np.linspace(lo, hi, 120).astype(np.float32)
    f = rates(grid)[0] + 0.5
    at = []
    for k, a in zip(*np.nonzero(np.floor(f[1:]) != np.floor(f[:-1]))):
        b = max(np.floor(f[k, a]), np.floor(f[k + 1, a]))
        at.append(np.float32(grid[k] + (grid[k + 1] - grid[k]) * (b - f[k, a]) / (f[k + 1, a] - f[k, a])))
    at = at[:: max(1, len(at) // 60)]
    print(f"rounding boundaries: {what}, {kw}, {len(at)} crossings", flush=True)
    if not at:
        return 0, []
    values = np.concatenate([t + np.arange(-24, 25) * np.spacing(t) * 8 for t in at]).astype(np.float32)
    x, q = rates(values)
    return q.size, [(float(values[k]), int(a), float(x[k, a]), int(q[k, a]))
                    for k, a in np.argwhere(q != np.floor(x + 0.5))]


@pytest.mark.parametrize("name", RATES)
@pytest.mark.parametrize("sigma", [0.0, 2.5])
def test_rates_at_rounding_boundaries(sim, name, sigma):
    fuel, row, grad, (pc, curing, fmc, pdf), col, (lo, hi) = RATES[name]
    land = sim.load_landscape(np.full((3, 3), fuel, np.uint8), _elevation(*grad), cell_m=1000, pc=pc, curing=curing)
    sim.set_landscape_fbp(land, fmc=fmc, pdf=pdf)
    n, bad = 0, []
    for rep in range(1 if sigma == 0.0 else 4):
        m, wrong = _wrong_at_boundaries(sim, land, row, col, lo, hi, 4, name, rep=rep, seed=3, sigma=sigma)
        n, bad = n + m, bad + wrong
    sim.unload_landscape(land)
    assert n > 0 and not bad, (len(bad), n, bad[:4])


@pytest.mark.parametrize("sigma", [1.0, 4.0, 7.0])
def test_rates_of_rare_draws_at_rounding_boundaries(sim, sigma):
    """The cells of 64 x 64 whose noise draws lie furthest out and whose rates
    are still of middling size."""
    land = sim.load_landscape(np.full((64, 64), 2, np.uint8))
    row = (92.0, 80.0, 25.0, 240.0)
    w = sim.set_weather(np.float32([[row]]))
    found = []
    for rep in range(40):
        top = sim.eval_ros(land, w, rep=rep, seed=9, sigma=sigma)["x8"].max(axis=1)
        for c in np.flatnonzero((top > 1.0) & (top < 2000.0)):
            found.append((float(top[c]), rep, int(c)))
    sim.unset_weather(w)
    n, bad = 0, []
    for _, rep, cell in sorted(found)[-6:]:
        m, wrong = _wrong_at_boundaries(sim, land, row, 1, 60.0, 100.0, cell, "rare draws", rep=rep, seed=9, sigma=sigma)
        n, bad = n + m, bad + wrong
    sim.unload_landscape(land)
    assert n > 0 and not bad, (len(bad), n, bad[:4])


# fuel, weather, slope, landscape; the fire is lit in the middle cell
FIRES = {
    "C-6": (6, (100.8279, 11.6323, 5.6439, 223.4224), (-1902, -4734), (100, 20, 1, 100)),
    "C-4": (4, (100.9728, 5.2478, 1.1493, 115.4707), (-390, -4530), (100, 20, 1, 100)),
}


@pytest.mark.parametrize("name", FIRES)
def test_burn_out_intensity_at_the_threshold(sim, name):
    fuel, row, grad, (pc, curing, fmc, pdf) = FIRES[name]
    grid, elev = np.full((3, 3), fuel, np.uint8), _elevation(*grad)
    wx = np.float32([[row]])
    land = sim.load_landscape(grid, elev, cell_m=1000, pc=pc, curing=curing)
    sim.set_landscape_fbp(land, fmc=fmc, pdf=pdf)
    w = sim.set_weather(wx, period_min=6000)
    hfi = sim.eval_ros(land, w)["hfi"][4]
    burned = set()
    for s in np.linspace(-1e-4, 1e-4, 41):
        kw = dict(n_periods=1, ignition_mode=0, ignition_cell=4, hfi_min=float(np.float32(hfi * (1.0 + s))))
        print(f"burn-out threshold: {name}, {kw['hfi_min']!r} at {hfi!r}", flush=True)
        g = sim.simulate(Request(landscape=land, weather=w, **kw))
        ref = oracle_run(grid, elev, wx, period_min=6000, cell_m=1000, pc=pc, curing=curing, fmc=fmc, pdf=pdf, **kw)
        assert_same_outputs(g, ref, where=f"{name} {kw}")
        burned.add(int(np.asarray(g["burned_cells"])[0]))
    assert len(burned) > 1   # the threshold decides
    sim.unload_landscape(land)
    sim.unset_weather(w)
