"""Timed cases of the framework's public entry points.

Every case is one request, batch or comparison as a user's program makes it
through paper_1905_09317_amd: the landscapes, weather and handles such a
program keeps are made by prepare(), and run() is one pass.  Landscapes
follow the recipe of paper_1905_09317_amd.inputs (thresholded Gaussian random
fields of correlation length 30 cells, 1/f^3 elevations, hourly weather), drawn
with torch on the device because the largest has 67 million cells.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1905_09317_amd import Request, Simulator, inputs

DEVICE = "cuda:0"
DENSE = ("scar", "arrival_period", "burn_count", "burned_cells")   # what a single fire is run for
MAPS = ("burn_count", "burned_cells")                              # what a Monte-Carlo run is run for
ALL = ("scar", "arrival_period", "arrival_minute", "burn_count", "burned_cells", "ignition_cell", "scenario")


def _fire(name, rows, cols, periods, reps, **kw):
    """A simulate() case: one request on one resident landscape."""
    c = {"name": name, "kind": "simulate", "rows": rows, "cols": cols, "periods": periods, "reps": reps,
         "scenarios": 1, "sigma": 0.0, "rounding": 0, "precision": 0, "fuels": "mixed", "outputs": "maps",
         "device_out": True, "options": False}
    c.update(kw)
    return c


def _scars(name, rows, cols, periods):
    return {"name": name, "kind": "scars", "rows": rows, "cols": cols, "periods": periods}


def listed():
    return [
        # the smallest call there is: one short fire on 20 x 20 cells of one
        # fuel, every output, to host arrays; launches and latency
        _fire("tiny-20x20", 20, 20, 10, 1, fuels="c2", outputs="all", device_out=False),
        # one long fire on a large heterogeneous landscape, FP32 rates: the
        # single-fire workload of bench.py
        _fire("single-2048-fp32", 2048, 2048, 48, 1, precision=1, outputs="dense"),
        # one fire with the default FP64 results on a grid of odd sides, to
        # host arrays: the interactive what-if call
        _fire("single-1203x907-fp64", 1203, 907, 24, 1, outputs="dense", device_out=False),
        # the README's call: a burn-probability map from 64 noisy replications
        _fire("mc-512-64reps", 512, 512, 24, 64, sigma=0.15, rounding=1, device_out=False),
        # the batched Monte-Carlo workload of bench.py: many more replications
        # than the device holds at once, 100 weather scenarios
        _fire("mc-1024-2048reps", 1024, 1024, 48, 2048, scenarios=100, sigma=0.15, rounding=1),
        # Monte Carlo in FP32 with the options on (ignition threshold, burning
        # window, burn-out rate and intensity, later ignition, ignition map),
        # every fuel code, odd sides
        _fire("mc-options-751x640-fp32", 751, 640, 36, 301, scenarios=10, sigma=0.2, rounding=1, precision=1,
              fuels="every", options=True),
        # the largest landscape: bench.py's default workload
        _fire("large-8192-64reps", 8192, 8192, 72, 64, sigma=0.15, rounding=1),
        # a landscape that arrives with the call: upload, preparation, eight
        # fires, release (the cost of new inputs)
        {"name": "new-landscape-1500x1100", "kind": "new", "rows": 1500, "cols": 1100, "periods": 12, "reps": 8,
         "scenarios": 4, "sigma": 0.15, "rounding": 1, "precision": 0},
        # fuel-treatment planning: derive plans of one landscape, run them in
        # one fused launch, drop them (bench.py's treatments workload, fewer plans)
        {"name": "treatments-1024-4x64reps", "kind": "plans", "rows": 1024, "cols": 1024, "periods": 48, "reps": 64,
         "plans": 4, "scenarios": 20, "sigma": 0.15, "rounding": 1, "precision": 0},
        # a burst of small and middling queries through the serving lanes
        {"name": "served-16-queries", "kind": "served", "side_min": 128, "side_max": 1024, "queries": 16,
         "reps_max": 256, "periods": 48, "scenarios": 100, "sigma": 0.15, "rounding": 1, "precision": 0},
        # comparison of a fire with 48 hourly reference scars (bench.py's scars workload)
        _scars("scars-2048x48", 2048, 2048, 48),
        # the same on a grid whose rows do not align to words
        _scars("scars-1001x777x24", 1001, 777, 24),
    ]


def _spread(rng, lo, hi):
    """A whole number spread evenly over the logarithm of [lo, hi], odd as often as even."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["fire", "fire", "mc", "mc", "mc", "options", "new", "plans", "served", "scars"])
    prec = rng.choice([0, 0, 1])
    rounding, sigma = rng.choice([(0, 0.0), (1, 0.15), (1, 0.15), (0, 0.1), (1, 0.25)])
    if kind == "fire":
        c = _fire("", _spread(rng, 20, 2048), _spread(rng, 20, 2048), rng.randint(6, 48), 1, precision=prec,
                  outputs=rng.choice(["dense", "all"]), device_out=rng.random() < 0.5)
    elif kind == "mc":
        side = _spread(rng, 100, 3000)
        most = max(2, min(1024, int(1.5e9 / (side * side))))
        c = _fire("", side, _spread(rng, max(64, side // 2), side), rng.randint(12, 48), _spread(rng, 2, most),
                  scenarios=rng.randint(1, 50), sigma=sigma, rounding=rounding, precision=prec,
                  device_out=rng.random() < 0.6)
    elif kind == "options":
        c = _fire("", _spread(rng, 64, 900), _spread(rng, 64, 900), rng.randint(12, 48), _spread(rng, 1, 512),
                  scenarios=rng.randint(1, 10), sigma=0.2, rounding=1, precision=prec, fuels="every", options=True,
                  device_out=rng.random() < 0.5)
    elif kind == "new":
        c = {"kind": "new", "rows": _spread(rng, 64, 2048), "cols": _spread(rng, 64, 2048),
             "periods": rng.randint(6, 24), "reps": rng.randint(1, 16), "scenarios": rng.randint(1, 8),
             "sigma": sigma, "rounding": rounding, "precision": prec}
    elif kind == "plans":
        c = {"kind": "plans", "rows": _spread(rng, 128, 1024), "cols": _spread(rng, 128, 1024),
             "periods": rng.randint(12, 48), "reps": rng.randint(8, 64), "plans": rng.randint(2, 6),
             "scenarios": rng.randint(1, 20), "sigma": sigma, "rounding": rounding, "precision": prec}
    elif kind == "served":
        c = {"kind": "served", "side_min": 128, "side_max": _spread(rng, 200, 1024), "queries": rng.randint(2, 16),
             "reps_max": _spread(rng, 4, 256), "periods": rng.randint(12, 48), "scenarios": rng.randint(1, 100),
             "sigma": sigma, "rounding": rounding, "precision": prec}
    else:
        c = _scars("", _spread(rng, 100, 2048), _spread(rng, 100, 2048), rng.randint(2, 48))
    c.pop("name", None)
    return c


# ------------------------------------------------------------------- inputs
def _gen(seed, salt):
    return torch.Generator(DEVICE).manual_seed(int(seed) * 1_000_003 + salt)


def _standard(field):
    field -= field.mean(dtype=torch.float64)
    return field / field.std()


def _smooth_field(rows, cols, gen, corr_len=30.0):
    """Standardised periodic Gaussian random field."""
    spec = torch.fft.rfft2(torch.randn(rows, cols, generator=gen, device=DEVICE))
    ky = torch.fft.fftfreq(rows, device=DEVICE)[:, None]
    kx = torch.fft.rfftfreq(cols, device=DEVICE)[None, :]
    spec *= torch.exp(-2.0 * math.pi ** 2 * corr_len ** 2 * ky ** 2)
    spec *= torch.exp(-2.0 * math.pi ** 2 * corr_len ** 2 * kx ** 2)
    return _standard(torch.fft.irfft2(spec, s=(rows, cols)))


def _classes(rows, cols, n, gen):
    """Class numbers 0 .. n-1, equally likely, in patches."""
    u = torch.special.ndtr(_smooth_field(rows, cols, gen))
    return torch.clamp((u * n).to(torch.uint8), max=n - 1)


def _elevation(rows, cols, gen, top=800.0):
    """Metres in [0, top] with a power spectrum of |f|^-3."""
    spec = torch.fft.rfft2(torch.randn(rows, cols, generator=gen, device=DEVICE))
    f2 = torch.fft.fftfreq(rows, device=DEVICE)[:, None] ** 2 + torch.fft.rfftfreq(cols, device=DEVICE)[None, :] ** 2
    f2[0, 0] = math.inf
    spec *= f2 ** -0.75
    z = torch.fft.irfft2(spec, s=(rows, cols))
    z = (z - z.min()) * (top / float(z.max() - z.min()))
    return torch.round(z).to(torch.int16)


def _landscape(case, seed):
    """(fuel codes, elevations) as host arrays, what load_landscape takes."""
    rows, cols = case["rows"], case["cols"]
    fuels = case.get("fuels", "mixed")
    if fuels == "c2":
        return np.full((rows, cols), 2, np.uint8), None
    g = _gen(seed, 1)
    fuel = _classes(rows, cols, 19 if fuels == "every" else 16, g)
    elev = _elevation(rows, cols, g)
    return fuel.cpu().numpy(), elev.cpu().numpy()


def _weather(case, seed):
    return inputs.weather_scenarios(case["scenarios"], case["periods"], 1000 * int(seed) + 6)


def _noise(case, seed):
    return dict(seed=int(seed) + 7, sigma=case["sigma"], rounding=case["rounding"], precision=case["precision"],
                scenario_mode=1 if case["scenarios"] > 1 else 0)


def _outputs(case):
    return {"all": ALL, "dense": DENSE, "maps": MAPS}[case["outputs"]]


def _arrival(rows, cols, periods, gen, pace):
    """Arrival minutes of a fire from the middle of the grid that spreads at an uneven pace; -1 = not burned."""
    y = torch.arange(rows, device=DEVICE, dtype=torch.float32)[:, None] - rows / 2
    x = torch.arange(cols, device=DEVICE, dtype=torch.float32)[None, :] - cols / 2
    dist = torch.sqrt((x / cols) ** 2 + (1.6 * y / rows) ** 2)
    slow = torch.exp(0.25 * _smooth_field(rows, cols, gen))
    minute = torch.round(dist * slow * pace * (60 * periods)).to(torch.int32)
    return torch.where(minute <= 60 * periods, minute, -1).reshape(-1)


def _scar_inputs(case, seed):
    rows, cols, periods = case["rows"], case["cols"], case["periods"]
    sim = _arrival(rows, cols, periods, _gen(seed, 2), 2.2)
    ref = _arrival(rows, cols, periods, _gen(seed, 3), 2.4)
    scars = torch.empty(periods, rows * cols, dtype=torch.uint8, device=DEVICE)
    for t in range(periods):
        scars[t] = (ref >= 0) & (ref <= 60 * (t + 1))
    return sim, scars


def prepare(case, seed):
    kind = case["kind"]
    sim = Simulator(0)
    state = {"case": case, "sim": sim}
    if kind == "scars":
        state["arrival"], state["reference"] = _scar_inputs(case, seed)
    elif kind == "simulate":
        fuel, elev = _landscape(case, seed)
        rows, cols = fuel.shape
        land = sim.load_landscape(fuel, elev)
        wx = sim.set_weather(_weather(case, seed))
        kw = _noise(case, seed)
        if case["reps"] > 1:
            kw["ignition_mode"] = 1
        elif case["fuels"] == "c2":
            kw.update(ignition_mode=0, ignition_cell=(rows // 2) * cols + cols // 2)
        else:
            kw["ignition_mode"] = 2
        if case["options"]:
            w = np.random.default_rng(seed).integers(0, 100, fuel.shape).astype(np.uint32)
            sim.set_ignition_map(land, np.where(fuel > 0, w, 0))
            sim.set_landscape_fbp(land, fmc=105.0, pdf=40.0)
            kw.update(ignition_mode=3, ignition_period=2, threshold=0.5, burn_hours=14, burnout=1.0, hfi_min=50.0)
        state["request"] = Request(landscape=land, weather=wx, n_periods=case["periods"], reps=case["reps"],
                                   outputs=_outputs(case), device_out=case["device_out"], **kw)
    elif kind == "new":
        state["fuel"], state["elev"] = _landscape(case, seed)
        state["weather"] = _weather(case, seed)
        state["noise"] = _noise(case, seed)
    elif kind == "plans":
        fuel, elev = _landscape(case, seed)
        rows, cols = fuel.shape
        state["base"] = sim.load_landscape(fuel, elev)
        state["wx"] = sim.set_weather(_weather(case, seed))
        state["noise"] = _noise(case, seed)
        rng = np.random.default_rng(seed)
        state["edits"] = []
        for _ in range(case["plans"]):
            # a fuel break of three cells' width and a harvest of 5 % of the cells
            c0 = int(rng.integers(8, cols - 11))
            strip = (np.arange(rows)[:, None] * cols + np.arange(c0, c0 + 3)[None, :]).ravel()
            cut = rng.choice(rows * cols, rows * cols // 20, replace=False)
            cells = np.concatenate([strip, cut]).astype(np.int32)
            state["edits"].append((cells, np.zeros(cells.size, np.uint8)))
    else:
        sim.set_serving(lanes=4, admit_bytes=16 << 30)
        rng = np.random.default_rng(seed)
        mix = np.random.default_rng(case["queries"])   # sides and replications are the case's, the rest is the seed's
        g = _gen(seed, 1)
        base = case["side_max"]
        fuel, elev = _classes(base, base, 16, g).cpu().numpy(), _elevation(base, base, g).cpu().numpy()
        wx = sim.set_weather(_weather(case, seed))
        state["requests"] = []
        for q in range(case["queries"]):
            u = (q + mix.random()) / case["queries"]
            side = int(round(case["side_min"] * (case["side_max"] / case["side_min"]) ** u))
            r0, c0 = rng.integers(0, base - side + 1, 2)
            land = sim.load_landscape(fuel[r0:r0 + side, c0:c0 + side], elev[r0:r0 + side, c0:c0 + side])
            kw = _noise(case, seed)
            kw["seed"] += q
            state["requests"].append(Request(landscape=land, weather=wx, n_periods=case["periods"],
                                             reps=int(mix.integers(1, case["reps_max"] + 1)), ignition_mode=1,
                                             outputs=MAPS, **kw))
        # a server's lanes are running when a burst arrives
        ticket, _ = sim.submit(state["requests"][0])
        sim.wait(ticket)
    return state


def run(state):
    case, sim = state["case"], state["sim"]
    kind = case["kind"]
    if kind == "simulate":
        return sim.simulate(state["request"])
    if kind == "scars":
        return sim.compare_scars(state["arrival"], state["reference"])
    if kind == "new":
        land = sim.load_landscape(state["fuel"], state["elev"])
        wx = sim.set_weather(state["weather"])
        out = sim.simulate(Request(landscape=land, weather=wx, n_periods=case["periods"], reps=case["reps"],
                                   ignition_mode=1, outputs=MAPS, **state["noise"]))
        sim.unload_landscape(land)
        sim.unset_weather(wx)
        return out
    if kind == "plans":
        lands = [sim.derive_landscape(state["base"], cells, fuels) for cells, fuels in state["edits"]]
        out = sim.simulate_batch([Request(landscape=lid, weather=state["wx"], n_periods=case["periods"],
                                          reps=case["reps"], ignition_mode=1, outputs=MAPS, device_out=True,
                                          **state["noise"]) for lid in [state["base"]] + lands])
        for lid in lands:
            sim.unload_landscape(lid)
        return out
    tickets = [sim.submit(r)[0] for r in state["requests"]]
    return [sim.wait(t) for t in tickets]


def exact(case, seed):
    """The scar comparison's figures in 64 bits; simulations return whole numbers only."""
    if case["kind"] != "scars":
        return None
    arrival, scars = _scar_inputs(case, seed)
    n = arrival.numel()
    mse, ssim = np.zeros(case["periods"]), np.zeros(case["periods"])
    for t in range(case["periods"]):
        x = (scars[t] != 0).double()
        y = ((arrival >= 0) & (arrival <= 60 * (t + 1))).double()
        d2 = float((x - y).square().sum())
        mx, my = float(x.mean()), float(y.mean())
        vx, vy = float((x - mx).square().sum()) / (n - 1), float((y - my).square().sum()) / (n - 1)
        cov = float(((x - mx) * (y - my)).sum()) / (n - 1)
        mse[t] = d2 / n
        ssim[t] = (2 * mx * my + 1e-4) * (2 * cov + 9e-4) / ((mx * mx + my * my + 1e-4) * (vx + vy + 9e-4))
    return {"mse": mse, "ssim": ssim, "delta_norm": math.sqrt(d2)}


def work(case):
    """Bytes a pass cannot do without: fuel and elevation (3 B a cell) and weather (16 B a row) in, the wanted
    outputs out.  Fires touch a part of their landscape that depends on the draw; it is not counted."""
    kind = case["kind"]
    if kind == "served":
        # the mean square of a side spread evenly over its logarithm
        lo, hi = case["side_min"], case["side_max"]
        cells = case["queries"] * (hi * hi - lo * lo) / (2 * math.log(hi / lo))
        return {"bytes": cells * 7 + 16 * case["scenarios"] * case["periods"], "flops": 0}
    n = case["rows"] * case["cols"]
    if kind == "scars":
        return {"bytes": n * (4 + case["periods"]), "flops": 0}
    weather = 16 * case["scenarios"] * case["periods"]
    if kind == "plans":
        # each plan's edits (5 B a cell, 5 % of them) and map beside the base landscape and its map
        return {"bytes": n * 7 + case["plans"] * n * (4 + 0.25) + weather, "flops": 0}
    per_rep = {"scar": 1, "arrival_period": 4, "arrival_minute": 4}
    outs = _outputs(case) if kind == "simulate" else MAPS
    return {"bytes": n * (3 + 4 + case["reps"] * sum(per_rep.get(o, 0) for o in outs)) + 8 * case["reps"] + weather,
            "flops": 0}
