"""Scar comparison of grids whose rows do not start on words: last lanes of 1
to 15 cells, blocks of one batch of periods and of more than one window,
reference and arrival fields that start off a 16-byte boundary.  Counts are
exact, so MSE and norm are equal; SSIM to 1e-9 (the oracle's sums)."""
import numpy as np
import pytest

import oracle
from paper_1905_09317_amd import Simulator

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sim():
    s = Simulator(0)
    yield s
    s.close()


@pytest.mark.parametrize("n,T", [(2, 9), (15, 8), (17, 130), (31, 1), (16383, 17), (16385, 3), (33_000, 1030),
                                 (300_007, 25), (5_000_001, 7)])
@pytest.mark.parametrize("offset", [0, 1])
def test_ragged_scars_equal_the_oracle(sim, n, T, offset):
    import torch
    print(f"ragged scars n={n} T={T} offset={offset}", flush=True)
    rng = np.random.default_rng(n + T)
    arr = np.where(rng.random(n) < 0.5, rng.integers(0, T * 60 + 90, n), -1).astype(np.int32)
    ref = (rng.random((T, n)) < rng.random((T, 1))).astype(np.uint8) * 255
    a = torch.zeros(n + offset, dtype=torch.int32, device="cuda:0")
    r = torch.zeros(T * n + 3 * offset, dtype=torch.uint8, device="cuda:0")
    a[offset:] = torch.from_numpy(arr).to("cuda:0")
    r[3 * offset:] = torch.from_numpy(ref.reshape(-1)).to("cuda:0")
    g = sim.compare_scars(a[offset:], r[3 * offset:].view(T, n))
    o = oracle.scar_metrics(arr, (ref != 0).astype(np.uint8))
    np.testing.assert_array_equal(g["mse"], o["mse"])
    np.testing.assert_allclose(g["ssim"], o["ssim"], rtol=1e-9, atol=1e-12)
    assert g["delta_norm"] == o["delta_norm"]
