"""Scar comparison where the last lane holds 1 to 15 of its 16 cells (read from
the row's last 16 bytes, or byte by byte in a grid of fewer than 16 cells),
with references at any byte offset: exact counts against numpy."""
import numpy as np
import pytest
import torch

from paper_1905_09317_amd import Simulator

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sim():
    s = Simulator(0)
    yield s
    s.close()


@pytest.mark.parametrize("base", [0, 16, 16384, 1024 * 16 * 3])
def test_every_tail(sim, base):
    rng = np.random.default_rng(base)
    for n in range(max(2, base), base + 34):
        for T in (1, 9):
            arr = rng.integers(-1, 60 * T + 30, n).astype(np.int32)
            ref = (rng.random((T, n)) < 0.4).astype(np.uint8) * rng.integers(1, 256, (T, n)).astype(np.uint8)
            off = int(rng.integers(0, 16))
            buf = torch.full((T * n + 64,), 255, dtype=torch.uint8, device="cuda")
            buf[off:off + T * n] = torch.from_numpy(ref.reshape(-1)).cuda()
            print(f"scar tail: {n} cells, {T} periods, offset {off}", flush=True)
            g = sim.compare_scars(torch.from_numpy(arr).cuda(), buf[off:off + T * n].view(T, n))
            x = ref != 0
            y = (arr[None] >= 0) & (arr[None] <= 60 * np.arange(1, T + 1)[:, None])
            d = (x != y).sum(axis=1)
            assert np.array_equal(g["mse"], d / n), (n, T)
            assert g["delta_norm"] == np.sqrt(float(d[-1])), (n, T)
            if n > 2:
                mx, my = x.mean(axis=1), y.mean(axis=1)
                c = ((x * y).sum(axis=1) * n - x.sum(axis=1) * y.sum(axis=1)) / (n * (n - 1.0))
                vx, vy = (v.sum(axis=1) * (n - v.sum(axis=1)) / (n * (n - 1.0)) for v in (x, y))
                ssim = (2 * mx * my + 1e-4) * (2 * c + 9e-4) / ((mx * mx + my * my + 1e-4) * (vx + vy + 9e-4))
                np.testing.assert_allclose(g["ssim"], ssim, rtol=1e-9)
