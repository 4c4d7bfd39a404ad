"""Tile counting, scattering and sorting at the edges of their blocks, against
the oracle's deposit bit for bit, and the step loop's sorted start against the
unsorted one (results follow the electrons' ids, not their order)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2110_14494_amd import workloads as W

pytestmark = pytest.mark.gpu


# the binned schedule starts at 2^18 particles; blocks of 8192 count and
# scatter; positions spread over tiles, in tile order, or all in one cell
@pytest.mark.parametrize("n", [2 ** 18, 2 ** 18 + 1, 34 * 8192 - 1, 300_007])
@pytest.mark.parametrize("order", ["spread", "sorted", "one cell"])
def test_binned_deposit_edges(n, order):
    from paper_2110_14494_amd import pic
    rng = np.random.default_rng(n)
    grid = {"E": np.zeros((21, 40, 33, 4), np.float32), "x0": -1e-4, "y0": 0.0, "z0": 2e-4, "dx": 1e-5}
    size = np.array([33, 40, 21]) * 1e-5
    u = rng.random((3, n)) if order != "one cell" else np.full((3, n), 0.5) + 1e-4 * rng.random((3, n))
    if order == "sorted":
        u = u[:, np.lexsort((u[0] // 0.24, u[1] // 0.2, u[2] // 0.38))]
    pos = (u * size[:, None] + np.array([-1e-4, 0.0, 2e-4])[:, None]).astype(np.float32)
    w = np.exp(rng.random(n) * 4).astype(np.float32)
    p = {"x": pos[0], "y": pos[1], "z": pos[2], "vx": 0 * w, "vy": 0 * w, "vz": 0 * w, "w": w,
         "id": np.arange(n, dtype=np.uint64)}
    print(f"[gpu] binned deposit n={n} {order}", flush=True)
    with pic.Context(0) as ctx:
        dg = pic.DeviceGrid(grid)
        rho = dg.zeros_rho()
        ctx.deposit(pic.Particles.from_numpy(p, n), dg, rho)
    assert np.array_equal(rho.cpu().numpy(), oracle.deposit(p["x"], p["y"], p["z"], p["w"], grid))


# 2^20 electrons and 8 steps start sorted by tile in blocks of 2^14
@pytest.mark.parametrize("n", [2 ** 20, 2 ** 20 + 1, 65 * 2 ** 14 - 1])
def test_sorted_start_changes_nothing(n):
    from paper_2110_14494_amd import pic
    cfg = W.streamer_config(n=n, grid_n=48, length=48 * 39e-6, dt=5e-13)
    runs = []
    print(f"[gpu] sorted start n={n}", flush=True)
    with pic.Context(0) as ctx:
        ctx.setup(cfg["species"], cfg["tables"])
        dg = pic.DeviceGrid(cfg["grid"])
        for parts in ((8,), (4, 4), (9,), (5, 4)):  # 4 and 5 steps keep the given order
            dp = pic.Particles.from_numpy(cfg["parts"], 2 * n)
            tot, s0 = 0, 0
            for k in parts:
                _, st = ctx.push_collide_deposit(dp, dg, cfg["dt"], k, cfg["seed"], step0=s0)
                tot, s0 = tot + st["trials"], s0 + k
            rho = dg.zeros_rho()
            ctx.deposit(dp, dg, rho)
            runs.append((rho, tot, dp.n, ctx.speed_quantile(dp)))
    for a, b in ((0, 1), (2, 3)):
        assert torch.equal(runs[a][0], runs[b][0]) and runs[a][1:] == runs[b][1:]
