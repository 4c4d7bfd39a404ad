"""The fluid step on both sides of its rule: a thread per cell on small grids,
waves of 64 columns by 2 rows by 4 planes that hand faces on from 5 * 2^19
cells (the smallest such grid, x a multiple of 64; and 2.5 tiles of x).  Random
densities in a random applied field, so that every face differs, against the
oracle with the bounds of the fluid parity tests (double-precision arithmetic,
single-precision field)."""
import numpy as np
import pytest
import torch

from oracle import fluid as FL
from paper_2110_14494_amd import workloads as W
from test_gpu_fluid import _table

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,steps", [((6, 10, 128), 2), ((18, 18, 66), 2), ((64, 320, 128), 1), ((96, 176, 160), 1)])
def test_fluid_tiles(shape, steps):
    from paper_2110_14494_amd import pic
    rng = np.random.default_rng(sum(shape))
    dx, gas_N = 1e-4, W.electron_species()["gas_N"]
    n0 = 1e17 * (1 + rng.random(shape))
    grid = {"E": np.zeros(shape + (4,), np.float32), "x0": 0.0, "y0": 0.0, "z0": 0.0, "dx": dx}
    grid["E"][..., :3] = rng.normal(0, 4e6, shape + (3,))
    tab = _table()
    ne_o, np_o, nn_o, info = FL.fluid_run(grid, n0, n0, np.zeros(shape), tab, gas_N, steps, 5e-12)
    print(f"[gpu] fluid tiles {shape}", flush=True)
    with pic.Context(0) as ctx:
        ctx.init_species(W.electron_species())
        t = [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (n0, n0.copy(), np.zeros(shape))]
        phi = torch.zeros(shape, dtype=torch.float64, device="cuda")
        E = torch.empty(shape + (4,), dtype=torch.float32, device="cuda")
        rc, hist, st = ctx.fluid_steps(pic.DeviceGrid(grid), *t, phi, tab, 5e-12, steps, mg_tol=1e-12, mg_max_cycles=80,
                                       E_out=E, check=False)
    assert rc == 0 and st["steps_done"] == steps
    assert np.allclose(hist, info["dt"], rtol=1e-9, atol=0)
    for g, o in zip(t, (ne_o, np_o, nn_o)):
        g = g.cpu().numpy()
        assert np.max(np.abs(g - o)) <= 1e-7 * np.max(np.abs(o))
