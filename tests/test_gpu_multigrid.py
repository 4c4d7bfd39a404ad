"""The potential solve on grids whose coarsest level is not 2 cells a side:
solved directly in double precision, or by sweeps where a side is too long
for the direct solve's matrices (arXiv:2110.14494 Sec. 2.5)."""
import numpy as np
import pytest
import torch

from oracle import field as F

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [
    (26, 22, 30),    # coarsest 13 x 11 x 15
    (5, 7, 9),       # a single odd level
    (16, 16, 16),    # halves to 2 x 2 x 2: sweeps
    (17, 16, 15),    # 4080 cells in one level
    (1, 6, 3),       # one plane between the two z faces
    (63, 1, 1),      # the longest side of the direct solve
    (64, 1, 3),      # one more: sweeps
    (80, 48, 112),   # three launched levels above the direct one
    (32, 32, 32),    # rows of 4 cells of a colour per thread
    (24, 24, 20),    # rows of 2 (20 / 2 is no multiple of 4)
    (20, 22, 18),    # rows of 1
    (22, 34, 30),    # rows of 1, an odd count of them
])
def test_potential_with_any_coarsest_level(shape):
    from paper_2110_14494_amd import pic
    nz, ny, nx = shape
    dx = 3e-5
    rng = np.random.default_rng(nz * 10007 + ny * 101 + nx)
    dens = [rng.integers(0, 2 ** 40, size=shape, dtype=np.int64) for _ in range(3)]
    dens[0][nz // 3:nz // 2 + 1, ny // 4:, : nx // 2 + 1] += 2 ** 42
    rho = F.charge_density(*dens, dx)
    ref = F.poisson(rho, dx)
    grid = {"E": np.zeros(shape + (4,), np.float32), "x0": 0.0, "y0": 0.0, "z0": 0.0, "dx": dx}
    phi = torch.zeros(shape, dtype=torch.float64, device="cuda")
    tol = 1e-10
    print(f"[gpu] potential {shape}", flush=True)
    with pic.Context(0) as ctx:
        _, rel = ctx.solve_potential(pic.DeviceGrid(grid), *[torch.from_numpy(a).cuda() for a in dens], phi, tol=tol,
                                     max_cycles=60)
    assert rel <= tol
    # the inverse's infinity norm: the discrete solution for a unit right-hand
    # side depends on z only and peaks at dx^2 (nz^2 + 1) / 8
    bound = tol * np.max(np.abs(rho)) / F.EPS0 * dx * dx * (nz * nz + 1) / 8
    assert np.max(np.abs(phi.cpu().numpy() - ref)) <= bound + 1e-13 * np.max(np.abs(ref))


@pytest.mark.parametrize("nx", [32, 20, 18])
def test_potential_off_16_bytes(nx):
    """A potential that starts 8 bytes off a 16-byte boundary gives the same."""
    from paper_2110_14494_amd import pic
    shape = (24, 20, nx)
    rng = np.random.default_rng(nx)
    dens = [torch.from_numpy(rng.integers(0, 2 ** 40, size=shape, dtype=np.int64)).cuda() for _ in range(3)]
    grid = pic.DeviceGrid({"E": np.zeros(shape + (4,), np.float32), "x0": 0.0, "y0": 0.0, "z0": 0.0, "dx": 3e-5})
    n = int(np.prod(shape))
    print(f"[gpu] unaligned potential {nx}", flush=True)
    with pic.Context(0) as ctx:
        out = []
        for off in (0, 1):
            phi = torch.zeros(n + 1, dtype=torch.float64, device="cuda")[off:off + n].view(shape)
            assert phi.data_ptr() % 16 == 8 * off
            ctx.solve_potential(grid, *dens, phi, tol=1e-10)
            out.append(phi.clone())
    assert torch.equal(out[0], out[1])
