"""The weight update's scratch: 41 B a particle with half as many again as room
for growth, the sort's own memory (its keys and values once more) and the
density grid."""
import pytest
import torch

from paper_2110_14494_amd import workloads as W
from test_gpu_weights import pic  # noqa: F401

pytestmark = pytest.mark.gpu


def test_memory_of_a_contexts_first_update(pic):  # noqa: F811
    n, cells = 2 ** 23, 128
    with pic.Context(0) as ctx:
        ctx.setup(W.electron_species(), W.air_like_tables())
        dg = pic.DeviceGrid(W.uniform_grid(cells, 39e-6))
        dp = pic.Particles.from_numpy(W.gaussian_particles(n, (64 * 39e-6,) * 3, 1e-3, seed=3), n + n // 4)
        print(f"[gpu] memory of update_weights n={n}", flush=True)
        ctx.push_collide_deposit(dp, dg, 1e-15, 1, 1, rho=dg.zeros_rho())  # the buffers of the steps and the deposit
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        rc, _ = ctx.update_weights(dp, dg, 1000.0, 1, 0, check=False)
        taken = before - torch.cuda.mem_get_info()[0]
    print(f"[gpu] first update took {taken / n:.1f} B a particle", flush=True)
    assert rc == 0
    sort = 12  # B a particle
    # two per cent for the sort's counters, 2 MiB for each of the ten allocations
    assert taken <= 1.02 * (41 + sort) * 1.5 * n + 8 * cells ** 3 + (20 << 20), taken
