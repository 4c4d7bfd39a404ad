"""The step kernel at the sizes where its first chunks stop covering the work.
A wave's first chunk is an even share of up to 256 electrons, at least 64, and
three quarters of one beyond, where the work counter hands out the rest: one
electron more than 256 a wave crosses that line (65536 for 256 waves, 524288
for 2048, 1048576 for 4096).  The default shape changes at 2^14 and 2^17
electrons.  The results follow the electrons' ids, so every shape must give the
same density and counters bit for bit."""
import pytest
import torch

from paper_2110_14494_amd import workloads as W

pytestmark = pytest.mark.gpu
COUNTERS = ("n", "trials", "null", "elastic", "excitation", "ionization", "attachment", "lost", "particle_steps")
SHAPES = ({}, {"block": 64, "blocks_per_cu": 1}, {"block": 512, "blocks_per_cu": 1}, {"block": 512, "blocks_per_cu": 2})


@pytest.mark.parametrize("n", [16383, 16384, 65536, 65537, 131071, 131072, 524288, 524289, 1048576, 1048577])
def test_first_chunks_and_grabs(n):
    from paper_2110_14494_amd import pic
    cfg = W.plain_swarm_config(n=n)
    cfg["grid"]["E"][..., 2] = 1e7  # births in most steps
    print(f"[gpu] first chunks and grabs n={n}", flush=True)
    runs, waves = [], []
    with pic.Context(0) as ctx:
        ctx.setup(cfg["species"], cfg["tables"])
        dg = pic.DeviceGrid(cfg["grid"])
        for shape in SHAPES:
            ctx.set_schedule(**shape)
            dp = pic.Particles.from_numpy(cfg["parts"], 4 * n + 64)
            rho = dg.zeros_rho()
            _, st = ctx.push_collide_deposit(dp, dg, cfg["dt"], 3, cfg["seed"], rho=rho)
            runs.append((rho, [st[k] for k in COUNTERS]))
            waves.append(st["launch_grid"] * st["launch_block"] // 64)
    cu = torch.cuda.get_device_properties(0).multi_processor_count
    assert waves == [cu if n < 2 ** 14 else 8 * cu if n < 2 ** 17 else 16 * cu, cu, 8 * cu, 16 * cu]
    for rho, counters in runs[1:]:
        assert torch.equal(rho, runs[0][0]) and counters == runs[0][1]
