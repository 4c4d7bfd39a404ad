"""The step kernel at the sizes where its work distribution changes: one
electron, a full and a barely started chunk per wave, and the first work
taken from the shared counter.  The results follow the electrons' ids, so
every launch shape must give the same density and counters bit for bit, and
the oracle the same electrons at the parity tests' bars (state within 1e-5,
at most 1e-4 of the flight segments deciding otherwise)."""
import pytest
import torch

import oracle
from paper_2110_14494_amd import workloads as W
from test_gpu_pic import compare

pytestmark = pytest.mark.gpu
COUNTERS = ("n", "trials", "null", "elastic", "excitation", "ionization", "attachment", "lost", "particle_steps")


# 256 one-wave blocks of 64-electron chunks below 2^17 electrons (16384 in
# first chunks), 4096 waves above (262144)
@pytest.mark.parametrize("n", [1, 64, 65, 16384, 16385, 131072, 262144, 262145, 600001])
def test_work_distribution_edges(n):
    from paper_2110_14494_amd import pic
    cfg = W.plain_swarm_config(n=n)
    cfg["grid"]["E"][..., 2] = 1e7  # births in most steps
    print(f"[gpu] step edges n={n}", flush=True)
    runs = []
    with pic.Context(0) as ctx:
        ctx.setup(cfg["species"], cfg["tables"])
        dg = pic.DeviceGrid(cfg["grid"])
        for shape in ({}, {"block": 64, "blocks_per_cu": 1}, {"block": 256, "blocks_per_cu": 2, "refill_min": 32}):
            ctx.set_schedule(**shape)
            dp = pic.Particles.from_numpy(cfg["parts"], 4 * n + 64)
            rho = dg.zeros_rho()
            _, st = ctx.push_collide_deposit(dp, dg, cfg["dt"], 3, cfg["seed"], rho=rho)
            runs.append((rho, [st[k] for k in COUNTERS], dp.to_numpy()))
    for rho, counters, _ in runs[1:]:
        assert torch.equal(rho, runs[0][0]) and counters == runs[0][1]
    if n > 16385:
        return
    g = runs[0][2]
    rc, o, ost = oracle.pic_run(cfg["species"], cfg["tables"], cfg["grid"], cfg["parts"], cfg["dt"], 3, cfg["seed"],
                                capacity=4 * n + 64)
    assert rc == 0
    cmp = compare(g, o, cfg["grid"]["dx"])
    assert cmp["flips"] <= max(2, 1e-4 * ost["trials"]) and cmp["w_equal"], cmp
