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


# newborns append behind the population and the holes are filled from the end
# of it: more holes than newborns, more newborns than holes, and no slot
# beyond the start count (the step first overflows that way and is run again
# with its newborns going into the holes)
@pytest.mark.parametrize("ion,att,room", [(5e10, 4e11, 2.0), (2e11, 5e10, 4.0), (1e11, 1.5e11, 1.0)])
def test_newborns_and_holes(ion, att, room):
    from paper_2110_14494_amd import pic
    n = 20011
    cap = int(room * n)
    sp, tab = W.electron_species(), W.rate_tables({W.ELASTIC: 1e12, W.IONIZATION: ion, W.ATTACHMENT: att})
    grid = W.uniform_grid(8, 1e-3, (0, 0, 1e6), x0=-4e-3)
    parts = W.uniform_box_particles(n, -1e-4, 1e-4, 1e6, seed=2)
    print(f"[gpu] newborns and holes {ion:g} {att:g} cap {cap}", flush=True)
    with pic.Context(0) as ctx:
        ctx.setup(sp, tab)
        dp, dg = pic.Particles.from_numpy(parts, cap), pic.DeviceGrid(grid)
        rc, st = ctx.push_collide_deposit(dp, dg, 1e-12, 4, 3, check=False)
        g = dp.to_numpy()
    orc, o, ost = oracle.pic_run(sp, tab, grid, parts, 1e-12, 4, 3, capacity=cap)
    assert rc == 0 and orc == 0 and st["steps_done"] == 4
    cmp = compare(g, o, 1e-3)
    assert cmp["flips"] <= max(2, 1e-4 * ost["trials"]), cmp


def test_step_beyond_any_capacity_keeps_the_previous_state():
    """Eight births per electron and step (a factor e^8): the first step
    outgrows the capacity and is not committed."""
    from paper_2110_14494_amd import pic
    n = 100
    sp, tab = W.electron_species(), W.rate_tables({W.IONIZATION: 8e12})
    parts = W.uniform_box_particles(n, -1e-4, 1e-4, 3e6, seed=2)
    print("[gpu] runaway step", flush=True)
    with pic.Context(0) as ctx:
        ctx.setup(sp, tab)
        dp = pic.Particles.from_numpy(parts, 5000)
        rc, st = ctx.push_collide_deposit(dp, pic.DeviceGrid(W.uniform_grid(8, 1e-3, x0=-4e-3)), 1e-12, 3, 1,
                                          check=False)
        g = dp.to_numpy()
    assert rc == -2 and st["steps_done"] == 0 and st["n"] == n
    for k in ("x", "vx", "id"):
        assert sorted(g[k].tolist()) == sorted(parts[k].tolist())


def test_ions_of_a_step_that_runs_again():
    """A self-consistent step whose newborns do not fit behind the population
    runs again; its ion events must count once (the charge balances exactly)."""
    from paper_2110_14494_amd import pic
    n = 20011
    sp, tab = W.electron_species(), W.rate_tables({W.ELASTIC: 1e12, W.IONIZATION: 1e11, W.ATTACHMENT: 1.5e11})
    print("[gpu] ions of a repeated step", flush=True)
    with pic.Context(0) as ctx:
        ctx.setup(sp, tab)
        dp = pic.Particles.from_numpy(W.uniform_box_particles(n, -1e-4, 1e-4, 1e6, seed=2), n)
        dg = pic.DeviceGrid(W.uniform_grid(16, 5e-4, (0, 0, 1e5), x0=-4e-3))
        n_pos, n_neg, n_e = dg.zeros_rho(), dg.zeros_rho(), dg.zeros_rho()
        ctx.deposit(dp, dg, n_pos)
        phi = torch.zeros(n_pos.shape, dtype=torch.float64, device="cuda")
        _, _, _, st = ctx.streamer_steps(dp, dg, n_pos, n_neg, phi, 1e-12, 3, 5, adaptive=False)
        ctx.deposit(dp, dg, n_e)
    assert st["steps_done"] == 3 and st["ionization"] > 1000 and st["attachment"] > 1000 and st["lost"] == 0
    assert int(n_pos.sum()) == (n + st["ionization"]) << 32 and int(n_neg.sum()) == st["attachment"] << 32
    assert int(n_e.sum()) == (n + st["ionization"] - st["attachment"]) << 32
