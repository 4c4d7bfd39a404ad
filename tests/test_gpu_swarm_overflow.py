"""Swarm steps that outgrow a region on a step that is sampled: the call ends
with the capacity error after the steps before, and the samples of these are
those of a call with room for all (bit for bit).  Ionization only, at a
constant frequency, without energy dependence."""
import numpy as np
import pytest

from paper_2110_14494_amd import workloads as W

pytestmark = pytest.mark.gpu
EN = np.array([5.0, 40.0, 300.0])
N0 = np.array([900, 64, 1500], dtype=np.int32)


def _run(growth, cap_factor, n0=N0):
    from paper_2110_14494_amd import pic
    print(f"[gpu] swarm overflow growth e^{growth:g} cap {cap_factor} n0 {n0.tolist()}", flush=True)
    with pic.Context(0) as ctx:
        ctx.setup(W.electron_species(), W.rate_tables({W.IONIZATION: 1e12}))
        return pic.swarm_batch(ctx, EN[:n0.size], n0, growth * 1e-12, 4, 23, sample_every=1, n_batches=2,
                               cap_factor=cap_factor, population_control=False, raw=True, check=False)


# e^3: twenty times the region's slots in the first step; e^0.8: 1, 2.2, 4.95
# and, in the third step, 11 electrons where there is room for 8
@pytest.mark.parametrize("growth,cap_factor,done", [(3.0, 4, 0), (0.8, 8, 2)])
def test_overflow_on_a_sampled_step(growth, cap_factor, done):
    rc, _, _, st, mom, cnt = _run(growth, cap_factor)
    assert rc == -2 and st["steps_done"] == done
    if done:
        rc, _, _, st, mom_all, cnt_all = _run(growth, 64)
        assert rc == 0 and st["steps_done"] == 4
        assert np.array_equal(mom[:, :done], mom_all[:, :done]) and np.array_equal(cnt[:, :done], cnt_all[:, :done])


def test_a_runaway_step_ends_at_its_first_overflow():
    """Twenty births per electron and step (a factor e^20): refused within some
    milliseconds.  A wave that ran 64 full queues of newborns first would take
    over a second (65536 rounds of its 64 lanes, 20 us or more each); the bound
    is well below that."""
    rc, _, _, st, _, _ = _run(20.0, 4, np.array([2000, 20000], dtype=np.int32))
    assert rc == -2 and st["steps_done"] == 0
    print(f"[gpu] runaway swarm step {st['step_kernel_ms']:.2f} ms", flush=True)
    assert st["step_kernel_ms"] < 250.0, st["step_kernel_ms"]


def test_a_waves_many_newborns_are_no_overflow():
    """64 electrons, all in one wave, with 9400 newborns a step: many times an
    even share of what the queue would hold, but they fit their region.  The
    shapes must agree bit for bit, and with the oracle's counts up to the rare
    decision flips."""
    import oracle
    from paper_2110_14494_amd import pic
    sp, tab = W.electron_species(), W.rate_tables({W.IONIZATION: 1e12})
    n0 = np.array([64], dtype=np.int32)
    runs = []
    with pic.Context(0) as ctx:
        ctx.setup(sp, tab)
        for shape in ({}, {"block": 64, "blocks_per_cu": 1}, {"block": 512, "blocks_per_cu": 2}):
            print(f"[gpu] many newborns of a wave {shape}", flush=True)
            runs.append(pic.swarm_batch(ctx, EN[:1], n0, 5e-12, 4, 23, sample_every=1, n_batches=2, cap_factor=600,
                                        raw=True, **shape))
    for r in runs[1:]:
        assert np.array_equal(r[4], runs[0][4]) and np.array_equal(r[5], runs[0][5])
    orc, _, oc, _ = oracle.swarm_run(sp, tab, EN[:1], n0, 5e-12, 4, 23, 1, cap_factor=600)
    assert orc == 0 and np.max(np.abs(runs[0][5][:, :, 0] - oc[:, :, 0])) <= 2


@pytest.mark.parametrize("growth,room,rc_want", [(5.0, 600, 0), (20.0, 4, -2)])
def test_the_particle_step_likewise(growth, room, rc_want):
    import oracle
    from paper_2110_14494_amd import pic
    from test_gpu_pic import compare
    n = 64 if rc_want == 0 else 20000
    sp, tab = W.electron_species(), W.rate_tables({W.IONIZATION: 1e12})
    grid, parts = W.uniform_grid(8, 1e-3, x0=-4e-3), W.uniform_box_particles(n, -1e-4, 1e-4, 3e6, seed=2)
    print(f"[gpu] particle step growth e^{growth:g}", flush=True)
    for shape in ({}, {"block": 512, "blocks_per_cu": 2}):
        with pic.Context(0) as ctx:
            ctx.setup(sp, tab)
            ctx.set_schedule(**shape)
            dp = pic.Particles.from_numpy(parts, room * n)
            rc, st = ctx.push_collide_deposit(dp, pic.DeviceGrid(grid), growth * 1e-12, 1, 5, check=False)
            g = dp.to_numpy()
        print(f"[gpu] growth e^{growth:g} {st['step_kernel_ms']:.2f} ms", flush=True)
        assert rc == rc_want and st["step_kernel_ms"] < 250.0, (rc, st["step_kernel_ms"])
        if rc_want == 0:
            orc, o, ost = oracle.pic_run(sp, tab, grid, parts, growth * 1e-12, 1, 5, capacity=room * n)
            assert orc == 0
            cmp = compare(g, o, 1e-3)
            assert cmp["flips"] <= max(2, 1e-4 * ost["trials"]), cmp
        else:
            assert sorted(g["x"].tolist()) == sorted(parts["x"].tolist())
