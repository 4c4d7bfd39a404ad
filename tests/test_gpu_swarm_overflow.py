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
