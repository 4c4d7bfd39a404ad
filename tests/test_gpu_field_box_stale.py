"""On large grids a call forms only the field records that its particles can
reach.  Here every record left from the call before is wrong (another field,
much stronger and of the other sign), so a record that the box should have
held and did not changes what its electrons do.  The reference is a context of
its own, in which two electrons in opposite corners make the box the whole
grid; the others' fates must be the same bit for bit."""
import numpy as np
import pytest

from paper_2110_14494_amd import workloads as W
from test_gpu_field_box import DX, SHAPE, _parts

pytestmark = pytest.mark.gpu


def _with_corners(p):
    ends = np.array([0.5, -0.5], np.float32) * np.float32(DX)
    top = np.array([0.0, 1.0], np.float32)
    q = {k: (ends + top * np.float32(s * DX)).astype(np.float32) for k, s in zip("xyz", SHAPE[::-1])}
    q |= {k: np.zeros(2, np.float32) for k in ("vx", "vy", "vz")}
    q |= {"w": np.ones(2, np.float32), "id": np.array([2 ** 60, 2 ** 60 + 1], np.uint64)}
    return {k: np.concatenate([p[k], q[k]]) for k in p}


@pytest.mark.parametrize("where,speed,steps", [("centre", 0.0, 1), ("centre", 1e6, 12), ("corner", 3e6, 5),
                                               ("edge", 2e7, 20), ("outside", 1e7, 3), ("centre", 2e8, 9)])
def test_no_record_of_the_call_before_is_read(where, speed, steps):
    from paper_2110_14494_amd import pic
    n = 3001
    E = np.random.default_rng(7).normal(0, 1e7, SHAPE + (4,)).astype(np.float32)  # every record differs
    grid = {"E": E, "x0": 0.0, "y0": 0.0, "z0": 0.0, "dx": DX}
    parts = _parts(where, speed, n)
    few = _with_corners({k: a[:2] for k, a in parts.items()})
    print(f"[gpu] stale records {where} {speed:g} {steps}", flush=True)
    out = []
    for boxed in (False, True):
        with pic.Context(0) as ctx:
            ctx.setup(W.electron_species(), W.air_like_tables())
            if boxed:  # the whole grid of another field
                dp = pic.Particles.from_numpy(few, 4000)
                ctx.push_collide_deposit(dp, pic.DeviceGrid(grid | {"E": -30 * E}), 1e-14, 1, 3)
            dp = pic.Particles.from_numpy(parts if boxed else _with_corners(parts), 300 * n)
            ctx.push_collide_deposit(dp, pic.DeviceGrid(grid), 1e-12, steps, 11)
            g = dp.to_numpy()
            o = np.argsort(g["id"])
            out.append({k: a[o] for k, a in g.items()})
    a, b = out
    common, ia, ib = np.intersect1d(a["id"], b["id"], return_indices=True)
    assert common.size == b["id"].size  # the corner electrons' own descendants aside, the same electrons
    for k in b:
        assert np.array_equal(a[k][ia], b[k][ib]), k
