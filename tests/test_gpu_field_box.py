"""On large grids only the field records that the particles can reach are
formed.  Two electrons in opposite corners make the box the whole grid; the
others' fates must not change by them (bit for bit), wherever these start and
however fast they are."""
import numpy as np
import pytest

from paper_2110_14494_amd import workloads as W

pytestmark = pytest.mark.gpu
SHAPE = (163, 161, 165)  # just above 2^22 cells
DX = 1e-5


def _parts(where, speed, n):
    rng = np.random.default_rng(n)
    size = np.array(SHAPE[::-1]) * DX
    at = {"centre": 0.5, "corner": 0.004, "edge": 0.998, "outside": 1.02}[where]
    pos = at * size[:, None] + 3e-6 * rng.standard_normal((3, n))
    d = rng.standard_normal((3, n))
    v = speed * d / np.linalg.norm(d, axis=0)
    f = {k: a.astype(np.float32) for k, a in zip(("x", "y", "z", "vx", "vy", "vz"), np.concatenate([pos, v]))}
    return f | {"w": np.ones(n, np.float32), "id": np.arange(n, dtype=np.uint64)}


@pytest.mark.parametrize("where,speed,steps", [("centre", 0.0, 1), ("centre", 1e6, 12), ("corner", 3e6, 5),
                                               ("edge", 2e7, 20), ("outside", 1e7, 3), ("centre", 2e8, 9)])
def test_reachable_records_suffice(where, speed, steps):
    from paper_2110_14494_amd import pic
    n = 3001
    rng = np.random.default_rng(7)
    E = rng.normal(0, 1e7, SHAPE + (4,)).astype(np.float32)  # every record differs
    grid = {"E": E, "x0": 0.0, "y0": 0.0, "z0": 0.0, "dx": DX}
    out = []
    print(f"[gpu] reach {where} {speed:g} {steps}", flush=True)
    with pic.Context(0) as ctx:
        ctx.setup(W.electron_species(), W.air_like_tables())
        dg = pic.DeviceGrid(grid)
        for far in (True, False):  # the whole grid first, then the box
            p = _parts(where, speed, n)
            if far:
                ends = np.array([0.5, -0.5], np.float32) * np.float32(DX)
                top = np.array([0.0, 1.0], np.float32)
                q = {k: (ends + top * np.float32(s * DX)).astype(np.float32) for k, s in zip("xyz", SHAPE[::-1])}
                q |= {k: np.zeros(2, np.float32) for k in ("vx", "vy", "vz")}
                q |= {"w": np.ones(2, np.float32), "id": np.array([2 ** 60, 2 ** 60 + 1], np.uint64)}
                p = {k: np.concatenate([p[k], q[k]]) for k in p}
            dp = pic.Particles.from_numpy(p, 300 * n)
            ctx.push_collide_deposit(dp, dg, 1e-12, steps, 11)
            g = dp.to_numpy()
            o = np.argsort(g["id"])
            out.append({k: a[o] for k, a in g.items()})
    a, b = out
    common, ia, ib = np.intersect1d(a["id"], b["id"], return_indices=True)
    assert common.size == b["id"].size  # the corner electrons' own descendants aside, the same electrons
    for k in b:
        assert np.array_equal(a[k][ia], b[k][ib]), k
