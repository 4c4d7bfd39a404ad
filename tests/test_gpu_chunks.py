"""First chunks of the step kernel's waves at their edges: one smallest chunk a
wave, an even share up to 256 electrons a wave, three quarters of one beyond.
With 256 waves and with the default launch the same electrons come out (random
numbers follow the ids), bit for bit."""
import numpy as np
import pytest

from paper_2110_14494_amd import workloads as W
from test_gpu_schedule import COUNTS, _run, pic  # noqa: F401

pytestmark = pytest.mark.gpu
WAVES = 256


@pytest.mark.parametrize("n", [1, WAVES * 64 - 1, WAVES * 64 + 1, WAVES * 255 + 1, WAVES * 256, WAVES * 256 + 1,
                               WAVES * 300 + 7])
def test_first_chunks(pic, n):  # noqa: F811
    cfg = W.tip_block_config(m=32, n=n)
    ref, rho_ref, st_ref = _run(pic, cfg, None, steps=2)
    for s in ({"block": 64, "blocks_per_cu": 1}, {"block": 64, "blocks_per_cu": 1, "chunk": 64}):
        g, rho, st = _run(pic, cfg, s, steps=2)
        assert st["launch_grid"] == WAVES and st["launch_block"] == 64
        for k in COUNTS:
            assert st[k] == st_ref[k], k
        assert np.array_equal(rho, rho_ref)
        for k in ref:
            assert np.array_equal(g[k], ref[k]), k


@pytest.mark.parametrize("n,block", [(2 ** 14 - 1, 64), (2 ** 14, None), (2 ** 17 - 1, None), (2 ** 17, None)])
def test_default_launch_of_small_populations(pic, n, block):  # noqa: F811
    cfg = W.tip_block_config(m=32, n=n)
    ref, rho_ref, st_ref = _run(pic, cfg, {"block": 64, "blocks_per_cu": 1}, steps=2)
    for s in (None, {"blocks_per_cu": 2}):  # the second keeps a block that fits twice
        g, rho, st = _run(pic, cfg, s, steps=2)
        if s is None:
            assert st["launch_block"] == block if block else st["launch_block"] > 64
            assert (st["launch_grid"] == WAVES) == (n < 2 ** 17)
        elif n < 2 ** 17:
            assert st["launch_block"] == 64 and st["launch_grid"] == 2 * WAVES
        for k in COUNTS:
            assert st[k] == st_ref[k], k
        assert np.array_equal(rho, rho_ref)
        for k in ref:
            assert np.array_equal(g[k], ref[k]), k


@pytest.mark.parametrize("n0,blocks", [((700,) * 5, 1), ((2 ** 17, 2 ** 17), 1), ((2 ** 17, 2 ** 17 + 1), None)])
def test_default_launch_of_few_swarm_electrons(pic, n0, blocks):  # noqa: F811
    EN = np.linspace(60.0, 400.0, len(n0))
    out = []
    with pic.Context(0) as ctx:
        ctx.setup(W.electron_species(), W.air_like_tables())
        for launch in ({}, {"block": 512, "blocks_per_cu": 2}):
            print(f"[gpu] swarms {n0[:2]} {launch}", flush=True)
            rc, val, err, st, mom, cnt = pic.swarm_batch(ctx, EN, np.array(n0), 1e-12, 40, 3, sample_every=10, n_batches=2,
                                                         raw=True, **launch)
            assert rc == 0
            out.append((mom, cnt, st))
    if blocks:
        assert out[0][2]["launch_grid"] == blocks * WAVES
    for k in range(2):
        assert np.array_equal(np.asarray(out[0][k]), np.asarray(out[1][k]))
