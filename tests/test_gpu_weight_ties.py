"""Weight update with merge candidates of equal energy in a cell, which pair in
order of their ids: none, some of few, and more than are put in order in place
(32), many of them at rest (least = 0) or not, against the oracle bit for bit."""
import numpy as np
import pytest

import oracle
from test_gpu_weights import _cloud, _gpu_update, _sorted, pic  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,cells,levels,least", [(4000, 4, 1, 0), (4000, 4, 1, 1), (20_000, 8, 40, 0),
                                                  (20_000, 8, 3, 0), (20_000, 8, 3, 1), (33, 1, 1, 1), (32, 1, 1, 1),
                                                  (2, 1, 1, 0), (2000, 4, 0, 0)])
def test_equal_energies_pair_by_id(pic, n, cells, levels, least):  # noqa: F811
    p, grid = _cloud(n, max(cells, 2), 80e-6 * 16 / max(cells, 2))
    if cells == 1:  # one cell
        for k in "xyz":
            p[k] = np.full(n, 0.25 * grid["dx"], np.float32)
    if levels:  # speeds on a few values, exact in single precision
        rng = np.random.default_rng(n)
        p["vx"] = ((least + rng.integers(0, levels, n)) * 65536.0).astype(np.float32)
        p["vy"] = np.zeros(n, np.float32)
        p["vz"] = np.zeros(n, np.float32)
    p["id"] = np.random.default_rng(3).permutation(p["id"])
    rc, g, cnt = _gpu_update(pic, p, grid, 4.0, seed=8, idx=2, capacity=2 * n + 16)
    orc, o, ocnt = oracle.update_weights(p, grid, 4.0, seed=8, update_index=2, capacity=2 * n + 16)
    assert rc == 0 and orc == 0 and cnt == ocnt
    gs, os_ = _sorted(g), _sorted(o)
    for k in ("x", "y", "z", "vx", "vy", "vz", "w", "id"):
        assert np.array_equal(gs[k], os_[k].astype(gs[k].dtype)), k
