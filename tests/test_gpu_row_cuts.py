"""Rows of tiles cut to share the workgroup slots out: with 335 to 2144 pieces
of 1 to 90 tiles, lists equal the oracle's and the pieces hold every tile."""
import numpy as np
import pytest

import oracle
from paper_2509_26279_amd import sas

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("tile_x", [2, 16, 64])
@pytest.mark.parametrize("side", [3, 5, 6, 7, 9, 10])
@pytest.mark.parametrize("n,first_epoch", [(1500, 0), (1500, 3), (8000, 0), (8000, 3)])
def test_lists(gpu, tile_x, side, n, first_epoch):
    E, n_min = 16, 4
    rng = np.random.default_rng(side)
    t = (np.arange(E, dtype=np.int64) * 2 * 65536) // (E - 1) + 99
    x = rng.integers(0, 700 * 256, n).astype(np.int32)
    y = rng.integers(0, 301 * 256, n).astype(np.int32)
    e = rng.integers(first_epoch, E, n).astype(np.uint8)
    a = (np.arange(side) - side // 2) * 512
    v = np.stack(np.meshgrid(a, a), axis=-1).reshape(-1, 2).astype(np.int32)
    plan = sas.Plan(v, t, 1024, n_min, (0, 700 * 256, 0, 301 * 256),
                    tuning=dict(vblock_x=1, vblock_y=1, tile_x=tile_x, tile_y=6,
                                coarse_log2=-1, prune=-1))
    try:
        info = plan.info()
        got = sas.Search(plan, n, cand_cap=1 << 18).run(x, y, e)
    finally:
        plan.close()
    assert info["n_tiles_kept"] == info["n_tiles"] >= info["n_items_kept"]
    ref = oracle.vote(x, y, e, t, v, 1024, n_min, "epochs", 65535)
    assert len(got) == len(ref) and (n < 8000 or len(ref) > 0)
    for k in ("v_idx", "bx", "by", "count", "flags"):
        assert np.array_equal(got[k], ref[k]), k
