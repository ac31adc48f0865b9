"""Rows of tiles walked several to a workgroup's turn, velocity blocks along
the footprint's long side, and window-index cells narrower than high: lists
must equal the oracle's for plans with enough rows for groups of two and four
(every vote form, with and without coverage pruning, a late first epoch, many
chips in one launch) and for tall, wide and odd footprints at the epoch counts
where a wave's index rows run out."""
import numpy as np
import pytest
import torch

import oracle
from paper_2509_26279_amd import sas

pytestmark = pytest.mark.gpu

FIELDS = ("v_idx", "bx", "by", "count", "flags")


def _catalog(n, E, width_q8, height_q8, seed, first_epoch=0):
    rng = np.random.default_rng(seed)
    t = (np.arange(E, dtype=np.int64) * 2 * 65536) // max(E - 1, 1) + 4321
    x = rng.integers(0, width_q8, n).astype(np.int32)
    y = rng.integers(0, height_q8, n).astype(np.int32)
    e = rng.integers(first_epoch, E, n).astype(np.uint8)
    # movers, so that the lists are not empty: 12 stacks of one detection an epoch
    for k in range(12):
        vx, vy = rng.integers(-8, 9, 2) * 256
        x0, y0 = rng.integers(width_q8 // 4, 3 * width_q8 // 4), rng.integers(
            height_q8 // 4, 3 * height_q8 // 4)
        for q in range(first_epoch, E):
            d = int(t[q] - t[first_epoch])
            i = (k * E + q) % n
            x[i] = np.clip(x0 + ((int(vx) * d) >> 16), 0, width_q8 - 1)
            y[i] = np.clip(y0 + ((int(vy) * d) >> 16), 0, height_q8 - 1)
            e[i] = q
    return x, y, e, t, (0, int(width_q8), 0, int(height_q8))


def _same(got, x, y, e, t, v, binw, n_min, mode, weight=None):
    kw = {} if weight is None else {"weight": weight}
    ref = oracle.vote(x, y, e, t, v, binw, n_min, mode, 65535, **kw)
    assert len(got) == len(ref) and len(ref) > 0
    for k in FIELDS:
        assert np.array_equal(got[k], ref[k]), k


def _grid(nx, ny, step=256):
    a = (np.arange(nx) - nx // 2) * step
    b = (np.arange(ny) - ny // 2) * step
    return np.stack(np.meshgrid(a, b), axis=-1).reshape(-1, 2).astype(np.int32)


# one velocity a block and one bin row a tile: rows of tiles = velocities x bin
# rows, in groups of two from 2.6e5 rows on and of four from 5.2e5
@pytest.mark.parametrize("rows", [2, 4])
@pytest.mark.parametrize("form", [{"groups": 1}, {"groups": 1, "packed": -1}, {"groups": 2},
                                  {"groups": 2, "packed": -1}, {"groups": 4}])
@pytest.mark.parametrize("mode,first_epoch", [("epochs", 0), ("epochs", 2), ("detections", 0)])
def test_row_groups(gpu, rows, form, mode, first_epoch):
    v = _grid(30, 30 * rows // 2)
    x, y, e, t, ext = _catalog(600, 12, 90 * 256, 400 * 256, 3, first_epoch)
    plan = sas.Plan(v, t, 256, 4, ext, mode=mode,
                    tuning=dict(form, vblock_x=1, vblock_y=1, tile_x=40, tile_y=1,
                                coarse_log2=-1))
    try:
        assert plan.info()["n_items_kept"] >= rows * 512 * 256
        got = sas.Search(plan, len(x), cand_cap=1 << 18).run(x, y, e)
    finally:
        plan.close()
    _same(got, x, y, e, t, v, 256, 4, mode)


def test_row_groups_weighted(gpu):
    v = _grid(30, 60)
    x, y, e, t, ext = _catalog(600, 12, 90 * 256, 400 * 256, 4)
    w = np.random.default_rng(5).integers(1, 256, len(x)).astype(np.uint8)
    plan = sas.Plan(v, t, 256, 700, ext, mode="weighted_epochs",
                    tuning=dict(vblock_x=1, vblock_y=1, tile_x=40, tile_y=1, coarse_log2=-1))
    try:
        got = sas.Search(plan, len(x), cand_cap=1 << 18).run(x, y, e, weight=w)
    finally:
        plan.close()
    _same(got, x, y, e, t, v, 256, 700, "weighted_epochs", w)


def test_row_groups_batch(gpu):
    v = _grid(30, 60)
    chips, cats = [], []
    try:
        for k, first in enumerate((0, 1, 0)):
            x, y, e, t, ext = _catalog(500 + 40 * k, 12, 90 * 256, 400 * 256, 20 + k, first)
            p = sas.Plan(v, t, 256, 4, ext,
                         tuning=dict(groups=2, vblock_x=1, vblock_y=1, tile_x=40 + k, tile_y=1,
                                     coarse_log2=-1))
            cats.append((x, y, e, t))
            chips.append((p, *(torch.as_tensor(a).cuda() for a in (x, y, e))))
        b = sas.Batch(chips, cand_cap=1 << 18)
        b.vote()
        for k, (x, y, e, t) in enumerate(cats):
            _same(b.peaks(k), x, y, e, t, v, 256, 4, "epochs")
    finally:
        for c in chips:
            c[0].close()


@pytest.mark.parametrize("w,h", [(601, 2400), (2400, 601), (1033, 1031)])
@pytest.mark.parametrize("E", [7, 64, 65, 128, 250])
@pytest.mark.parametrize("tuning", [{}, {"groups": 2}, {"groups": 1}, {"cell_log2": 9},
                                    {"coarse_log2": 3}, {"groups": 2, "coarse_log2": 2}])
def test_footprints(gpu, w, h, E, tuning):
    v = _grid(9, 9, 512)
    x, y, e, t, ext = _catalog(3000, E, w * 256 + 3, h * 256 + 1, E)
    n_min = max(3, E // 3)
    plan = sas.Plan(v, t, 1024, n_min, ext, tuning=dict(tuning, n_det_hint=len(x)))
    try:
        got = sas.Search(plan, len(x), cand_cap=1 << 18).run(x, y, e)
    finally:
        plan.close()
    _same(got, x, y, e, t, v, 1024, n_min, "epochs")
