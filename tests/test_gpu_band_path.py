"""The sort path's band items against the oracle and against the sort itself
(an explicit sort_vblock): footprints whose bins fill one band, several, the
last that bands take and the first that they do not; epoch counts around the
workgroup's two ways of sharing them and around the mask sizes; thresholds
that every occupied bin reaches; negative positions."""
import numpy as np
import pytest

import oracle
from paper_2509_26279_amd import sas

pytestmark = pytest.mark.gpu

FIELDS = ("v_idx", "bx", "by", "count", "flags")


def _same(a, b):
    assert len(a) == len(b), (len(a), len(b))
    for k in FIELDS:
        assert np.array_equal(a[k], b[k]), k


def _catalog(n, E, w, h, seed, x0=0, y0=0):
    rng = np.random.default_rng(seed)
    t = (np.arange(E, dtype=np.int64) * 65536) // max(E - 1, 1) + 5
    x = rng.integers(x0, x0 + w, n).astype(np.int32)
    y = rng.integers(y0, y0 + h, n).astype(np.int32)
    x[: n // 4] = x[n // 4: n // 4 + n // 4]  # bins that several epochs share
    y[: n // 4] = y[n // 4: n // 4 + n // 4]
    return x, y, rng.integers(0, E, n).astype(np.uint8), t, (x0, x0 + w, y0, y0 + h)


def _lists(x, y, e, t, ext, v, b, n_min, mode, sat=65535):
    out = []
    for tun in (None, {"sort_vblock": 3}):
        plan = sas.Plan(v, t, b, n_min, ext, mode=mode, count_sat=sat, path="sort", tuning=tun)
        try:
            out.append(sas.Search(plan, len(x), cand_cap=1 << 20).run(x, y, e))
        finally:
            plan.close()
    out.append(oracle.vote(x, y, e, t, v, b, n_min, mode, sat))
    return out


V = np.array([[0, 0], [512, -256], [-700, 300], [1300, 900], [-1, 1]], np.int32)


# bins in x, in y: one band; bands of one row; the last and the first beyond of
# both limits (16384 bins a row, 32 bands)
@pytest.mark.parametrize("nx,ny", [(40, 30), (120, 300), (16382, 20), (16384, 3), (16385, 3),
                                   (9000, 31), (9000, 33)])
def test_footprints(gpu, nx, ny):
    v = np.array([[0, 0], [-1, 1]], np.int32)
    x, y, e, t, ext = _catalog(6000, 20, nx * 64, ny * 64, nx + ny, -500, -900)
    band, srt, ref = _lists(x, y, e, t, ext, v, 64, 2, "epochs")
    assert len(ref) > 0
    _same(band, ref)
    _same(srt, ref)


@pytest.mark.parametrize("E", [1, 15, 16, 17, 64, 65, 256])
@pytest.mark.parametrize("n_min,mode", [(1, "epochs"), (2, "epochs"), (6, "epochs"),
                                        (2, "detections")])
def test_epochs_and_thresholds(gpu, E, n_min, mode):
    x, y, e, t, ext = _catalog(9000, E, 200 * 256, 170 * 256, E)
    band, srt, ref = _lists(x, y, e, t, ext, V, 1024, n_min, mode, 255)
    _same(band, ref)
    _same(srt, ref)


def test_more_hot_bins_than_masks(gpu):
    # every bin of 256 epochs holds four detections at least: 64 masks' worth of bins
    x, y, e, t, ext = _catalog(60000, 256, 128 * 64, 64 * 64, 3)
    band, srt, ref = _lists(x, y, e, t, ext, V[:2], 64, 9, "epochs")
    assert len(ref) > 256
    _same(band, ref)
    _same(srt, ref)
