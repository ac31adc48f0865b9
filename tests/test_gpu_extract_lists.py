"""Extraction where a cell's contributors fill or exceed what the kernel
lists at a time (256), over epoch counts around a wave's 64 lanes, and where
more clusters are ranked than a tile of keys or one wave's share holds.
Clusters and owners must equal the oracle's loop."""
import numpy as np
import pytest

from test_gpu_extract import _case

pytestmark = pytest.mark.gpu

V = np.array([[0, 0], [256, 0], [0, -256]], np.int32)
EXT = (0, 256 * 256, 0, 256 * 256)


@pytest.mark.parametrize("E", [63, 64, 65, 256])
@pytest.mark.parametrize("k", [255, 256, 257, 700])
def test_long_lists(gpu, E, k):
    rng = np.random.default_rng(E + k)
    t = (np.arange(E, dtype=np.int64) * 65536) // (E - 1) + 3
    # k detections of one bin (well inside it at every epoch), some more nearby
    x = np.concatenate([rng.integers(40 * 1024 + 300, 40 * 1024 + 600, k),
                        rng.integers(38 * 1024, 43 * 1024, 400)]).astype(np.int32)
    y = np.concatenate([rng.integers(30 * 1024 + 300, 30 * 1024 + 600, k),
                        rng.integers(28 * 1024, 33 * 1024, 400)]).astype(np.int32)
    e = rng.integers(0, E, len(x)).astype(np.uint8)
    for mode, n_min in (("detections", 40), ("epochs", max(20, E // 4))):
        ref = _case(x, y, e, t, V, 1024, n_min, mode, extent=EXT, rounds=(0, -1), member_cap=1)
        assert len(ref) > 0


@pytest.mark.parametrize("clusters", [1, 3, 4, 5, 16, 17, 1030])
def test_ranked_clusters(gpu, clusters):
    # one stack of 4 to 7 detections per cluster, far from the others
    rng = np.random.default_rng(clusters)
    E = 8
    t = np.arange(E, dtype=np.int64) * 4096
    side = 40
    cell = rng.permutation(side * side)[:clusters]
    xs, ys, es = [], [], []
    for c in cell:
        ep = rng.permutation(E)[: rng.integers(4, 8)]
        xs += [(c % side) * 1600 + 500] * len(ep)
        ys += [(c // side) * 1600 + 700] * len(ep)
        es += list(ep)
    x, y = np.array(xs, np.int32), np.array(ys, np.int32)
    ref = _case(x, y, np.array(es, np.uint8), t, V, 1024, 4, extent=EXT, rounds=(0, -1))
    assert len(ref) == clusters
