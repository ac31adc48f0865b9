"""Bands of the sort path over many velocities: few (a workgroup for each band),
and on either side of the number from which a workgroup takes every band of a
velocity (16384), with different numbers of bands.  Against the sort itself
and, where it is quick, the oracle."""
import numpy as np
import pytest

import oracle
from paper_2509_26279_amd import sas
from test_gpu_band_path import _catalog, _same

pytestmark = pytest.mark.gpu


def _grid(n, step, seed):
    side = int(np.ceil(np.sqrt(n)))
    v = np.stack(np.meshgrid(np.arange(side), np.arange(side)), -1).reshape(-1, 2)
    v = (v - side // 2) * step
    return np.random.default_rng(seed).permutation(v)[:n].astype(np.int32)


# velocities, bins in x and y, detections
@pytest.mark.parametrize("n_v,nx,ny,n", [
    (3, 60, 50, 4000), (600, 200, 300, 4000), (1300, 300, 700, 4000), (16384, 200, 300, 700),
    (16385, 200, 300, 700), (70000, 150, 200, 300)])
@pytest.mark.parametrize("mode", ["epochs", "detections"])
def test_many_velocities(gpu, n_v, nx, ny, n, mode):
    x, y, e, t, ext = _catalog(n, 20, nx * 64, ny * 64, n_v, -3000, 700)
    v = _grid(n_v, 7, n_v)
    lists = []
    for tun in ({"sort_vblock": -1}, {"sort_vblock": 1000}):
        plan = sas.Plan(v, t, 64, 3, ext, mode=mode, path="sort", tuning=tun)
        try:
            lists.append(sas.Search(plan, n, cand_cap=1 << 21).run(x, y, e))
        finally:
            plan.close()
    _same(lists[0], lists[1])
    if n_v < 70000:
        ref = oracle.vote(x, y, e, t, v, 64, 3, mode, 65535)
        assert len(ref) > 0
        _same(lists[0], ref)
