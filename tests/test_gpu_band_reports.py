"""Bands of the sort path that report much: every occupied bin (a threshold of
1), more bins than the epoch masks hold at a time, and more candidates than
the buffer takes, whose total stays exact and whose records are of the list."""
import numpy as np
import pytest

import oracle
from paper_2509_26279_amd import sas
from test_gpu_band_path import V, _catalog, _same

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", ["epochs", "detections"])
@pytest.mark.parametrize("E,n_min", [(20, 1), (20, 2), (256, 1)])
@pytest.mark.parametrize("v", [V, np.arange(40000, dtype=np.int32).reshape(-1, 2) % 300],
                         ids=["few", "many"])
def test_reports(gpu, E, n_min, mode, v):
    few = len(v) < 100
    n = 30000 if few else 12
    x, y, e, t, ext = _catalog(n, E, 190 * 64, 170 * 64, E)
    plan = sas.Plan(v, t, 64, n_min, ext, mode=mode, path="sort", tuning={"sort_vblock": -1})
    try:
        ref = oracle.vote(x, y, e, t, v, 64, n_min, mode, 65535)
        _same(sas.Search(plan, n, cand_cap=len(ref)).run(x, y, e), ref)
        s = sas.Search(plan, n, cand_cap=len(ref) - 1)
        s.vote(*s.upload(x, y, e))
        assert s.result()["n_cand"] == len(ref)
        got = {tuple(r) for r in s.cand.cpu().numpy().view(sas.CAND_DTYPE).reshape(-1).tolist()}
        assert len(got) == len(ref) - 1 and got < {tuple(r) for r in ref.tolist()}
    finally:
        plan.close()
