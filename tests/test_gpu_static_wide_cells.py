"""sas_vote_static where the refinement list leaves room only for wider window-
index cells than the plan's own: the list of sas_vote, cell width by width."""
import numpy as np
import pytest

from paper_2509_26279_amd import sas, synth
from test_zz_no_alloc import _both, _same

pytestmark = pytest.mark.gpu


def test_wider_cells(gpu):
    torch = gpu
    wl = synth.make_wide(seed=4, n_epochs=60, noise_per_epoch=1500)
    v = sas.grid_from_spec(wl.grid, wl.binw_q8, wl.span_q16)
    v = v[np.random.default_rng(1).permutation(len(v))[:700]]
    dev = [torch.as_tensor(a).cuda() for a in (wl.x_q8, wl.y_q8, wl.epoch)]

    def plan(cap):
        return sas.Plan(v, wl.t_q16, wl.binw_q8, 7, wl.extent_q8,
                        tuning={"n_det_hint": wl.n, "refine_cap": cap, "cell_log2": 10})
    p = plan(1)
    index = p.workspace_size(wl.n)          # bytes but for the list
    p.close()
    lists = 0
    # the whole index fits beside the list, and shrinking parts of it
    for part in (1.02, 0.98, 0.7, 0.5, 0.4):
        p = plan(int((sas.STATIC_SCRATCH_BYTES - part * index) // 16))
        try:
            assert (p.workspace_size(wl.n) > sas.STATIC_SCRATCH_BYTES) == (part < 1)
            ref, got = _both(p, *dev, 1 << 18)
            _same(ref, got)
            lists += len(ref) > 100
        finally:
            p.close()
    assert lists == 5
