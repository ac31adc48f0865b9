"""What sas_vote_static's array holds, without a GPU: plans whose narrow
window-index cells do not leave room for their refinement list are voted with
wider cells; what does not fit with the widest is refused."""
import pytest

from recorder_case import run


@pytest.mark.parametrize("cap,fits", [(1 << 20, True), (3_000_000, True), (3_400_000, True),
                                      (4_200_000, False)])
def test_wide_chip(tmp_path, cap, fits):
    out = run(tmp_path, """
from paper_2509_26279_amd import synth
wl = synth.make_wide(seed=5, n_epochs=100, noise_per_epoch=3000)
v = sas.grid_from_spec(wl.grid, wl.binw_q8, wl.span_q16)
p = sas.Plan(v, wl.t_q16, wl.binw_q8, wl.n_min, wl.extent_q8,
             tuning={"n_det_hint": wl.n, "refine_cap": %d})
b = buffer(4096)
launches()
st = lib.sas_vote_static(p.handle, b, b, b, wl.n, b, 16, b, None)
out = [st, p.workspace_size(wl.n), len(launches())]
""" % cap)
    status, default, n_launches = out
    assert (status == 0) == fits and status in (0, -6)
    assert (n_launches > 0) == fits
    assert (default <= 64 << 20) == (cap == 1 << 20)
