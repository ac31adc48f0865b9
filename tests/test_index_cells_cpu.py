"""Window-index cells by the work of a vote, without a GPU: short votes keep
nearly square cells, whose offsets the preparation clears and scans, and long
ones get narrow cells; a caller's own width is kept."""
from recorder_case import run


def test_width_follows_the_work(tmp_path):
    out = run(tmp_path, """
from paper_2509_26279_amd import synth
wl = synth.make_wide(seed=5, n_epochs=100, noise_per_epoch=3000)
v = sas.grid_from_spec(wl.grid, wl.binw_q8, wl.span_q16)

def cells(vel, **tuning):
    p = sas.Plan(vel, wl.t_q16, wl.binw_q8, wl.n_min, wl.extent_q8,
                 tuning=dict(n_det_hint=wl.n, refine_cap=1, **tuning))
    return p.info()["cell_log2"], p.workspace_size(wl.n)

out = [cells(v), cells(v[:4000]), cells(v[:1000]), cells(v[:20])]
w = out[0][0]
out.append(cells(v[:20], cell_log2=w))
""")
    width = [w for w, _ in out]
    size = [b for _, b in out]
    assert width[0] <= width[1] <= width[2] <= width[3] and width[0] < width[3]
    assert size[0] > 2 * size[3]
    assert width[4] == width[0]
