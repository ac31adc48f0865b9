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


def test_height_follows_the_epochs(tmp_path):
    ws = run(tmp_path, """
w = 1024 * 256
v = np.stack(np.meshgrid(np.arange(90), np.arange(90)), -1).reshape(-1, 2)[:8000].astype(np.int32)

def size(E, cell):
    t = np.arange(E, dtype=np.int64) * 65536 * 4 // (E - 1)
    p = sas.Plan(v * 256, t, 1024, E // 2, (0, w, 0, w),
                 tuning=dict(n_det_hint=200000, coarse_log2=-1, cell_log2=cell))
    return p.workspace_size(200000)

out = [(size(E, 11) - size(E, 14)) / (4 * E * 128 * 128) for E in (8, 20, 60)]
""")
    # offsets of 128 x 128 cells a copy and epoch (8 px high) and of 128 x 64 (16 px)
    copies = [round(q) for q in ws]
    assert copies[0] == copies[1] and copies[0] == 2 * copies[2] and copies[2] >= 1
