"""Rows of tiles against the workgroup slots, without a GPU: some more rows than
slots (512, two on each compute unit) are cut, as whole rows would leave most
slots idle in their last turn; no tile is lost."""
from recorder_case import run


def test_rows_are_cut(tmp_path):
    items, kept, tiles = run(tmp_path, """
t = (np.arange(60, dtype=np.int64) * 65536 * 4) // 59
s = 4096 * 65536 // int(t[-1] - t[0])
v = np.stack(np.meshgrid(np.arange(45), np.arange(45)), -1).reshape(-1, 2)[:2000] * s + 20 * s
i = sas.Plan(v.astype(np.int32), t, 4096, 40, (0, 2048 * 256, 0, 4096 * 256),
             tuning=dict(n_det_hint=200000, prune=-1)).info()
out = i["n_items_kept"], i["n_tiles_kept"], i["n_tiles"]
""")
    # two turns of the slots or more: whole rows are 1.4 turns of them
    assert items >= 1024 and kept == tiles
