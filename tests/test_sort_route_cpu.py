"""Which way the sort path takes for a catalog, and the workspace it asks for,
without a GPU: bands in place of the sort where they are expected to be faster
(many detections a band), the sort where a band's share is small, and a
workspace sized for a catalog serves every smaller one, whichever way those
take."""
from recorder_case import run

_BODY = """
from paper_2509_26279_amd import synth
wl = synth.make_fast(seed=5, n_epochs=60, noise_per_epoch=3000)
v = sas.grid_from_spec(wl.grid, wl.binw_q8, wl.span_q16)
few = v[(len(v) - 512) // 2:][:512]
b = buffer(4096)

def way(p, n, ws):
    launches()
    st = lib.sas_vote(p.handle, b, b, b, n, b, 16, b, b, ws, None)
    names = {g[0] for g in launches()}
    assert st == 0, (n, sas.load().sas_last_error())
    assert ("k_band_vote" in names) != ("k_sort_keygen" in names)
    return "bands" if "k_band_vote" in names else "sort"

def plan(vel, n_min=wl.n_min, **tuning):
    return sas.Plan(vel, wl.t_q16, wl.binw_q8, n_min, wl.extent_q8, path="sort", tuning=tuning)

out = {}
"""


def test_way_by_catalog_size(tmp_path):
    out = run(tmp_path, _BODY + """
p = plan(v, n_det_hint=1024)       # 1.2e6 velocities of 2 to 26 bands
out["whole"] = [way(p, n, p.workspace_size(n)) for n in (100, 1000, 180000)]
p = plan(few, n_det_hint=180000)
out["few"] = [way(p, n, p.workspace_size(n)) for n in (1, 4000, 180000)]
p = plan(few, n_det_hint=180000, sort_vblock=100)
out["sort asked for"] = [way(p, n, p.workspace_size(n)) for n in (4000, 180000)]
p = plan(v[:20000], n_det_hint=1000, sort_vblock=-1)
out["bands asked for"] = [way(p, n, p.workspace_size(n)) for n in (1, 1000)]
""")
    assert out["whole"] == ["sort", "sort", "bands"]
    assert out["few"] == ["bands"] * 3
    assert out["sort asked for"] == ["sort"] * 2
    assert out["bands asked for"] == ["bands"] * 2


def test_workspace(tmp_path):
    out = run(tmp_path, _BODY + """
p = plan(few, n_det_hint=180000)
out["few"] = p.workspace_size(180000)
p = plan(few, n_det_hint=180000, sort_vblock=512)
out["sorted"] = p.workspace_size(180000)
sizes = [0, 1, 2, 3, 1000, 4096, 4097, 8192, 16384, 20000, 32768, 32769, 65536, 100000, 180000]
out["grow"] = []
for q in (plan(v[:60000], n_det_hint=2000), plan(v[::7], n_det_hint=0), plan(few, 1)):
    ws = [q.workspace_size(n) for n in sizes]
    out["grow"].append(ws)
    for n in sizes[1:]:
        way(q, n, ws[-1])          # a workspace for the largest serves all
""")
    # bands write no keys: what is left is the window index (the sort's keys: 1.5 GB)
    assert out["few"] < 16 << 20 < 1 << 30 < out["sorted"]
    for ws in out["grow"]:
        assert ws == sorted(ws)
