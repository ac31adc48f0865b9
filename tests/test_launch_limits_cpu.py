"""Launches of the largest calls, counted without a GPU: a launch must hold
fewer than 2^32 threads (a larger grid is refused or wraps)."""
from recorder_case import run


def test_bands_of_the_whole_fast_grid(tmp_path):
    # 1.2e6 velocities of 2 to 26 bands each: 1.6e7 bands of 512 threads
    out = run(tmp_path, """
import resource
from paper_2509_26279_amd import synth
wl = synth.make_fast(seed=5, n_epochs=60, noise_per_epoch=3000)
v = sas.grid_from_spec(wl.grid, wl.binw_q8, wl.span_q16)
before = resource.getrusage(resource.RUSAGE_SELF).ru_maxrss
p = sas.Plan(v, wl.t_q16, wl.binw_q8, wl.n_min, wl.extent_q8, path="sort",
             tuning={"n_det_hint": wl.n})
grown = resource.getrusage(resource.RUSAGE_SELF).ru_maxrss - before
b = buffer(4096)
launches()
st = lib.sas_vote(p.handle, b, b, b, wl.n, b, 16, b, b, p.workspace_size(wl.n), None)
got = launches()
out = {"status": st, "n_v": len(v), "grown": grown, "launches": got}
""")
    assert out["status"] == 0 and out["n_v"] > 1 << 20
    bands = [g for g in out["launches"] if g[0] == "k_band_vote"]
    assert bands  # this many detections are counted in bands
    assert all(grid * block < 1 << 32 for _, grid, block in out["launches"])
    # no table of the bands: 80 bytes of host memory a velocity are the segments' and the sort's
    assert out["grown"] * 1024 < 160 * out["n_v"]


def test_features_of_the_longest_lists(tmp_path):
    # the neighbour table of more than 2^30 candidates has 2^32 slots
    out = run(tmp_path, """
V = np.zeros((4, 2), np.int32)
p = sas.Plan(V, np.arange(8) * 4096, 1024, 3, (0, 1 << 14, 0, 1 << 14))
b = buffer(4096)
out = []
for k in (1, 128, 129, 1 << 30, (1 << 30) + 1, (1 << 31) - 1):
    size = ctypes.c_size_t()
    assert lib.sas_features_scratch_size(ctypes.c_int64(k), ctypes.byref(size)) == 0
    launches()
    st = lib.sas_features(p.handle, b, p.workspace_size(100), 100, None, b,
                          ctypes.c_int64(k), 1024, b, size.value, b, None)
    out.append([k, st, launches()])
""")
    for k, status, got in out:
        assert status == 0
        names = [g[0] for g in got]
        assert names == ["k_table_clear", "k_table_insert", "k_neighbours", "k_features"]
        assert all(0 < grid * block < 1 << 32 for _, grid, block in got), k
