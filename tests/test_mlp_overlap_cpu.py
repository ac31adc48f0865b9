"""Logits written over the rows they are computed from, without a GPU: such a
call goes through a buffer of the network's own, at most max_batch rows at a
time; buffers that only touch do not."""
from recorder_case import run


def test_overlapping_buffers(tmp_path):
    out = run(tmp_path, """
net = ctypes.c_void_p()
assert lib.sas_mlp_create(ctypes.c_int64(64), ctypes.c_uint64(1), ctypes.byref(net)) == 0
n = 150
x = buffer(4 * 32 * n + 8 * n) + 4 * n
out = {}
for name, z in (("before", x - 4 * n), ("first row", x - 4 * n + 4), ("same", x),
                ("last value", x + 4 * 32 * n - 4), ("after", x + 4 * 32 * n)):
    launches()
    assert lib.sas_mlp_forward(net, ctypes.c_void_p(x), ctypes.c_int64(n), ctypes.c_void_p(z),
                               None) == 0
    out[name] = [g[0] for g in launches()]
""")
    apart, through = ["k_mlp_forward"], ["k_mlp_forward", "k_mlp_copy"] * 3
    assert out == {"before": apart, "first row": through, "same": through,
                   "last value": through, "after": apart}
