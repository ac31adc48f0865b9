"""The width of the window-index cells as a plan reports it and as a tuning
asks for it, without a GPU: a plan's reported width asks for the plan again,
and the tuner's candidates try the widths beside it."""
import pytest

from recorder_case import run

_BODY = """
from paper_2509_26279_amd import synth
wl = getattr(synth, "make_" + %r)(seed=5)
v = sas.grid_from_spec(wl.grid, wl.binw_q8, wl.span_q16)[::%d]
hint = {"n_det_hint": wl.n}
args = (v, wl.t_q16, wl.binw_q8, wl.n_min, wl.extent_q8)

def plan(**tuning):
    p = sas.Plan(*args, path=%r, tuning=dict(hint, **tuning))
    return p.info(), p.workspace_size(wl.n)

out = {"default": plan()}
w = out["default"][0]["cell_log2"]
out["again"] = plan(cell_log2=w)
out["wider"] = plan(cell_log2=w + 1)
"""


@pytest.mark.parametrize("style,every,path", [("tiny", 1, "dense"), ("wide", 40, "dense"),
                                              ("fast", 400, "dense"), ("fast", 400, "sort")])
def test_reported_width_gives_the_plan_again(tmp_path, style, every, path):
    out = run(tmp_path, _BODY % (style, every, path))
    assert out["again"] == out["default"]
    info, ws = out["wider"]
    assert info["cell_log2"] == out["default"][0]["cell_log2"] + 1
    assert ws < out["default"][1]            # fewer offsets


def test_tuner_varies_the_width(tmp_path):
    out = run(tmp_path, _BODY % ("wide", 40, "dense") + """
cands = sas.autotune_default_candidates(*args, base=hint)
out = [w, sorted({c["cell_log2"] for c in cands if "cell_log2" in c})]
""")
    assert out[1] == [out[0] - 1, out[0] + 1]
