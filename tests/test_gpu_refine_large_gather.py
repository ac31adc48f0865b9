"""Fits that gather more detections than a set holds (512): the status, the true
number, and in place of the set that could not be kept the one that was
fitted, with nothing that another cluster left."""
import numpy as np
import pytest

from paper_2509_26279_amd import sas
from test_gpu_refine import STARTS, gpu_refine

pytestmark = pytest.mark.gpu

TOO_LARGE = {v: k for k, v in sas.REFINE_STATUS.items()}["too_large"]


def _scene(n_line, E=40, seed=2):
    """n_line detections within 1 px of a slow mover's line, some noise far off."""
    rng = np.random.default_rng(seed)
    t = (np.arange(E) * (3 * 65536) // (E - 1)).astype(np.int64)
    e = np.concatenate([np.arange(n_line) % E, rng.integers(0, E, 300)]).astype(np.uint8)
    th = t[e] / 65536.0
    x, y = 200 + 4.0 * th, 150 - 2.0 * th
    r, a = rng.uniform(0, 1.0, len(e)), rng.uniform(0, 2 * np.pi, len(e))
    x, y = x + r * np.cos(a), y + r * np.sin(a)
    x[n_line:] = rng.uniform(0, 400, 300)
    y[n_line:] = rng.uniform(250, 400, 300)
    return np.floor(256 * x).astype(np.int32), np.floor(256 * y).astype(np.int32), e, t


@pytest.mark.parametrize("cap", [512, 50, 7])
def test_fitted_set_in_place_of_the_gathered_one(gpu, cap):
    x, y, e, t = _scene(700)
    ext = (0, 400 * 256, 0, 400 * 256)
    # first a cluster that fills the sets of a workgroup, then short ones
    clusters = [np.arange(0, 500), np.arange(3, 33)[::-1], np.arange(100, 180, 2)]
    recs, gath, subs = gpu_refine(x, y, e, t, np.array([[0, 0]], np.int32), 1024, 5, clusters,
                                  STARTS[:64], radius_q8=4 * 256, extent=ext, gather_cap=cap)
    for r, g, s, cl in zip(recs, gath, subs, clusters):
        assert int(r["status"]) == TOO_LARGE and int(r["rounds"]) == 1
        assert int(r["n_gathered"]) == 700
        assert np.array_equal(g, np.sort(cl)[:cap])
        assert len(s) == (len(cl) + 4) // 2 and set(s.tolist()) <= set(cl.tolist())


def test_buffer_past_the_fitted_set(gpu):
    torch = gpu
    x, y, e, t = _scene(600)
    plan = sas.Plan(np.array([[0, 0]], np.int32), t, 1024, 5, (0, 400 * 256, 0, 400 * 256))
    try:
        s = sas.Search(plan, len(x), cand_cap=1 << 12)
        dev = s.upload(x, y, e)
        s.vote(*dev)
        first = torch.tensor([0, 30], dtype=torch.int32, device="cuda")
        members = torch.arange(30, dtype=torch.int32, device="cuda")
        starts = torch.as_tensor(STARTS[:64].view(np.int32)).cuda()
        out = torch.zeros((1, sas.REFINED_DTYPE.itemsize), dtype=torch.uint8, device="cuda")
        gath = torch.full((600,), -7, dtype=torch.int32, device="cuda")
        assert sas.load().sas_refine_clusters(
            plan.handle, s.ws.data_ptr(), s.ws.numel(), *(a.data_ptr() for a in dev), len(x),
            first.data_ptr(), members.data_ptr(), 30, 1, starts.data_ptr(), 64, 1024,
            out.data_ptr(), gath.data_ptr(), 600, None, None) == sas.SAS_OK
        torch.cuda.synchronize()
        got = gath.cpu().numpy()
        assert np.array_equal(got[:30], np.arange(30))
        assert (got[30:512] == -1).all() and (got[512:] == -7).all()
    finally:
        plan.close()
