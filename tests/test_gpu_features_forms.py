"""Candidate features at the edges of the kernel's forms, against the
oracle's FP64 definitions: epoch counts on either side of a wave's 64 and at
the limit, bins with more contributors than the kernel lists at a time, all
detections in one epoch, candidates that share a neighbour key or lie beyond
the key's range, and no neighbour look-up at all.

The features are FP32 roundings of FP64 sums: 2e-6 relative, and 2e-6 of a
bin or a unit where a sum cancels (a few hundred FP64 terms below 1e3 leave
errors below 1e-12, under the square root of f14, f15 and f31 1e-6)."""
import numpy as np
import pytest

from oracle import features as of
from paper_2509_26279_amd import sas

pytestmark = pytest.mark.gpu


def _run(x, y, e, t, v, n_min, extent, spacing, mode="epochs", cand=None):
    import torch
    plan = sas.Plan(v, t, 1024, n_min, extent, mode=mode)
    try:
        s = sas.Search(plan, len(x), cand_cap=1 << 16)
        dev = s.upload(x, y, e)
        s.vote(*dev)
        s.peaks()
        if cand is not None:  # a list of the caller's own
            s.cand[:len(cand)].copy_(torch.as_tensor(cand.view(np.int32).reshape(-1, 4)))
            s.res[0] = len(cand)
        snr = np.random.default_rng(3).uniform(3, 9, len(x)).astype(np.float32)
        recs, feat = s.features(len(x), torch.as_tensor(snr).cuda(), spacing_q8=spacing)
    finally:
        plan.close()
    ref = of.candidate_features(x, y, e, snr, t, v, 1024, recs, spacing_q8=spacing)
    return recs, feat, ref


def _same(feat, ref):
    assert feat.shape == ref.shape and len(ref)
    np.testing.assert_allclose(feat, ref, rtol=2e-6, atol=2e-6)


def _scene(E, per_epoch, seed, copies=1):
    """A slow mover seen `copies` times in every epoch, and noise."""
    rng = np.random.default_rng(seed)
    t = (np.arange(E, dtype=np.int64) * 65536) // max(E - 1, 1) + 99
    th = (t - t[0]) / 65536.0
    ee = np.repeat(np.arange(E), copies)
    x = 50.2 + 8.0 * th[ee] + rng.normal(0, 0.3, len(ee))
    y = 61.0 - 4.0 * th[ee] + rng.normal(0, 0.3, len(ee))
    m = per_epoch * E
    x = np.concatenate([x, rng.uniform(0, 128, m)])
    y = np.concatenate([y, rng.uniform(0, 128, m)])
    e = np.concatenate([ee, np.repeat(np.arange(E), per_epoch)]).astype(np.uint8)
    return (np.floor(256 * np.clip(x, 0, 127.9)).astype(np.int32),
            np.floor(256 * np.clip(y, 0, 127.9)).astype(np.int32), e, t)


V = np.array([[a, b] for b in (-2048, -1024, 0) for a in (1024, 2048, 3072)], np.int32)
EXT = (0, 128 * 256, 0, 128 * 256)


@pytest.mark.parametrize("E", [1, 2, 63, 64, 65, 128, 129, 256])
def test_epoch_counts(gpu, E):
    x, y, e, t = _scene(E, 60, E)
    _same(*_run(x, y, e, t, V, max(1, E // 3), EXT, 1024)[1:])


@pytest.mark.parametrize("copies", [4, 6, 40])
def test_more_contributors_than_a_list(gpu, copies):
    # 64 epochs: 256, 384 and 2560 detections of one bin, far more of its row
    x, y, e, t = _scene(64, 5, copies, copies)
    recs, feat, ref = _run(x, y, e, t, V, 40, EXT, 1024)
    assert ref[:, 1].max() * 64 > 192
    _same(feat, ref)


def test_no_neighbours_asked_for(gpu):
    x, y, e, t = _scene(30, 40, 5)
    recs, feat, ref = _run(x, y, e, t, V, 10, EXT, 0)
    assert np.all(feat[:, 9:11] == 0)
    _same(feat, ref)


def test_shared_and_unpackable_keys(gpu):
    """Velocities that round to one lattice index share keys (the largest
    count stands); bins and indices beyond the key's range have none."""
    x, y, e, t = _scene(30, 60, 6)
    v = np.concatenate([V, V + 100, V - 90, [[1024 * 1022, 0], [1024 * 1023, 0], [-1024 * 1023, 0],
                                              [1024 * 1022 + 511, 0], [1024 * 1022 + 512, 0]]])
    v = v.astype(np.int32)
    rng = np.random.default_rng(1)
    n = 700
    cand = np.zeros(n, dtype=sas.CAND_DTYPE)
    cand["v_idx"] = rng.integers(0, len(v), n)
    cand["bx"] = rng.integers(10, 16, n)
    cand["by"] = rng.integers(13, 18, n)
    cand["count"] = rng.integers(1, 9, n)
    cand["bx"][::50] = 16382
    cand["bx"][1::50] = 16383
    cand["by"][2::50] = -16382
    cand["by"][3::50] = -16383
    cand["count"][4::50] = 5000  # counts are capped at 4095
    recs, feat, ref = _run(x, y, e, t, v, 10, EXT, 1024, cand=cand)
    assert np.array_equal(recs, cand) and (ref[:, 9] > 0).any() and (ref[:, 9] == 0).any()
    assert np.any(ref[:, 1] == 0)  # bins without detections
    _same(feat, ref)
