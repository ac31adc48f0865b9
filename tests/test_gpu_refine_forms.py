"""The forms of the Steps 4-6 kernel against the oracle: sets on either side
of the sizes at which a start takes more points per lane or a whole wave,
points whose distances tie exactly, start counts that fill no wave, and
clusters whose gathered sets repeat in a cycle until the round limit.

Same comparison as tests/test_gpu_refine.py: status, rounds, subsets and
gathered sets identical, the fit within 1e-9 and 1e-6."""
import numpy as np
import pytest

from oracle import refine as R
from paper_2509_26279_amd import sas, synth
from test_gpu_refine import _movers_in_noise, check, gpu_refine

pytestmark = pytest.mark.gpu

V0 = np.array([[0, 0]], np.int32)


def _cloud(seed, n, E=64, size=600.0):
    """One slow mover seen n times among E epochs (repeats in an epoch share
    the position exactly every fourth time), in sparse noise."""
    rng = np.random.default_rng(seed)
    t = (np.arange(E) * (3 * 65536) // (E - 1)).astype(np.int64) - 4321
    th = (t - t[0]) / 65536.0
    ee = np.sort(rng.integers(0, E, n))
    x = 300 + 5.0 * th[ee] + rng.normal(0, 0.6, n)
    y = 280 - 3.0 * th[ee] + rng.normal(0, 0.6, n)
    for i in range(1, n, 4):  # exact duplicates: every distance of the pair ties
        x[i], y[i], ee[i] = x[i - 1], y[i - 1], ee[i - 1]
    m = 3000
    xs = np.concatenate([x, rng.uniform(0, size, m)])
    ys = np.concatenate([y, rng.uniform(0, size, m)])
    e = np.concatenate([ee, rng.integers(0, E, m)]).astype(np.uint8)
    return (np.floor(256 * xs).astype(np.int32), np.floor(256 * ys).astype(np.int32), e, t,
            [np.arange(n)], (0, int(size) * 256, 0, int(size) * 256))


@pytest.mark.parametrize("n", [5, 6, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 480])
def test_set_sizes(gpu, n):
    x, y, e, t, clusters, ext = _cloud(n, n)
    st = synth.mcd_starts(3, 41 if n > 128 else 130)
    got = gpu_refine(x, y, e, t, V0, 1024, 3, clusters, starts=st, extent=ext)
    check(got, x, y, e, t, clusters, 4.0, starts=st)


@pytest.mark.parametrize("k", [63, 64, 65, 1024])
def test_start_counts(gpu, k):
    # not a handful: the 4 points of a start are equally far from their mean
    # in exact arithmetic, so which of them one C-step takes can hang on the
    # last bit of an implementation; among many starts the best does not
    x, y, e, t, clusters = _movers_in_noise(11, n_movers=4, outlier_frac=0.4)
    st = synth.mcd_starts(5, k)
    got = gpu_refine(x, y, e, t, V0, 1024, 3, clusters, starts=st,
                     extent=(0, 800 * 256, 0, 800 * 256))
    check(got, x, y, e, t, clusters, 4.0, starts=st)


@pytest.mark.parametrize("seed", [1, 2, 21])
def test_cycles_of_sets_end_like_the_last_round(gpu, seed):
    x, y, e, t, clusters = _movers_in_noise(seed, n_movers=10, E=24, n_noise=9000,
                                            outlier_frac=0.6, size=400.0)
    st = synth.mcd_starts(7, 60)
    ref = [R.refine_cluster(x, y, e, t, c, st, 6.0) for c in clusters]
    limit = [i for i, o in enumerate(ref) if o["status"] == R.STATUS_MAX_ROUNDS]
    assert limit  # the case holds clusters that never settle
    got = gpu_refine(x, y, e, t, V0, 1024, 3, clusters, starts=st, radius_q8=6 * 256,
                     extent=(0, 400 * 256, 0, 400 * 256))
    for i in limit:
        assert int(got[0][i]["status"]) == R.STATUS_MAX_ROUNDS
        assert int(got[0][i]["rounds"]) == 10
    check(got, x, y, e, t, clusters, 6.0, starts=st)
