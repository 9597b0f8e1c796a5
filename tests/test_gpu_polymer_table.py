"""The polymer's B x B threshold matrix built on the device equals
floor(2^32 e^D) with the C library's exp, entry by entry: at the edges of the
tiles, with weights whose 2^32 e^D are whole numbers (so that the device
leaves entries, or whole tiles, to the host), and across set / get /
checkpoint."""
import math

import numpy as np
import pytest

from synth import polymer_walk

pytestmark = pytest.mark.gpu


def make(n_bins, chains=4, n_beads=6):
    from paper_1312_2213_amd import muca
    cfg = muca.muca_config_default("polymer", 0, 2, chains, 3, n_beads=n_beads, n_bins=n_bins)
    return muca.Run(cfg, positions=polymer_walk(n_beads, chains, 3))


def reference(lnw):
    B = len(lnw)
    T = np.zeros((B, B), np.uint32)
    for b in range(B):
        for k in range(B):
            D = lnw[k] - lnw[b]
            if D >= 0.0:
                T[b, k] = 0xFFFFFFFF
            elif D >= -23.0:
                v = math.exp(D) * 4294967296.0
                T[b, k] = 0xFFFFFFFF if v >= 4294967295.0 else int(v)
    return T.ravel()


def weights(kind, n):
    rng = np.random.default_rng(n)
    if kind == "smooth":
        return np.cumsum(0.05 * rng.normal(size=n))
    if kind == "halves":  # 2^32 e^D is a whole number for every pair
        return math.log(2.0) * rng.integers(0, 24, size=n)
    counts = rng.integers(1, 9, size=n).astype(np.float64)  # ratios of small counts
    return np.cumsum(np.log(counts[1:]) - np.log(counts[:-1]), dtype=np.float64).tolist() + [0.0]


@pytest.mark.parametrize("kind", ["smooth", "halves", "counts"])
@pytest.mark.parametrize("n_bins", [63, 64, 128, 129, 257, 385])
def test_matrix_equals_the_c_library(kind, n_bins):
    print(f"{kind}, {n_bins} bins", flush=True)
    g = make(n_bins)
    lnw = np.array(weights(kind, n_bins), np.float64)
    g.set_lnw(lnw)
    assert np.array_equal(g.thresholds(), reference(lnw))


def test_set_get_checkpoint():
    g, h = make(200), make(200)
    T = np.random.default_rng(1).integers(0, 1 << 32, size=200 * 200, dtype=np.uint32)
    g.set_thresholds(T)
    assert np.array_equal(g.thresholds(), T)
    h.restore(g.checkpoint())
    assert np.array_equal(h.thresholds(), T)
    for r in (g, h):
        r.run_iteration(3)
        r.merge_update()
    assert np.array_equal(g.last_hist(), h.last_hist()) and np.array_equal(g.thresholds(), h.thresholds())
