"""One wavefront per chain, a tile of up to 64 sites decided at a time: the
oracle's chains bit for bit where the fixed point is hardest to reach.

The weights jump from bin to bin (so a guessed bin gives wrong outcomes and
tiles take many passes), the binned range is cut close around the start
energies (so guesses leave the table and moves that leave it are rejected),
chain counts are not multiples of a workgroup's, and a launch's sweeps are
not a multiple of the four (two) sweeps that share a random-number batch on
lattices of one tile."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from gpu_common import assert_same_state, pair  # noqa: E402

pytestmark = pytest.mark.gpu

SHAPES = [("ising", L, 2, lay) for L in (4, 8, 16, 24, 32, 48, 64) for lay in (1, 2)] + \
         [("muma", L, 2, 1 + L // 8 % 2) for L in (4, 8, 16, 24, 32, 48, 64)] + \
         [("potts", L, q, 0) for L, q in ((4, 2), (8, 3), (16, 10), (24, 255), (32, 4), (48, 8), (64, 2))]


def rough(model, n_bins, scale):
    """A canonical slope plus independent noise of `scale` per bin."""
    rng = np.random.default_rng(n_bins)
    b = np.arange(n_bins)
    slope = {"ising": -1.2, "potts": -0.7, "muma": 0.0}[model]
    return slope * b + scale * rng.normal(size=n_bins)


@pytest.mark.parametrize("tlds", [0, 1])
@pytest.mark.parametrize("model,L,q,layout", SHAPES)
def test_rough_weights(model, L, q, layout, tlds):
    chains = {0: 17, 1: 5}[tlds]
    print(f"{model} L={L} q={q} layout={layout} tlds={tlds} chains={chains}", flush=True)
    fits = not (tlds == 1 and L == 64 and model in ("muma", "potts"))
    o, g = pair(model, L, chains, seed=500 + L, q=q, layout=layout, lpc=16, tlds=tlds if fits else -1)
    lnw = rough(model, g.n_bins, 1.0)
    g.set_lnw(lnw)
    T = o.thresholds(lnw)
    assert np.array_equal(g.thresholds(), T)
    o.sweeps(3, T, record=False)
    o.advance(3)
    g.thermalize(3)
    H = o.sweeps(6, T)
    acc = o.take_accepted()
    g.run_iteration(5)
    g.run_iteration(1)
    st = g.merge_update()
    assert np.array_equal(g.last_hist(), H), "histogram"
    assert st["accept_rate"] == acc / (6 * chains * L * L)
    assert_same_state(o, g)


@pytest.mark.parametrize("model,L,q", [("ising", 8, 2), ("ising", 64, 2), ("muma", 32, 2), ("potts", 16, 4),
                                       ("potts", 48, 3)])
def test_guesses_that_leave_the_range(model, L, q):
    """A range that ends at the lowest and highest start value."""
    chains, step = 64, {"ising": 4, "muma": 2, "potts": 1}[model]
    o, _ = pair(model, L, chains, seed=77 + L, q=q, lpc=16)
    b = o.bins()
    lo, hi = int(o.lo + step * b.min()), int(o.lo + step * b.max())
    for tlds in (0, 1):
        o, g = pair(model, L, chains, seed=77 + L, q=q, lo=lo, hi=hi, lpc=16, tlds=tlds)
        print(f"{model} L={L} range [{lo}, {hi}]: {g.n_bins} bins, tlds={tlds}", flush=True)
        lnw = 0.3 * np.random.default_rng(1).normal(size=g.n_bins)
        g.set_lnw(lnw)
        T = o.thresholds(lnw)
        H = o.sweeps(9, T)
        g.run_iteration(9)
        g.merge_update()
        assert np.array_equal(g.last_hist(), H)
        assert_same_state(o, g)


@pytest.mark.parametrize("chains_per_block", [4, 8, 16, 32])
def test_workgroup_shapes_and_counter_flushes(chains_per_block):
    """Workgroups of 4 to 16 wavefronts, and a launch long enough that the
    16-bit counters of one must be flushed on the way."""
    sweeps = 2 * (65535 // min(16, chains_per_block)) + 3 if chains_per_block >= 16 else 70
    print(f"ising L=4, 40 chains, {chains_per_block} per block, {sweeps} sweeps", flush=True)
    o, g = pair("ising", 4, 40, seed=3, cpb=chains_per_block, lpc=16)
    assert g.blocks_shape()[1] == chains_per_block
    lnw = rough("ising", g.n_bins, 0.3)
    g.set_lnw(lnw)
    H = o.sweeps(sweeps, o.thresholds(lnw))
    g.run_iteration(sweeps)
    g.merge_update()
    assert np.array_equal(g.last_hist(), H)
    assert_same_state(o, g)


@pytest.mark.parametrize("model,L,chains,tlds", [("ising", 8, 6912, 1), ("ising", 8, 6976, 1), ("potts", 8, 9216, 1),
                                                 ("potts", 8, 9280, 0), ("muma", 8, 10752, 0), ("muma", 8, 10816, 1),
                                                 ("muma", 4, 4096, 1), ("ising", 4, 4160, 1)])
def test_default_kernel_on_either_side_of_its_line(model, L, chains, tlds):
    """The default choice by chain count, against four lanes per chain."""
    from paper_1312_2213_amd import muca
    got = []
    for lpc in (0, 4):
        g = muca.Run(muca.muca_config_default(model, L, 3, chains, 5, lanes_per_chain=lpc, table_in_lds=tlds))
        g.set_lnw(rough(model, g.n_bins, 0.3))
        g.run_iteration(5)
        st = g.merge_update()
        s, b, _ = g.chain_state()
        got.append((g.last_hist(), st["accept_rate"], s, b))
    for x, y in zip(*got):
        assert np.array_equal(x, y)
