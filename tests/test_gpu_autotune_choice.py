"""What the autotuners pick where the candidates are far apart."""
import pytest

pytestmark = pytest.mark.gpu


def test_workgroups_of_eight_chains(monkeypatch):
    """2048 chains of Potts L = 48: sixteen chains per workgroup leave half of
    the CUs idle, four make two rounds; eight are 1.3 times as fast."""
    from paper_1312_2213_amd import muca
    monkeypatch.delenv("MUCA_AUTOTUNE_CACHE", raising=False)
    best, _ = muca.muca_autotune(muca.muca_config_default("potts", 48, 8, 2048, 3), 60)
    assert (best.lanes_per_chain, best.chains_per_block) == (16, 8)


def test_candidates_are_timed_on_weights_that_move(monkeypatch):
    """16384 chains of Ising L = 32: on flat weights one wavefront per chain
    is the fastest, on those of a run in progress it takes 1.15 to 1.25 times
    as long as four lanes per chain."""
    from paper_1312_2213_amd import muca
    monkeypatch.delenv("MUCA_AUTOTUNE_CACHE", raising=False)
    best, _ = muca.muca_autotune(muca.muca_config_default("ising", 32, 2, 16384, 3, layout=muca.MUCA_LAYOUT_BIT), 60)
    assert best.lanes_per_chain == 4


def test_item_times_are_those_of_weights_that_move(monkeypatch):
    """A fresh run has flat weights, on which sixteen wavefronts take 0.21 of
    the time of 64 chains at four lanes each; in progress 0.36 and more.  The
    run itself keeps its flat weights, thresholds and chains."""
    import numpy as np
    from paper_1312_2213_amd import muca
    monkeypatch.delenv("MUCA_AUTOTUNE_CACHE", raising=False)
    r = muca.Run(muca.muca_config_default("ising", 32, 2, 64, 3, layout=muca.MUCA_LAYOUT_BIT))
    T, state = r.thresholds(), r.checkpoint()
    us = muca.batch_tune(r)["us_per_sweep"]
    print(f"  {us}", flush=True)
    assert us["16_lanes"]["lds"] > 0.28 * us["4_lanes"]["lds"]
    assert np.array_equal(r.thresholds(), T) and not r.lnw().any() and r.checkpoint() == state
