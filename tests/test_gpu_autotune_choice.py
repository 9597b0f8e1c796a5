"""What the autotuners pick where the candidates are far apart."""
import pytest

pytestmark = pytest.mark.gpu


def test_workgroups_of_eight_chains(monkeypatch):
    """2048 chains of Potts L = 48: sixteen chains per workgroup leave half of
    the CUs idle, four make two rounds; eight are 1.3 times as fast."""
    from paper_1312_2213_amd import muca
    monkeypatch.delenv("MUCA_AUTOTUNE_CACHE", raising=False)
    best, _ = muca.muca_autotune(muca.muca_config_default("potts", 48, 8, 2048, 3), 10)
    assert (best.lanes_per_chain, best.chains_per_block) == (16, 8)


def test_candidates_are_timed_on_weights_that_move(monkeypatch):
    """16384 chains of Ising L = 32: on flat weights one wavefront per chain
    is the fastest, on those of a run in progress it takes 1.15 to 1.25 times
    as long as four lanes per chain."""
    from paper_1312_2213_amd import muca
    monkeypatch.delenv("MUCA_AUTOTUNE_CACHE", raising=False)
    best, _ = muca.muca_autotune(muca.muca_config_default("ising", 32, 2, 16384, 3, layout=muca.MUCA_LAYOUT_BIT), 20)
    assert best.lanes_per_chain == 4
