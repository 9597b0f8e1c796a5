"""Polymer sweeps on both sides of the rule for keeping the pair terms in LDS
(a workgroup of four chains of 64 beads leaves room for two per CU, with 6000
bins for one, as 80 beads do: more of those than fit at once do without, and
101 beads too),
one and two beads per lane, shifts and the full move set: histograms, bins and float
positions equal the oracle's."""
import numpy as np
import pytest

from synth import polymer_walk

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("moves", [0, 1])
@pytest.mark.parametrize("N,chains,n_bins", [(64, 129, 1000), (64, 2053, 1000), (64, 1029, 6000), (65, 130, 1000),
                                            (80, 1029, 1000), (101, 5, 1000)])
def test_pair_terms_kept_or_not(N, chains, n_bins, moves):
    from oracle import oracle as orc
    from paper_1312_2213_amd import muca
    print(f"N={N}, {chains} chains, {n_bins} bins, moves={moves}", flush=True)
    pos = np.tile(polymer_walk(N, 8, 17), (chains // 8 + 1, 1, 1))[:chains]
    rng = dict(x_lo=-400.0, x_hi=100.0, n_bins=n_bins)
    o = orc.PolymerRun(n_beads=N, n_chains=chains, seed=9, pos=pos, moves=moves, **rng)
    cfg = muca.muca_config_default("polymer", 0, 2, chains, 9, n_beads=N, moves=moves, **rng)
    g = muca.Run(cfg, positions=pos)
    lnw = -0.9 * o.bin_centres()
    o.lnW = np.array(lnw, np.float64)
    g.set_lnw(lnw)
    sweeps = 2 if chains > 1000 else 12
    H = o.sweeps(sweeps)
    g.run_iteration(sweeps)
    g.merge_update()
    assert np.array_equal(g.last_hist(), H)
    got, bins, _ = g.chain_state()
    assert np.array_equal(bins, o.bin)
    assert np.array_equal(got, o.pos)
