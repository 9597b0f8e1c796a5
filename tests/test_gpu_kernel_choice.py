"""Which kernel a lattice run's plain launch takes by default (muca_tile_chains),
and that a run which changes it between iterations stays the same run."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def make(model, L, q, chains, **kw):
    from paper_1312_2213_amd import muca
    return muca.Run(muca.muca_config_default(model, L, q, chains, 5, **kw))


@pytest.mark.parametrize("model,L,q,tlds,line", [
    ("ising", 64, 2, -1, 10240), ("ising", 64, 2, 0, 12288), ("ising", 32, 2, -1, 8192), ("ising", 8, 2, -1, 8192),
    ("potts", 48, 8, -1, 12288), ("potts", 64, 3, -1, 24576), ("potts", 24, 3, -1, 6144), ("potts", 4, 3, -1, 1536),
    ("muma", 32, 2, -1, 20480), ("muma", 64, 2, -1, 40960), ("muma", 4, 2, -1, 4096)])
def test_either_side_of_the_line(model, L, q, tlds, line):
    print(f"{model} L={L} q={q} tlds={tlds}: {line} chains", flush=True)
    assert make(model, L, q, line, table_in_lds=tlds).tile_chains() == (16 if line > 2048 else 8)
    assert make(model, L, q, line + 1, table_in_lds=tlds).tile_chains() == 0


def test_explicit_lanes_and_workgroup_sizes():
    for lanes, want in ((1, 0), (2, 0), (4, 0), (16, 16)):
        assert make("ising", 16, 2, 4096, lanes_per_chain=lanes).tile_chains() == want
    for chains, want in ((64, 4), (1024, 4), (1025, 8), (2048, 8), (2049, 16), (4096, 16)):
        assert make("potts", 16, 3, chains).tile_chains() == want
    for cpb in (4, 8, 16):
        assert make("ising", 16, 2, 4096, lanes_per_chain=16, chains_per_block=cpb).tile_chains() == cpb


@pytest.mark.parametrize("model,L,q,chains", [("ising", 16, 2, 6144), ("potts", 8, 3, 8000)])
def test_a_run_that_changes_its_kernel(model, L, q, chains):
    """Flat weights take one wavefront per chain, those of the first
    iterations four lanes, settled ones a wavefront again; histograms, weights,
    spins, bins and per-block histograms are those of four lanes throughout,
    and a restored run takes the kernel of the one that was saved."""
    import torch
    a, b = make(model, L, q, chains), make(model, L, q, chains, lanes_per_chain=4)
    assert a.blocks_shape() == b.blocks_shape()
    shape = a.blocks_shape()[0], a.n_bins
    blocks = [torch.zeros(shape, dtype=torch.int64, device="cuda") for _ in range(2)]
    taken = []
    for it in range(8):
        sweeps = 10 if it < 3 else 300
        taken.append(a.tile_chains())
        print(f"  iteration {it}: {taken[-1]} chains per workgroup", flush=True)
        for r, h in zip((a, b), blocks):
            r.run_iteration(sweeps // 2)
            r.run_iteration_blocks(sweeps - sweeps // 2, h)
        sa, sb = a.merge_update(), b.merge_update()
        assert sa == sb
        assert np.array_equal(a.last_hist(), b.last_hist()) and np.array_equal(a.lnw(), b.lnw())
        assert torch.equal(blocks[0], blocks[1])
        for x, y in zip(a.chain_state()[:2], b.chain_state()[:2]):
            assert np.array_equal(x, y)
        c = make(model, L, q, chains)
        c.restore(a.checkpoint())
        assert c.tile_chains() == a.tile_chains()
    assert taken[0] == 16 and taken[1] == 0 and taken[-1] == 16, taken
