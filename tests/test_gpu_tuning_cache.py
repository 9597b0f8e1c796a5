"""What an entry of MUCA_AUTOTUNE_CACHE may be read for: the kernels that it
was measured with, and a work item of as many chains."""
import json

import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture
def cache(tmp_path, monkeypatch):
    path = tmp_path / "tune.json"
    monkeypatch.setenv("MUCA_AUTOTUNE_CACHE", str(path))
    return path


def make(chains):
    from paper_1312_2213_amd import muca
    return muca.Run(muca.muca_config_default("ising", 16, 2, chains, 3, layout=muca.MUCA_LAYOUT_BIT))


def test_few_chains_are_not_an_item(cache):
    """A run of 3 chains fills 3 of an item's 16 wavefronts: its times are
    not those of a run of 64, whichever is tuned first."""
    from paper_1312_2213_amd import muca
    assert not muca.batch_tune(make(3))["from_cache"]
    assert not muca.batch_tune(make(64))["from_cache"]
    assert muca.batch_tune(make(3))["from_cache"]
    assert muca.batch_tune(make(100))["from_cache"] and muca.batch_tune(make(16))["from_cache"]
    assert not muca.batch_tune(make(15))["from_cache"]


def test_entries_of_other_kernels_are_not_read(cache):
    """Entries whose keys bear no revision, or another one."""
    import torch
    from paper_1312_2213_amd import muca
    cfg = muca.muca_config_default("ising", 16, 2, 64, 3, layout=muca.MUCA_LAYOUT_BIT)
    assert muca.muca_autotune(cfg, 5)[1] > 0
    assert not muca.batch_tune(make(64))["from_cache"]
    kept = json.loads(cache.read_text())
    assert len(kept) == 2 and torch.cuda.get_device_properties(0).gcnArchName.split(":")[0] in "".join(kept)
    for old in (lambda k: k[:k.rindex("/r")], lambda k: k[:k.rindex("/r")] + "/r1",
                lambda k: k[:k.rindex("/r")].replace("/c16", "")):
        cache.write_text("{\n" + ",\n".join(f'  "{old(k)}": {json.dumps(v)}' for k, v in kept.items()) + "\n}\n")
        assert muca.muca_autotune(cfg, 5)[1] > 0
        assert not muca.batch_tune(make(64))["from_cache"]
    assert muca.muca_autotune(cfg, 5)[1] == -1.0
    assert muca.batch_tune(make(64))["from_cache"]
