"""The search's launch shape and whether builds of few partitions get teams: what is set is what holds,
reading and setting back changes nothing, and tuning on a large batch leaves the teams of small builds."""

import ctypes as C

import numpy as np
import pytest

from paper_2404_18497_amd import autotune, binding, synth

TEAMS = 1


@pytest.fixture(autouse=True)
def restored():
    before = binding.get_search_config()
    yield
    binding.set_search_config(**before)
    assert binding.get_search_config() == before


def _set(*words):
    assert binding.lib().phobic_set_search_config(C.byref(binding.SearchConfig(*words))) == 0


def _reserved():
    cfg = binding.SearchConfig()
    assert binding.lib().phobic_get_search_config(C.byref(cfg)) == 0
    return cfg.reserved


def test_default_and_explicit_shapes():
    assert _reserved() == TEAMS
    before = binding.get_search_config()
    assert before == dict(waves_per_group=1, groups_per_cu=0, items_per_grab=1, teams=True)
    _set(1, 0, 1, 0)  # one wavefront per partition for every build
    assert _reserved() == 0 and "teams" not in binding.get_search_config()
    binding.set_search_config(**before)
    assert _reserved() == TEAMS
    _set(2, 0, 1, 7)  # values without a meaning are taken as 0
    assert _reserved() == 0
    binding.set_search_config(waves_per_group=8, groups_per_cu=4)
    assert _reserved() == 0


@pytest.mark.parametrize("cands", [None, [dict(waves_per_group=8, groups_per_cu=4, items_per_grab=1)]])
def test_tuning_keeps_the_teams(cands):
    class Built:
        def build_info(self):
            return {"search_ms": 1.0 if binding.get_search_config()["waves_per_group"] == 8 else 2.0}

        def close(self):
            pass

    best, table = autotune.tune(lambda: [Built()], repeats=1, cands=cands)
    assert best["waves_per_group"] == 8 and len(table) == (1 if cands else len(autotune.candidates()))
    assert binding.get_search_config() == best and _reserved() == TEAMS
    autotune.tune(lambda: [Built()], repeats=1, cands=[dict(waves_per_group=8, teams=False)])
    assert _reserved() == 0


@pytest.mark.gpu
def test_shapes_and_teams_give_the_same_image():
    import torch

    keys = torch.from_numpy(synth.u64_keys(60_000, 31).view(np.int64)).cuda()
    prm = binding.params(lam=9.0)
    want = binding.build_u64(keys, prm).serialize()
    for words in [(1, 0, 1, 0), (1, 0, 1, TEAMS), (8, 4, 4, 0), (8, 4, 4, TEAMS)]:
        _set(*words)
        assert np.array_equal(binding.build_u64(keys, prm).serialize(), want), words
