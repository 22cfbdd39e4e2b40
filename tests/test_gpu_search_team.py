"""The team search on the device: images equal the oracle's on both sides of every partition count at
which the launch rule changes the wavefronts per partition (256 compute units: 1, 3, 6, 12, 16, 32
and 64 times that), and in every table layout of the kernel."""

import numpy as np
import pytest
import torch

import oracle
from paper_2404_18497_amd import binding, synth

pytestmark = pytest.mark.gpu


def _image(keys, prm):
    return binding.build_u64(torch.from_numpy(keys.view(np.int64)).cuda(), prm).serialize()


@pytest.mark.parametrize("P,K,lam,alpha", [
    (100, 1, 7.0, (1, 1)), (100, 256, 5.0, (1, 1)), (100, 257, 5.0, (1, 1)), (100, 768, 7.0, (1, 1)),
    (100, 769, 7.0, (1, 1)), (100, 1536, 7.0, (1, 1)), (100, 1537, 7.0, (9, 10)), (100, 3072, 5.5, (1, 1)),
    (100, 3073, 7.0, (1, 1)),
    (2500, 2, 11.0, (1, 1)),  # sixteen wavefronts
    (2500, 30, 9.0, (1, 1)), (500, 257, 10.0, (1, 1)),  # many pilots per bucket
    (8150, 1, 7.0, (1, 1)), (8200, 2, 7.0, (1, 1)),  # around 8192 slots: whole seeds or parts of one
    (10_000, 3, 6.0, (9, 10)), (70_000, 2, 7.0, (1, 1)),  # no shifted bitmap
])
def test_images_equal_the_oracle(P, K, lam, alpha):
    keys = synth.u64_keys(P * K - (P // 3 if K > 1 else 0), 7 + K)
    got = _image(keys, binding.params(partition_size=P, lam=lam, alpha=alpha))
    want = oracle.build_u64(keys, oracle.params(partition_size=P, lam=lam, alpha=alpha), threads=8).image()
    assert np.array_equal(got, want)


@pytest.mark.parametrize("P,K,lam", [(500, 4096, 10.5), (500, 4097, 10.5), (500, 8192, 11.0), (500, 1600, 11.0)])
def test_many_pilots_per_bucket(P, K, lam):
    # the oracle takes minutes here: the one-wavefront search, asked for by its shape, is the reference
    keys = synth.u64_keys(P * K, K)
    prm = binding.params(partition_size=P, lam=lam)
    got = _image(keys, prm)
    before = binding.get_search_config()
    try:
        binding.set_search_config(waves_per_group=2)
        want = _image(keys, prm)
    finally:
        binding.set_search_config(**before)
    assert np.array_equal(got, want)


@pytest.mark.parametrize("P,K,lam", [(4000, 1792, 7.0), (4000, 1793, 7.0), (6500, 1400, 9.0), (20_000, 768, 7.0),
                                     (20_000, 1025, 7.0), (50_000, 520, 7.0)])
def test_teams_limited_by_lds(P, K, lam):
    # around the counts from which the LDS no longer holds every partition's team; reference as above
    keys = synth.u64_keys(P * K, K)
    prm = binding.params(partition_size=P, lam=lam)
    got = _image(keys, prm)
    before = binding.get_search_config()
    try:
        binding.set_search_config(waves_per_group=2)
        want = _image(keys, prm)
    finally:
        binding.set_search_config(**before)
    assert np.array_equal(got, want)


def test_batch_members_equal_the_oracle():
    # several MPHFs: pilots go to the members' encoder-major arrays
    sets = [synth.u64_keys(n, 50 + n) for n in (1, 700, 2500, 9001, 40_000)]
    hs = binding.build_batch_u64([torch.from_numpy(k.view(np.int64)).cuda() for k in sets], binding.params(lam=8.0))
    for k, h in zip(sets, hs):
        assert np.array_equal(h.serialize(), oracle.build_u64(k, oracle.params(lam=8.0)).image())


@pytest.mark.parametrize("where", [0, 1])
def test_duplicates_and_limits(where):
    keys = synth.u64_keys(5000, 3)
    with pytest.raises(binding.PhobicError) as e:
        _image(np.append(keys, keys[where]), binding.params(lam=9.0, pilot_limit=5000 if where else 0))
    assert e.value.code == binding.E_DUPLICATE
    with pytest.raises(binding.PhobicError) as e:
        _image(keys, binding.params(lam=9.0, pilot_limit=3))
    assert e.value.code == binding.E_PILOT_OVERFLOW
