"""The bucket sort of wide partitions: images equal the oracle's where its layout changes (start offsets in
LDS up to 16384 buckets, in global memory above) and over its sort sizes, including partitions of a few keys."""

import numpy as np
import pytest
import torch

import oracle
from paper_2404_18497_amd import binding, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("P,n,lam", [
    (8_400, 25_000, 9.0),      # 1024 sort keys
    (16_000, 40_000, 7.0),     # 4096
    (50_000, 101_000, 6.5),    # 8192
    (81_920, 81_920, 5.0),     # 16384 buckets
    (81_925, 170_000, 5.0),    # 16385
    (120_000, 33, 4.0), (120_000, 0, 4.0), (120_000, 250_000, 4.5),
])
def test_images_equal_the_oracle(P, n, lam):
    keys = synth.u64_keys(n, 3)
    h = binding.build_u64(torch.from_numpy(keys.view(np.int64)).cuda(), binding.params(partition_size=P, lam=lam))
    want = oracle.build_u64(keys, oracle.params(partition_size=P, lam=lam), threads=8).image()
    assert np.array_equal(h.serialize(), want)
