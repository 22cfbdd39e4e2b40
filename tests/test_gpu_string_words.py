"""String hashing on the device at every length from 0 to 42 bytes and every start modulo 8, with the last
string ending on the buffer's last byte: images and positions equal the oracle's."""

import numpy as np
import pytest
import torch

import oracle
from paper_2404_18497_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lead", range(8))
def test_lengths_and_alignments(lead):
    rng = np.random.default_rng(11 + lead)
    lens = np.concatenate([[0], rng.permutation(np.repeat(np.arange(4, 43), 40))])
    offs = np.concatenate([[lead], lead + np.cumsum(lens)]).astype(np.uint64)
    data = rng.integers(0, 256, int(offs[-1]), dtype=np.uint8)
    d, o = torch.from_numpy(data).cuda(), torch.from_numpy(offs.view(np.int64)).cuda()
    h = binding.build_str(d, o, binding.params(lam=5.0, partition_size=500))
    r = oracle.build_str(data, offs, oracle.params(lam=5.0, partition_size=500))
    assert np.array_equal(h.serialize(), r.image())
    pos = h.query_str(d, o).cpu().numpy().view(np.uint64)
    assert np.array_equal(np.sort(pos), np.arange(lens.size, dtype=np.uint64))
    assert np.array_equal(pos, r.query_str(data, offs))
