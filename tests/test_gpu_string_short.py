"""Strings of 1 to 3 bytes, the shortest that the word reader masks, at every start modulo 8 (one word, or two
where the string begins in the last bytes of the first): images and positions equal the oracle's."""

import numpy as np
import pytest
import torch

import oracle
from paper_2404_18497_amd import binding

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lead", range(8))
def test_one_to_three_bytes(lead):
    rng = np.random.default_rng(40 + lead)
    words = [int(v).to_bytes(k, "little") for k, m in ((1, 200), (2, 400), (3, 400))
             for v in rng.choice(256 ** k, m, replace=False)]
    words = [words[i] for i in rng.permutation(len(words))]
    offs = np.concatenate([[lead], lead + np.cumsum([len(w) for w in words])]).astype(np.uint64)
    data = np.frombuffer(bytes(lead) + b"".join(words), dtype=np.uint8).copy()
    d, o = torch.from_numpy(data).cuda(), torch.from_numpy(offs.view(np.int64)).cuda()
    h = binding.build_str(d, o, binding.params(lam=5.0, partition_size=500))
    r = oracle.build_str(data, offs, oracle.params(lam=5.0, partition_size=500))
    assert np.array_equal(h.serialize(), r.image())
    pos = h.query_str(d, o).cpu().numpy().view(np.uint64)
    assert np.array_equal(pos, r.query_str(data, offs))
    assert np.array_equal(np.sort(pos), np.arange(len(words), dtype=np.uint64))
