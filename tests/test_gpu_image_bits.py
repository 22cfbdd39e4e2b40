"""Single flipped bits in images whose sections the device checks: each is accepted or refused as a plain
numpy reading of the format says."""

import numpy as np
import pytest
import torch

from paper_2404_18497_amd import binding, synth
from test_gpu_image_check import _sections_ok

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,kw", [(1_500_000, dict()), (1_200_000, dict(alpha=(99, 100))), (1_500_000, dict(n_compact=64)),
                                  (4_500_000, dict(coding="compact")),
                                  (600_000, dict(coding="compact", alpha=(9, 10)))])
def test_flipped_bits(n, kw):
    keys = torch.from_numpy(synth.u64_keys(n, 5).view(np.int64)).cuda()
    h = binding.build_u64(keys, binding.params(lam=7.0, **kw))
    img = h.serialize()
    rng = np.random.default_rng(n)
    secs = [int(x) for x in img[12:18]] + [img.size]
    words = [int(x) for a, b in zip(secs, secs[1:]) if b > a for x in rng.integers(a, b, 3)]
    words += [b - 1 for b in secs[1:]] + [a for a in secs[:-1] if a < img.size]
    for word in words:
        bad = img.copy()
        bad[word] ^= np.uint64(1) << np.uint64(rng.integers(0, 64))
        if _sections_ok(bad):
            binding.deserialize(bad).close()
        else:
            with pytest.raises(binding.PhobicError) as e:
                binding.deserialize(bad)
            assert e.value.code == binding.E_FORMAT, word
    again = binding.deserialize(img)
    assert np.array_equal(again.serialize(), img)
    assert torch.equal(again.query_u64(keys), h.query_u64(keys))
