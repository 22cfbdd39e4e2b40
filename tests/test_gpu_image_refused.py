"""Loading images that are wrong, or merely unusual, in more than one bit, at a size whose sections the
device checks."""

import numpy as np
import pytest
import torch

from paper_2404_18497_amd import binding, synth
from synth_images import long_gap, swapped_select

pytestmark = pytest.mark.gpu
N = 2_000_000


@pytest.fixture(scope="module")
def image():
    keys = torch.from_numpy(synth.u64_keys(N, 8).view(np.int64)).cuda()
    return binding.build_u64(keys, binding.params(lam=7.0)).serialize()


def _refused(img):
    with pytest.raises(binding.PhobicError) as e:
        binding.deserialize(img)
    return e.value.code == binding.E_FORMAT


def test_select_entries_out_of_order(image):
    assert _refused(swapped_select(image))


def test_long_gap_is_accepted(image):
    img = long_gap(image, 1000, 2000)
    assert np.array_equal(binding.deserialize(img).serialize(), img)


@pytest.mark.parametrize("word", [1, 2, 3, 9, 11, 12, 13, 14, 15, 16, 17, 19, 20, 21, 23])
def test_header_words(image, word):
    # n, K, B, total, offset width, section starts, remap entries, unary bits, words, Compact encoders
    v = int(image[word])
    for x in (v + 64, v - 64, v + (1 << 40), (1 << 64) - 1):
        bad = image.copy()
        bad[word] = np.uint64(x & (1 << 64) - 1)
        assert _refused(bad), (word, x)
