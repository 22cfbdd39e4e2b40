"""Image checks on load, on both sides of the size from which the sections are checked on the device
(2^13 words): single flipped bits all over an image are accepted or refused exactly as a plain numpy
reading of the format says, for minimal, non-minimal, Compact and mixed images."""

import numpy as np
import pytest
import torch

import oracle
from paper_2404_18497_amd import binding, synth

pytestmark = pytest.mark.gpu


def _fields(w, sec, count, width):
    if width == 0:
        return np.zeros(count, dtype=np.uint64)
    pos = np.arange(count, dtype=np.uint64) * np.uint64(width)
    i, sh = (pos >> np.uint64(6)).astype(np.int64) + sec, pos & np.uint64(63)
    hi = np.where(sh > 0, w[i + 1] << ((np.uint64(64) - sh) & np.uint64(63)), 0).astype(np.uint64)
    return ((w[i] >> sh) | hi) & np.uint64((1 << width) - 1)


def _sections_ok(w):
    n, K, B, total, c = int(w[1]), int(w[2]), int(w[3]), int(w[9]), int(w[23])
    so, se, sd, su, ss, sr = (int(x) for x in w[12:18])
    j = np.arange(K + 1, dtype=object)
    dmin = int(w[10]) - (1 << 64 if int(w[10]) >> 63 else 0)
    off = [(int(x) * int(w[22]) >> 32) + dmin + int(f) for x, f in zip(j, _fields(w, so, K + 1, int(w[11])))]
    if off[0] != 0 or off[-1] != total or any(x > y for x, y in zip(off, off[1:])):
        return False
    for e in w[se:se + B]:
        if int(e) & 255 > 32 or (int(e) >> 8) + (int(e) & 255) * K > (su - sd - 1) * 64:
            return False
    if int(w[7]) & 255 == 0:
        U = (int(w[20]) + 63) // 64
        ones = np.nonzero(np.unpackbits(w[su:su + U].view(np.uint8), bitorder="little"))[0]
        if ones.size != K * (B - c) or w[ss - 1] != 0:
            return False
        for s in range((ones.size + 255) // 256):
            a = int(ones[256 * s])
            want = a
            for k in (1, 2, 3):
                if 256 * s + 64 * k < ones.size:
                    want |= min(int(ones[256 * s + 64 * k]) - a, 1023) << (32 + 10 * (k - 1))
            if int(w[ss + s]) != want:
                return False
    return total == n or bool((_fields(w, sr, total - n, int(w[18])) < np.uint64(n)).all())


@pytest.mark.parametrize("n", [20_000, 700_000])
@pytest.mark.parametrize("kw", [dict(), dict(alpha=(99, 100)), dict(coding="compact"), dict(n_compact=64)])
def test_flipped_bits(n, kw):
    keys = torch.from_numpy(synth.u64_keys(n, 5).view(np.int64)).cuda()
    h = binding.build_u64(keys, binding.params(lam=7.0, **kw))
    img = h.serialize()
    assert (img.size < 1 << 13) == (n == 20_000)
    rng = np.random.default_rng(n)
    secs = [int(x) for x in img[12:18]] + [img.size]
    words = [rng.integers(a, b, 3) for a, b in zip(secs, secs[1:]) if b > a]
    words = [int(x) for ws in words for x in ws] + [b - 1 for b in secs[1:]] + secs[:-1]
    accepted = 0
    for word in words:
        bad = img.copy()
        bad[min(word, img.size - 1)] ^= np.uint64(1) << np.uint64(rng.integers(0, 64))
        if _sections_ok(bad):
            accepted += 1
            binding.deserialize(bad).close()
        else:
            with pytest.raises(binding.PhobicError) as e:
                binding.deserialize(bad)
            assert e.value.code == binding.E_FORMAT, word
    assert accepted < len(words)
    again = binding.deserialize(img)
    assert np.array_equal(again.serialize(), img)
    assert torch.equal(again.query_u64(keys), h.query_u64(keys))
