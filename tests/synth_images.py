"""Images altered in ways that single flipped bits do not reach, for the tests of loading."""

import numpy as np

N_HEADER = 24
KK, KB, SEC_UNARY, SEC_SEL, SEC_REMAP, UBITS, WORDS, NCOMPACT = 2, 3, 15, 16, 17, 20, 21, 23


def swapped_select(img):
    """Every odd select entry names the last one of the unary stream, so that the entries do not ascend."""
    bad = img.copy()
    su, ss, sr = (int(bad[x]) for x in (SEC_UNARY, SEC_SEL, SEC_REMAP))
    ones = np.nonzero(np.unpackbits(bad[su:ss - 1].view(np.uint8), bitorder="little"))[0]
    bad[ss + 1:sr - 1:2] = np.uint64(ones[-1])
    return bad


def long_gap(img, at, words):
    """`words` zero words in the unary stream before its word `at`, and the select entries that fit it: a
    consistent image (whose positions mean nothing)."""
    su, ss, sr = (int(img[x]) for x in (SEC_UNARY, SEC_SEL, SEC_REMAP))
    un = np.concatenate([img[su:su + at], np.zeros(words, dtype=np.uint64), img[su + at:ss]])
    ones = np.nonzero(np.unpackbits(un.view(np.uint8), bitorder="little"))[0].astype(np.int64)
    sel = np.zeros(sr - ss, dtype=np.uint64)
    for s in range(sr - ss - 1):
        a = int(ones[256 * s])
        e = a
        for k in (1, 2, 3):
            if 256 * s + 64 * k < ones.size:
                e |= min(int(ones[256 * s + 64 * k]) - a, 1023) << (32 + 10 * (k - 1))
        sel[s] = np.uint64(e)
    out = np.concatenate([img[:su], un, sel, img[sr:]])
    out[UBITS] += np.uint64(64 * words)
    out[[SEC_SEL, SEC_REMAP, WORDS]] += np.uint64(words)
    return out
