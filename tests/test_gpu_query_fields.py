"""Lookups where the image's fields lie awkwardly: offset residues of more than 16 bits (a pair then spans
three 4-byte words), long unary runs (many empty buckets) that leave the first 128-bit window, one-word
sections, and value 0 of the unary stream.  Members and other keys against the oracle, alone and in one
multi-request call."""

import numpy as np
import pytest
import torch

import oracle
from paper_2404_18497_amd import binding, synth

pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).cuda()


def _lopsided(n, seed):
    # keys of the lower 90% of the hash range only: the offsets are up to n / 10 from their expectation
    keys = synth.u64_keys(n, seed)
    hi, _ = oracle.hash_u64(keys, 0x5EED)
    return keys[hi < np.uint64((9 << 64) // 10)]


CASES = [
    ("wide offsets", dict(lam=6.0, partition_size=2000), lambda: _lopsided(900_000, 1)),
    ("wide offsets, mixed", dict(lam=6.0, partition_size=2000, n_compact=16), lambda: _lopsided(900_000, 2)),
    ("wide offsets, compact", dict(lam=6.0, partition_size=2000, coding="compact"), lambda: _lopsided(900_000, 3)),
    ("wide offsets, alpha", dict(lam=6.0, partition_size=2000, alpha=(9, 10)), lambda: _lopsided(900_000, 4)),
    ("many buckets", dict(lam=2.2, partition_size=2500), lambda: synth.u64_keys(30_000, 5)),
    ("few values", dict(lam=10.0, partition_size=40), lambda: synth.u64_keys(37, 6)),
    ("one key", dict(lam=1.0, partition_size=1), lambda: synth.u64_keys(1, 7)),
    ("small partitions", dict(lam=5.0, partition_size=60), lambda: synth.u64_keys(50_000, 8)),
]


def test_positions_equal_the_oracle():
    hs, ks, wants = [], [], []
    for name, kw, make in CASES:
        keys = make()
        prm = binding.params(**kw)
        rkw = dict(kw)
        r = oracle.build_u64(keys, oracle.params(**rkw), threads=8)
        q = np.concatenate([keys, synth.u64_keys(1001, 99)])
        h = binding.build_u64(_dev(keys), prm)
        want = r.query_u64(q)
        assert np.array_equal(h.query_u64(_dev(q)).cpu().numpy().view(np.uint64), want), name
        hs.append(h)
        ks.append(_dev(q))
        wants.append(want)
    outs = [torch.empty_like(k) for k in ks]
    binding.query_multi_u64(hs, ks, outs)
    for (name, _, _), o, want in zip(CASES, outs, wants):
        assert np.array_equal(o.cpu().numpy().view(np.uint64), want), name


@pytest.mark.parametrize("kw,n", [(dict(lam=7.0), 100_000), (dict(lam=5.0, coding="compact"), 30_000),
                                  (dict(lam=2.0, n_compact=16), 30_000), (dict(lam=7.0, alpha=(9, 10)), 30_000),
                                  (dict(lam=6.0, partition_size=9000), 40_000), (dict(lam=7.0), 0)])
def test_counts_around_the_kernels_line(kw, n):
    # one lookup per thread up to 2^19 of them, two above; nothing is written past the last one
    keys = synth.u64_keys(n, 11)
    r = oracle.build_u64(keys, oracle.params(**kw), threads=8)
    h = binding.build_u64(_dev(keys), binding.params(**kw))
    q = np.resize(np.concatenate([keys, synth.u64_keys(1001, 98)]), (1 << 19) + 1)
    want, dq = r.query_u64(q), _dev(q)
    for count in (1, 63, 64, 255, 256, 257, 1025, (1 << 19) - 1, 1 << 19, (1 << 19) + 1):
        out = torch.full((len(q) + 8,), -7, dtype=torch.int64, device="cuda")
        h.query_u64(dq[:count], out=out[:count])
        got = out.cpu().numpy()
        assert np.array_equal(got[:count].view(np.uint64), want[:count]) and (got[count:] == -7).all(), count


def test_counts_around_the_staged_kernels_line():
    # two lookups per thread up to 2^24 of them, four above
    keys = synth.u64_keys(30_000, 12)
    for kw in (dict(lam=7.0), dict(lam=6.0, partition_size=9000)):
        h = binding.build_u64(_dev(keys), binding.params(**kw))
        want = oracle.build_u64(keys, oracle.params(**kw)).query_u64(keys)
        dq, dw = _dev(keys).repeat(560)[:(1 << 24) + 1], _dev(want).repeat(560)[:(1 << 24) + 1]
        for count in ((1 << 19) + 511, (1 << 19) + 257, 1 << 24, (1 << 24) + 1):
            out = torch.full((len(dq) + 8,), -7, dtype=torch.int64, device="cuda")
            h.query_u64(dq[:count], out=out[:count])
            assert torch.equal(out[:count], dw[:count]) and bool((out[count:] == -7).all()), count
