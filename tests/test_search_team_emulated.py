"""The team search's logic (several wavefronts per partition) run on the CPU against the oracle.

`tests/emu/search_team_emu.cpp` compiles `search_team` with g++ and AddressSanitizer and interleaves
the wavefronts of a team at random (several seeds per case); a wavefront that leaves before a barrier
the others wait at is reported.  The cases cover units of whole seeds and units of a part of a seed
(more than 128 windows of 64 displacements), position scratch with and without a bit per slot (8192),
claim tables smaller than the table, packed and big buckets, one bucket per wavefront and fewer
buckets than wavefronts, non-minimal tables, and the duplicate and pilot-limit errors.
"""

import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle
from paper_2404_18497_amd import binding
from test_search_emulated import HERE, ROOT, SEARCH_SRC, _mix_b, _partition


@pytest.fixture(scope="module")
def team(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    out = str(tmp_path_factory.mktemp("team") / "search_team_emu")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address", "-fno-omit-frame-pointer", "-Wno-attributes",
           "-I", os.path.join(HERE, "emu"), "-I", os.path.join(ROOT, "include"),
           "-I", os.path.join(ROOT, "paper_2404_18497_amd", "csrc"), f'-DSEARCH_SRC="{SEARCH_SRC}"',
           "-x", "c++", os.path.join(HERE, "emu", "search_team_emu.cpp"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return out


def _input(path, hi, lo, m, prm, limit):
    B = oracle.num_buckets(prm.partition_size, prm.lambda_)
    T = oracle.bucket_table(prm.lambda_, prm.partition_size, (prm.alpha_num, prm.alpha_den))
    b = oracle.buckets(lo, T, B)
    sz = np.bincount(b, minlength=B)
    order = sorted((i for i in range(B) if sz[i]), key=lambda i: (-int(sz[i]), -i))
    fps = [int(lo[k]) ^ _mix_b(int(hi[k])) for i in order for k in np.nonzero(b == i)[0]]
    with open(path, "wb") as f:
        np.array([m, limit, B, len(fps), len(order)], dtype=np.uint64).tofile(f)
        np.array(fps, dtype=np.uint64).tofile(f)
        np.array([(int(sz[i]) << 16) | i for i in order], dtype=np.uint32).tofile(f)
    return B


def _run(team, tmp_path, waves, seed, hi, lo, m, prm, limit=0xFFFFFFFF):
    fi, fo = str(tmp_path / "in"), str(tmp_path / "out")
    B = _input(fi, hi, lo, m, prm, limit)
    r = subprocess.run([team, str(waves), str(seed), fi, fo], capture_output=True, text=True,
                       timeout=600)
    assert r.returncode == 0, r.stderr[-4000:]
    out = np.fromfile(fo, dtype=np.uint32)
    return out[:B], int(out[B])


@pytest.mark.parametrize("P,n,lam,waves", [
    (2500, 2500, 5.0, 8), (2500, 2500, 7.0, 2), (2500, 2500, 9.0, 16), (2500, 2500, 11.0, 4),
    (2500, 1000, 7.0, 8),  # fewer keys than the partition size: nearly all buckets of a few keys
    (64, 64, 7.0, 16), (10, 5, 2.0, 16), (1, 1, 1.0, 4),  # fewer buckets than wavefronts
    (8128, 8128, 7.0, 4),  # 128 windows, a claim table smaller than the table
    (10_000, 10_000, 6.0, 4),   # more: parts of a seed, a scratch smaller than the table
    (66_000, 66_000, 8.0, 2),  # no shifted bitmap
])
def test_team_matches_oracle(team, tmp_path, P, n, lam, waves):
    prm = oracle.params(partition_size=P, lam=lam)
    hi, lo = _partition(n, lam, 0, nparts=1)
    want, _ = oracle.search_partition(hi, lo, hi.size, prm)
    for seed in (1, 2) if n < 10_000 else (1,):
        got, err = _run(team, tmp_path, waves, seed, hi, lo, hi.size, prm)
        assert err == 0 and np.array_equal(got, want), seed


def test_team_nonminimal_table(team, tmp_path):
    prm = oracle.params(lam=7.0, alpha=(9, 10))
    hi, lo = _partition(2500, 7.0, 0)
    m = -(-hi.size * 10 // 9)
    want, _ = oracle.search_partition(hi, lo, m, prm)
    got, err = _run(team, tmp_path, 16, 3, hi, lo, m, prm)
    assert err == 0 and np.array_equal(got, want)


@pytest.mark.parametrize("place", ["anywhere", "largest bucket"])
def test_team_duplicate_key(team, tmp_path, place):
    prm = oracle.params(lam=7.0)
    hi, lo = _partition(2500, 7.0, 0, dup=place == "anywhere")
    if place == "largest bucket":
        b = oracle.buckets(lo, oracle.bucket_table(7.0, 2500), oracle.num_buckets(2500, 7.0))
        k = np.nonzero(b == np.argmax(np.bincount(b)))[0][0]
        hi, lo = np.append(hi, hi[k]), np.append(lo, lo[k])
    for seed in (1, 2):
        _, err = _run(team, tmp_path, 16, seed, hi, lo, hi.size, prm)
        assert err == 1 << binding.E_DUPLICATE


@pytest.mark.parametrize("lam,j", [(9.0, 1)])
def test_team_pilot_limit(team, tmp_path, lam, j):
    # as the one-wavefront search: limits around the largest pilot of a small bucket, and one so low
    # that only displacements of seed 0 remain
    hi, lo = _partition(2500, lam, j)
    prm = oracle.params(lam=lam)
    pil, _ = oracle.search_partition(hi, lo, hi.size, prm)
    B = oracle.num_buckets(2500, lam)
    sz = np.bincount(oracle.buckets(lo, oracle.bucket_table(lam, 2500), B), minlength=B)
    top = int(pil[(sz >= 2) & (sz <= 24)].max())
    for limit in (top - 1, top, top + 1, hi.size // 2):
        p = oracle.params(lam=lam, pilot_limit=limit)
        try:
            want, _ = oracle.search_partition(hi, lo, hi.size, p)
            code = 0
        except oracle.OracleError as e:
            want, code = None, e.code
        got, err = _run(team, tmp_path, 4, limit, hi, lo, hi.size, p, limit)
        if code == 0:
            assert err == 0 and np.array_equal(got, want), limit
        else:
            assert err == 1 << code, (limit, err)


def test_team_duplicate_after_overflow(team, tmp_path):
    # a pilot limit that fails early and a duplicate in the smallest bucket: the duplicate is reported
    prm = oracle.params(lam=9.0, pilot_limit=3)
    hi, lo = _partition(2500, 9.0, 0)
    b = oracle.buckets(lo, oracle.bucket_table(9.0, 2500), oracle.num_buckets(2500, 9.0))
    cnt = np.bincount(b)
    k = np.nonzero(b == np.nonzero(cnt == cnt[cnt > 0].min())[0][0])[0][0]
    hi, lo = np.append(hi, hi[k]), np.append(lo, lo[k])
    _, err = _run(team, tmp_path, 8, 5, hi, lo, hi.size, prm, 3)
    assert err == 1 << binding.E_DUPLICATE
