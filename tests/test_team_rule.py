"""The launch rule of the search gives teams of wavefronts where they were measured to gain, and one
wavefront per partition where teams were measured slower (the times stand beside the rule)."""

import os
import shutil
import subprocess

import pytest

import oracle
from test_search_emulated import HERE, ROOT, SEARCH_SRC

# (P, partitions, lambda): wavefronts per partition
CASES = {
    (2500, 1, 7.0): 8, (2500, 160, 12.0): 16, (2500, 520, 9.0): 8, (2500, 1000, 7.0): 4, (2500, 1400, 11.0): 8,
    (2500, 1700, 7.0): 4, (2500, 2200, 7.0): 1, (2500, 3000, 7.0): 1, (2500, 3072, 8.0): 1, (2500, 2200, 9.0): 4,
    (2500, 3072, 9.8): 4, (2500, 1536, 4.0): 1, (2500, 900, 4.0): 4, (2500, 1536, 3.0): 1, (1000, 2800, 7.0): 4,
    (1500, 3072, 7.0): 1, (1500, 2200, 7.0): 4, (3000, 1537, 7.0): 4, (3000, 1800, 7.0): 1, (4000, 1800, 7.0): 1,
    (5000, 1280, 7.0): 4, (5000, 1400, 7.0): 1, (5000, 1400, 9.0): 4, (6500, 1536, 5.0): 1,
    (2500, 6000, 10.9): 4, (3000, 6000, 10.9): 1, (3000, 4096, 10.9): 4, (3000, 12_000, 11.9): 1,
    (2500, 40_000, 7.0): 1, (20_000, 100, 7.0): 16,
}


def _largest_bucket(P, lam):
    B, T = oracle.num_buckets(P, lam), oracle.bucket_table(lam, P, (1, 1))
    k = 1 + next(i for i, t in enumerate(T[1:]) if int(t) * B >= 1 << 32)
    return P * k / (len(T) - 1)


@pytest.fixture(scope="module")
def rule(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path_factory.mktemp("rule") / "rule")
    cmd = ["g++", "-std=c++17", "-O1", "-Wno-attributes", "-I", os.path.join(HERE, "emu"),
           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2404_18497_amd", "csrc"),
           f'-DSEARCH_SRC="{SEARCH_SRC}"', "-x", "c++", os.path.join(HERE, "emu", "team_rule_emu.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]

    def run(cases):  # (P, partitions, lambda, load)
        lines = "".join("%g %d %g %g %d\n" % (P, K, lam, _largest_bucket(P, lam), load) for P, K, lam, load in cases)
        out = subprocess.run([exe], input=lines, capture_output=True, text=True, check=True).stdout.split()
        return list(map(int, out))

    return run


def test_measured_cases(rule):
    out = rule([(P, K, lam, K) for P, K, lam in CASES])
    assert dict(zip(CASES, out)) == CASES


def test_builds_beside_each_other(rule):
    # other builds in flight fill the device as more partitions would; alone, and where they leave it idle, teams
    assert rule([(2500, 1600, 7.0, 1600), (2500, 1600, 7.0, 4 * 1600), (2500, 80, 7.0, 8 * 80), (2500, 1, 7.0, 8)]) == [4, 1, 8, 8]
