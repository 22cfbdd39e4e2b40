"""The benchmark names the kernel that its lookups and its search run on."""

import re

import pytest

import bench
from paper_2404_18497_amd import build_lib

DEFAULT = dict(waves_per_group=1, groups_per_cu=0, items_per_grab=1, teams=True)


def test_query_lines_are_the_library_s():
    src = open(next(s for s in build_lib.sources() if s.endswith("query.hip"))).read()
    few, mid = (1 << int(re.search(rf"constexpr uint64_t {k} = 1ull << (\d+);", src).group(1)) for k in ("kQFew", "kQMid"))
    enc = int(re.search(r"constexpr uint32_t kQEncLds = (\d+);", src).group(1))
    names = [bench.query_kernel_name(m, enc) for m in (1, few, few + 1, mid, mid + 1)]
    assert names == ["k_query_few", "k_query_few", "k_query_mid", "k_query_mid", "k_query_u64<true>"]
    assert bench.query_kernel_name(mid + 1, enc + 1) == "k_query_u64<false>"


@pytest.mark.parametrize("cfg,partitions,name", [
    (DEFAULT, 40_000, "k_search<1, false>"), (DEFAULT, 16_384, None), (DEFAULT, 1, None),
    (DEFAULT | dict(teams=False), 1, "k_search<1, false>"),
    (dict(waves_per_group=8, groups_per_cu=4, items_per_grab=1), 400, "k_search_persistent<8, false>"),
])
def test_search_kernel(cfg, partitions, name):
    assert bench.search_kernel_name(cfg, partitions, 256) == name
