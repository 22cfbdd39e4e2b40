"""The checks of a loaded image, run on the CPU with every read of the device's part counted and checked.

`tests/emu/image_check_emu.cpp` compiles the library's image_check.h with g++ and AddressSanitizer.  The
images are the oracle's; whatever their words say, the device's part reads inside the image, and accepts
only what the host's check accepts.
"""

import os
import shutil
import subprocess

import numpy as np
import pytest

import oracle
from paper_2404_18497_amd import synth
from synth_images import long_gap, swapped_select

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
HEADER = 24
KINDS = {"rice": {}, "remap": dict(alpha=(99, 100)), "compact": dict(coding="compact"), "mixed": dict(n_compact=64)}


@pytest.fixture(scope="module")
def emu(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    out = str(tmp_path_factory.mktemp("image") / "image_check_emu")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address", "-Wno-attributes", "-I", os.path.join(HERE, "emu"),
           "-I", os.path.join(ROOT, "include"), "-I", os.path.join(ROOT, "paper_2404_18497_amd", "csrc"),
           "-x", "c++", os.path.join(HERE, "emu", "image_check_emu.cpp"), "-o", out]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return out


@pytest.fixture(scope="module")
def images():
    keys = synth.u64_keys(60_000, 5)
    return {k: oracle.build_u64(keys, oracle.params(lam=5.0, **kw), threads=8).image() for k, kw in KINDS.items()}


def _check(emu, tmp_path, first, uploaded=None, threads=4096):
    a, b = str(tmp_path / "a"), str(tmp_path / "b")
    first.tofile(a)
    (first if uploaded is None else uploaded).tofile(b)
    r = subprocess.run([emu, str(threads), a, b], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-4000:]
    keys = ("header", "fit", "bad", "host", "most", "all", "outside", "device")
    return dict(zip(keys, map(int, r.stdout.split())))


@pytest.mark.parametrize("kind", KINDS)
def test_header_words(emu, images, tmp_path, kind):
    # every header word altered: refused, or checked without a read outside the image
    img = images[kind]
    good = _check(emu, tmp_path, img)
    assert good["header"] and good["fit"] and good["bad"] == 0 and good["host"] and good["outside"] == 0
    for word in range(HEADER):
        v = int(img[word])
        for x in {0, 1, v + 1, v - 1, 2 * v, v ^ (1 << 20), v ^ (1 << 40), v ^ (1 << 63), (1 << 64) - 1} - {v}:
            bad = img.copy()
            bad[word] = np.uint64(x & (1 << 64) - 1)
            r = _check(emu, tmp_path, bad)
            assert r["outside"] == 0, (word, x)
            assert not (r["fit"] and r["bad"] == 0) or r["host"], (word, x)


@pytest.mark.parametrize("kind", KINDS)
def test_header_is_read_once(emu, images, tmp_path, kind):
    # the caller's memory changes after its header was checked: the sections are still found by the checked one
    img = images[kind]
    up = img.copy()
    up[:HEADER] = np.uint64(0x0123456789ABCDEF)
    r = _check(emu, tmp_path, img, up)
    assert r["outside"] == 0 and r["fit"] and r["bad"] == 0 and r["host"]


def test_select_entries_out_of_order(emu, tmp_path):
    # refused, and no thread walks the stream for it: a thread reads a segment's share of it at most
    img = oracle.build_u64(synth.u64_keys(400_000, 6), oracle.params(lam=5.0), threads=8).image()
    nsel = int(img[17] - img[16]) - 1
    good = _check(emu, tmp_path, img)
    assert good["bad"] == 0 and nsel < 4096
    r = _check(emu, tmp_path, swapped_select(img))
    assert r["bad"] and not r["host"] and r["outside"] == 0
    assert r["most"] <= 2 * 256 and r["all"] <= 2 * good["all"]


@pytest.mark.parametrize("at", [0, 1, 300])
def test_long_gaps_are_left_to_the_host(emu, images, tmp_path, at):
    # a gap of 200 words stays within the words a thread reads of a segment, one of 2000 does not
    img = long_gap(images["rice"], at, 200)
    r = _check(emu, tmp_path, img)
    assert r["fit"] and r["host"] and r["bad"] == 0
    r = _check(emu, tmp_path, long_gap(images["rice"], at, 2000))
    assert r["fit"] and r["host"] and r["bad"] and r["most"] <= 2 * 256 and r["outside"] == 0


@pytest.mark.parametrize("n,kw,device", [
    (300_000, dict(coding="compact"), False),  # the host reads the offsets and encoders alone
    (300_000, {}, False), (700_000, {}, True),  # 10 000 and 22 000 words with a unary stream
    (300_000, dict(n_compact=490), False),
    (200_000, dict(coding="compact", alpha=(9, 10)), False), (500_000, dict(coding="compact", alpha=(9, 10)), True),
])
def test_the_checker_follows_the_work(emu, tmp_path, n, kw, device):
    img = oracle.build_u64(synth.u64_keys(n, 7), oracle.params(lam=5.0, **kw), threads=8).image()
    assert img.size > 1 << 12
    assert _check(emu, tmp_path, img)["device"] == device
