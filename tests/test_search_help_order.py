"""Wavefronts of a team that talk to each other between two barriers do it through atomics.

In the search variant for many pilots per bucket, idle wavefronts wait in a loop for a word of the LDS
that another one writes.  A plain load there may be taken out of the loop (nothing in the loop changes
the word), and the wait would then never end, so the compiled form is checked: the word is read with
acquire and written with release at workgroup scope, and the helpers' best pilot is read atomically.
"""

import os
import re
import subprocess

import pytest

from paper_2404_18497_amd import build_lib


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(build_lib.hipcc()):
        pytest.skip("hipcc not available")
    src = next(s for s in build_lib.sources() if s.endswith("search.hip"))
    flags = [f for f in build_lib.FLAGS if f != "-shared"]
    r = subprocess.run([build_lib.hipcc(), *flags, "-I", build_lib.INCLUDE, "-I", os.path.dirname(src),
                        "--cuda-device-only", "-S", "-emit-llvm", src, "-o", "-"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    return {m.group(1): m.group(2)
            for m in re.finditer(r"^define amdgpu_kernel void @(\w+)\((.*?)^}", r.stdout, re.M | re.S)}


def test_help_words_are_atomic(kernels):
    many = [body for name, body in kernels.items() if "k_search_teamILb1ELb1ELb1E" in name]
    assert len(many) == 1
    lds = r"ptr addrspace\(3\) %\w+ syncscope\(\"workgroup\"\) "
    # rounds of big and of packed buckets: the wait and the look at further help, the ask, the last part
    # and the end, and the look for a pilot that a helper has found
    assert len(re.findall(r"load atomic i32, " + lds + "acquire", many[0])) >= 4
    assert len(re.findall(r"store atomic i32 \S+, " + lds + "release", many[0])) >= 6
    assert len(re.findall(r"load atomic i64, " + lds + "monotonic", many[0])) >= 2
