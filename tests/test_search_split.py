"""Workgroups of the resident search: they wait for each other, so all of them need a place at the same time, also on a
partition of the device with a few CUs; on the whole device the split by blocks decides."""
import os
import shutil
import subprocess

import pytest

from paper_2602_17698_amd import build

CASES = [(N, step, cus) for N in (1, 2048, 2049, 65536, 65537, 430080, 524288, 524289, 2**21, 3147776, 2**23, 2**24)
         for step in (0, 1) for cus in (1, 2, 8, 32, 64, 128, 256)]


@pytest.fixture(scope="module")
def wgs(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("needs g++")
    d = tmp_path_factory.mktemp("split")
    (d / "main.cpp").write_text('#include <stdio.h>\n#include "alloc_split.hpp"\nint main() { long long n; int s, c; while '
                                '(scanf("%lld %d %d", &n, &s, &c) == 3) printf("%u\\n", sbits::search_wgs(n, s != 0, c)); }\n')
    exe = str(d / "split")
    subprocess.check_call([cxx, "-std=c++17", "-I" + build.CSRC, str(d / "main.cpp"), "-o", exe])
    out = subprocess.run([exe], input="\n".join("%d %d %d" % c for c in CASES), stdout=subprocess.PIPE, text=True, check=True).stdout
    return dict(zip(CASES, map(int, out.split())))


def test_all_workgroups_have_a_place_twice_over(wgs):
    for (N, step, cus), g in wgs.items():
        assert 1 <= g <= max(1, cus // 2) * (2 if step else 1), (N, step, cus, g)
        assert g <= (N + 2047) // 2048


def test_the_whole_device_is_split_by_blocks(wgs):
    want = {1: 1, 2048: 1, 2049: 2, 65536: 32, 65537: 17, 430080: 105, 524288: 128, 524289: 128}
    for N, g in want.items():
        assert wgs[N, 0, 256] == wgs[N, 1, 256] == g
    assert wgs[2**24, 0, 256] == 128 and wgs[2**24, 1, 256] == 256 and wgs[3147776, 1, 256] == 192 and wgs[2**21, 1, 256] == 128
