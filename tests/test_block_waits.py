"""The build's check of the wait for the x of a block (the product of many rows): it passes on this build's object, and refuses
listings in which more or fewer loads are behind that x than the wait counts."""
import os
import re

import pytest

from paper_2602_17698_amd import build


@pytest.fixture(scope="module")
def listing():
    if not os.path.exists(build.HIPCC):
        pytest.skip("needs hipcc")
    obj = os.path.join(build.HERE, "_build", "mpgemm.o")
    if not os.path.exists(obj):
        build.build()
    return build.device_listing(obj)


def test_the_loads_behind_the_x_of_a_block_are_as_many_as_its_wait_counts(listing):
    assert build.check_block_waits(listing) == 20


@pytest.mark.parametrize("change", ["merged", "more", "other wait"])
def test_a_block_with_other_loads_is_refused(listing, change):
    at = listing.index("mp_gemm_many_kernelILi128ELi4ELi4ELi8ELb0E")
    wait = re.compile(r"s_waitcnt vmcnt\(16\)\s[^\n]*\n(?:(?!s_barrier|s_cbranch)[^\n]*\n){0,16}?\s*ds_read_b128").search(listing, at)
    scale = re.compile(r"\n[^\n]*global_load_dword v[^\n]*").search(listing, wait.end())
    if change == "merged":                                  # two scales in one load
        bad = listing[:scale.start()] + listing[scale.end():]
    elif change == "more":                                  # a load in the switch between the bitwidths
        bad = listing[:scale.start()] + listing[scale.start():scale.end()] + listing[scale.start():]
    else:
        bad = listing[:wait.start()] + "s_waitcnt vmcnt(17)" + listing[wait.start() + len("s_waitcnt vmcnt(16)"):]
    with pytest.raises(RuntimeError):
        build.check_block_waits(bad)
