"""The build's check of the waits that count loads (the product of many rows): it passes on this build's object, and refuses
listings in which a step has too few loads, or its loads in another order."""
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


def test_the_loads_of_every_step_are_as_many_as_the_waits_count(listing):
    assert build.check_counted_waits(listing) == 6


@pytest.mark.parametrize("change", ["scalar", "merged", "late", "moved"])
def test_a_step_with_other_loads_is_refused(listing, change):
    at = listing.index("mp_gemm_wide_kernelILi128ELi4ELi4E")
    wait = re.compile(r"s_waitcnt vmcnt\(22\) lgkmcnt\(0\)").search(listing, at).end()
    if change == "scalar":                                  # the uniform offset through the scalar cache
        bad = listing[:wait] + listing[wait:].replace("global_load_dwordx2", "s_load_dwordx2", 1)
    elif change == "merged":                                # two scales in one load
        bad = listing[:wait] + re.sub(r"\n[^\n]*global_load_dword v[^\n]*", "", listing[wait:], count=1)
    elif change == "late":                                  # a load of x behind the others
        loads = list(re.finditer(r"\n[^\n]*buffer_load_dwordx4 v\d+, [^\n]*lds[^\n]*", listing[wait:wait + 20000]))
        offset = re.compile(r"\n[^\n]*global_load_dwordx2[^\n]*").search(listing, wait).end()
        cut = (wait + loads[0].start(), wait + loads[0].end())
        bad = listing[:cut[0]] + listing[cut[1]:offset] + listing[cut[0]:cut[1]] + listing[offset:]
    else:                                                   # another wait than the kernel's own
        bad = listing[:wait].replace("vmcnt(22) lgkmcnt(0)", "vmcnt(23) lgkmcnt(0)") + listing[wait:]
    with pytest.raises(RuntimeError):
        build.check_counted_waits(bad)
