"""Kernels that have no registers to spare keep what they need in them: what the compiler says of spills (hipcc, no GPU)."""
from tests import asm_util as A


def test_searches_for_the_nearest_centre_use_no_scratch():
    found = {k: v for k, v in A.spills("pact_centres.hip").items() if "nearest_centre_kernel" in k}
    assert len(found) >= 10
    for name, (vgprs, scratch, _) in found.items():
        assert vgprs == 0 and scratch == 0, name
