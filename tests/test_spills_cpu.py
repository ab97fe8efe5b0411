"""Kernels that have no registers to spare keep what they need in them: what the compiler says of spills (hipcc, no GPU)."""
from tests import asm_util as A


def test_searches_for_the_nearest_centre_use_no_scratch():
    found = {k: v for k, v in A.spills("pact_centres.hip").items() if "nearest_centre_kernel" in k}
    assert len(found) >= 10
    for name, (vgprs, scratch, _) in found.items():
        assert vgprs == 0 and scratch == 0, name


def test_logits_spill_nothing():
    found = {k: v for k, v in A.spills("pact_euti.hip").items() if "score_logits_kernel" in k}
    assert len(found) == 6                                          # two types, three ways
    for name, spilled in found.items():
        assert spilled == (0, 0, 0), name
