"""The build's own rules, on the host."""
import os
import re

from paper_2602_03152_amd import build as B


def test_every_source_that_merges_partials_has_its_assembly_checked():
    """The merge's hand-placed loads are safe only as checked: no source that calls it, itself or by a header, is left out."""
    read = lambda name: open(os.path.join(B.CSRC, name)).read()
    calls = lambda text: re.search(r"\b(combine_row|agent_b128_issue)\s*[<(]", re.sub(r"//.*", "", text))
    assert [s for s in B.SOURCES if calls(read(s))] == B.ASM_CHECKED and "offload.hip" in B.ASM_CHECKED
    # the one header that may hold such a call is the one that defines them
    assert [h for h in os.listdir(B.CSRC) if h.endswith(".h") and calls(read(h))] == ["attend_common.h"]
