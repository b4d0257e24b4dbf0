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


def test_the_marshalling_module_is_this_interpreters_own():
    """Its name carries the ABI it was built for, so that another interpreter on the same tree does not load it."""
    import importlib.machinery
    import sysconfig
    from paper_2602_03152_amd import binding as fb
    tag = sysconfig.get_config_var("EXT_SUFFIX")
    assert tag != ".so" and tag == importlib.machinery.EXTENSION_SUFFIXES[0]
    assert B.PYCALL.endswith("_pycall" + tag) and os.path.samefile(fb._pycall.__file__, B.PYCALL)
    assert not os.path.exists(B.PYCALL_UNTAGGED)
