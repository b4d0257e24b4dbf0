"""An FC's workgroup looks for the full head's set once, a bounded number of times, and then goes by the state word: one waiting loop in each of the
calibration's kernels, and no way from one into another."""
import os
import re
import shutil

import pytest

from paper_2602_03152_amd import build as B

KERNEL = re.compile(r"^(_ZN4fasa\w*calib_\w*):[^\n]*\n(.*?)^\t?\.Lfunc_end", re.M | re.S)


@pytest.mark.skipif(shutil.which(B.HIPCC) is None and not os.path.exists(B.HIPCC), reason="no hipcc")
def test_an_fc_waits_in_one_place(tmp_path):
    out = os.path.join(str(tmp_path), "calib_dev.s")
    flags = [f for f in B.FLAGS if f != "-fPIC"]
    B._run([B.HIPCC, *flags, "--cuda-device-only", "-S", os.path.join(B.CSRC, "calib.hip"), "-o", out], False)
    waits = {m.group(1): len(re.findall(r"^\ts_sleep\b", m.group(2), re.M)) for m in KERNEL.finditer(open(out).read())}
    waiting = {n: c for n, c in waits.items() if "calib_kernel" in n or "calib_fc_kernel" in n}
    assert sum("calib_kernel" in n for n in waiting) == 2 and sum("calib_fc_kernel" in n for n in waiting) >= 6, sorted(waits)
    assert set(waiting.values()) == {1}, waiting
    assert not any(c for n, c in waits.items() if n not in waiting), waits
