"""bench.py's byte model knows every kernel of the paths it times (host logic only; no GPU)."""
import os
import re

import bench
from paper_2602_03152_amd import build as B
from paper_2602_03152_amd import workload as W


def _launched(source):
    """Kernel names a source launches or returns for launching ("fasa_..." literals)."""
    return set(re.findall(r'"(fasa_[a-z_]+)"', open(os.path.join(B.CSRC, source)).read()))


def test_every_kernel_of_the_step_has_a_byte_count():
    step = set().union(*(_launched(s) for s in ("score.hip", "topk.hip", "attend.hip", "fused.hip", "step.hip")))
    step -= {"fasa_hist", "fasa_ws_clear"}              # fasa_topk on its own, workspace initialisation
    assert step and "fasa_step" in step and "fasa_row" in step
    for w in W.WORKLOADS.values():
        known = bench.kernel_bytes(w)
        assert step <= set(known), step - set(known)
        assert all(v > 0 for v in known.values())


def test_measured_traffic_names_known_kernels():
    known = set(bench.kernel_bytes(W.WORKLOADS[1]))
    for key in bench.MEASURED_TRAFFIC:
        if key != "source_hash":
            assert key[0] in W.WORKLOADS and key[1] in known
