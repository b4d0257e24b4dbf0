"""Where the decode step's row form (one workgroup per row after the scoring launch) begins and ends: row counts around 64
and around what the split form holds at once, budgets on both sides of the line in rows * N, lists that have
only just room and lists that overflow.  The form is told by the kernels that ran; the parity bar is the step's."""
import numpy as np
import pytest

from paper_2602_03152_amd import workload as W
from tests.test_gpu_decode_step import compare_step, fb, run_step  # noqa: F401

pytestmark = pytest.mark.gpu

LINES = [
    # (workload, row form or not)
    (dict(cid=2, batch=8, n_ctx=16384, budget=256), False), (dict(cid=2, batch=9, n_ctx=16384, budget=256), True),
    (dict(cid=3, batch=24, n_ctx=5119, budget=100), False), (dict(cid=3, batch=24, n_ctx=5120, budget=100), True),
    (dict(cid=2, batch=16, n_ctx=8192, budget=512), True), (dict(cid=2, batch=16, n_ctx=8192, budget=513), False),
    (dict(cid=2, batch=10, n_ctx=24577, budget=960), True),
    # few rows, each of more 4096-token pieces than fit: 57 rows of 9
    (dict(cid=2, batch=19, n_kv_heads=3, n_q_heads=3, n_ctx=32769, budget=64), True),
    (dict(cid=2, batch=19, n_kv_heads=3, n_q_heads=3, n_ctx=32768, budget=64), False),
    # the list's room: 44 rows of 50000
    (dict(cid=2, batch=22, n_kv_heads=2, n_q_heads=2, n_ctx=50001, budget=600), True),
    (dict(cid=2, batch=22, n_kv_heads=2, n_q_heads=2, n_ctx=50001, budget=900), False),
    (dict(cid=0, batch=72, n_ctx=5000, budget=170), True), (dict(cid=0, batch=72, n_ctx=5000, budget=180), False),
    (dict(cid=0, batch=64, n_kv_heads=2, n_q_heads=8, n_ctx=12321, budget=512), True),
    (dict(cid=0, batch=64, n_kv_heads=2, n_q_heads=8, n_ctx=12321, budget=513), False),
    (dict(cid=0, batch=64, n_kv_heads=2, n_q_heads=10, n_ctx=12321, budget=100), False),
]


def _inputs(w):
    """One sequence drawn as ever, and the batch made of it: the tokens in another rotation for every entry."""
    x = W.make_inputs(w.scaled(batch=1), n_cap=(w.n_ctx + 63) // 64 * 64)
    for name in ("K", "V"):
        one = x[name][0]
        x[name] = np.stack([one] * w.batch)
        for b in range(1, w.batch):
            x[name][b, :, :w.n_ctx] = np.roll(one[:, :w.n_ctx], 97 * b, axis=1)
    x["q"] = np.repeat(x["q"], w.batch, axis=0)
    return x


@pytest.mark.parametrize("kw,row_form", LINES, ids=str)
def test_lines_of_the_row_form(fb, kw, row_form):  # noqa: F811
    kw = dict(kw); cid = kw.pop("cid")
    w = W.WORKLOADS[cid].scaled(**kw)
    x = _inputs(w)
    print("row form", kw, flush=True)
    fb.fasa_profile_reset()
    fb.fasa_profile_enable(True)
    try:
        d = run_step(fb, w, x)
        names = set(fb.profile_summary())
    finally:
        fb.fasa_profile_enable(False)
        fb.fasa_profile_reset()
    assert ("fasa_row" in names) == row_form, names
    compare_step(w, x["q"], x["K"], x["V"], x["fc_idx"], d, w.n_ctx, w.budget, rows=[0, w.batch // 2, w.batch - 1])
