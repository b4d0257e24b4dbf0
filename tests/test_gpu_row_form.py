"""Where the decode step's forms begin and end: the one-launch step, lists and selection out of them, the row form of float32
caches (one workgroup per row after the scoring launch) and the split form.  Row counts around 64 and around what the split
form holds at once, budgets on both sides of the line in rows * N, lists that have only just room and lists that overflow, row
lengths and budgets past which no list is made.  The form is told by the kernels that ran; the parity bar is the step's."""
import numpy as np
import pytest

from paper_2602_03152_amd import workload as W
from tests.test_gpu_decode_step import compare_step, fb, run_step  # noqa: F401

pytestmark = pytest.mark.gpu

STEP, LIST, ROW, SPLIT = "fasa_step", "fasa_list", "fasa_row", "fasa_select_attend"
LINES = [
    # (workload, kernel that selects and attends).  bf16: one launch up to 4 slices of 2048 tokens, 256 workgroups and B = 320
    (dict(cid=1, n_ctx=2048, budget=1024), STEP), (dict(cid=1, n_ctx=2048, budget=1025), LIST),
    (dict(cid=1, n_ctx=6144, budget=320), STEP), (dict(cid=1, n_ctx=6144, budget=321), LIST), (dict(cid=1, n_ctx=6145, budget=320), LIST),
    (dict(cid=1, batch=4, n_ctx=8192, budget=256), LIST), (dict(cid=1, batch=5, n_ctx=8192, budget=256), STEP),
    (dict(cid=1, batch=8, n_ctx=8192, budget=256), STEP), (dict(cid=1, batch=9, n_ctx=8192, budget=256), LIST),
    # lists of rows of any number, and what they end at: entries that the threads have no room for, shares of more than 2048
    (dict(cid=2, batch=8, n_ctx=16384, budget=256), LIST), (dict(cid=2, batch=9, n_ctx=16384, budget=256), LIST),
    (dict(cid=3, batch=24, n_ctx=5120, budget=100), LIST), (dict(cid=2, batch=16, n_ctx=8193, budget=513), LIST),
    (dict(cid=2, batch=10, n_ctx=24577, budget=960), LIST),
    (dict(cid=2, batch=19, n_kv_heads=3, n_q_heads=3, n_ctx=32769, budget=64), LIST),
    (dict(cid=2, batch=22, n_kv_heads=2, n_q_heads=2, n_ctx=50001, budget=900), LIST),
    (dict(cid=1, n_kv_heads=1, n_q_heads=4, n_ctx=16385, budget=8192), LIST),
    (dict(cid=1, n_kv_heads=1, n_q_heads=4, n_ctx=20000, budget=9000), SPLIT),
    (dict(cid=2, batch=128, n_kv_heads=1, n_q_heads=4, n_ctx=5000, budget=4096), LIST),
    (dict(cid=2, batch=128, n_kv_heads=1, n_q_heads=4, n_ctx=5000, budget=4097), SPLIT),
    # float32
    (dict(cid=0, batch=72, n_ctx=5000, budget=170), ROW), (dict(cid=0, batch=72, n_ctx=5000, budget=180), SPLIT),
    (dict(cid=0, batch=64, n_kv_heads=2, n_q_heads=8, n_ctx=12321, budget=512), ROW),
    (dict(cid=0, batch=64, n_kv_heads=2, n_q_heads=8, n_ctx=12321, budget=513), SPLIT),
    (dict(cid=0, batch=64, n_kv_heads=2, n_q_heads=10, n_ctx=12321, budget=100), SPLIT),
    # few rows, each of more 4096-token pieces than fit at once (57 rows of 9), and the list's room: 44 rows of 50000
    (dict(cid=0, batch=19, n_kv_heads=3, n_q_heads=3, n_ctx=32769, budget=64), ROW),
    (dict(cid=0, batch=19, n_kv_heads=3, n_q_heads=3, n_ctx=32768, budget=64), SPLIT),
    (dict(cid=0, batch=22, n_kv_heads=2, n_q_heads=2, n_ctx=50001, budget=600), ROW),
    (dict(cid=0, batch=22, n_kv_heads=2, n_q_heads=2, n_ctx=50001, budget=900), SPLIT),
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


@pytest.mark.parametrize("kw,kernel", LINES, ids=str)
def test_lines_of_the_forms(fb, kw, kernel):  # noqa: F811
    kw = dict(kw); cid = kw.pop("cid")
    w = W.WORKLOADS[cid].scaled(**kw)
    x = _inputs(w)
    print("forms", kw, kernel, flush=True)
    fb.fasa_profile_reset()
    fb.fasa_profile_enable(True)
    try:
        d = run_step(fb, w, x)
        names = set(fb.profile_summary())
    finally:
        fb.fasa_profile_enable(False)
        fb.fasa_profile_reset()
    assert names & {STEP, LIST, ROW, SPLIT} == {kernel}, names
    compare_step(w, x["q"], x["K"], x["V"], x["fc_idx"], d, w.n_ctx, w.budget, rows=[0, w.batch // 2, w.batch - 1])
