"""Every instance of the one-launch step: list lengths with and without one of their own, one query head, up to four and up to
eight, one slice of a row and several, both storage types, with an appended row."""
import pytest

from paper_2602_03152_amd import workload as W
from tests.test_gpu_decode_step import compare_step, fb, run_step  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_fc", [7, 8, 16, 24, 32, 33])
@pytest.mark.parametrize("kw", [
    dict(cid=0, n_ctx=1021, n_q_heads=2, n_kv_heads=2), dict(cid=0, n_ctx=5003), dict(cid=0, n_ctx=1024, n_q_heads=4),
    dict(cid=0, n_ctx=517, n_q_heads=16, n_kv_heads=2), dict(cid=3, batch=1, n_ctx=1999), dict(cid=1, n_ctx=5003)], ids=str)
def test_instances(fb, kw, n_fc):  # noqa: F811
    kw = dict(kw); cid = kw.pop("cid")
    w = W.WORKLOADS[cid].scaled(budget=60, n_fc=n_fc, **kw)
    x = W.make_inputs(w, n_cap=(w.n_ctx + 63) // 64 * 64)
    app = W.make_append(w, x["fc_idx"], 1, w.n_ctx - 1)
    print("instance", kw, n_fc, flush=True)
    fb.fasa_profile_reset()
    fb.fasa_profile_enable(True)
    try:
        d = run_step(fb, w, x, k_new=app["k_new"], v_new=app["v_new"], q=app["q"])
        assert "fasa_step" in fb.profile_summary()
    finally:
        fb.fasa_profile_enable(False)
        fb.fasa_profile_reset()
    x["K"][:, :, w.n_ctx - 1] = app["k_new"]
    x["V"][:, :, w.n_ctx - 1] = app["v_new"]
    compare_step(w, app["q"], x["K"], x["V"], x["fc_idx"], d, w.n_ctx, w.budget)
