"""Calibration in one launch (bf16, 8 rows or more, of 8193 .. 32768 tokens) on what its ordinary paths leave: scores that are equal by the hundred and the thousand,
infinite, or no numbers; more of the K best than lists have room for; lists that no threads hold; the other storage order of the pairs; and a full
head whose set comes late, so that FCs leave theirs and its workgroup counts them.  The bar is exact, but for NaNs, whose rank is unspecified."""
import numpy as np
import pytest

from paper_2602_03152_amd import workload as W
from tests.test_gpu_calibration import _calibrate, _exact_counts, fb  # noqa: F401
from tests.test_gpu_calibration_inf import _inputs
from tests.test_gpu_decode_step import _tied_inputs

pytestmark = pytest.mark.gpu


def _workload(n_ctx, batch, heads):
    return W.WORKLOADS[1].scaled(budget=1, n_ctx=n_ctx, batch=batch, n_q_heads=heads[0], n_kv_heads=heads[1])


def _one_launch(fb, w, x, top_k, pairing="half"):  # noqa: F811
    fb.fasa_profile_reset()
    fb.fasa_profile_enable(True)
    try:
        got = _calibrate(fb, w, x, [x["q"]], top_k, pairing)
        assert "fasa_calib_clear" in fb.profile_summary()
    finally:
        fb.fasa_profile_enable(False)
        fb.fasa_profile_reset()
    cnt = np.rint(got * top_k).astype(int)
    assert np.abs(got * top_k - cnt).max() < 1e-3
    return cnt


@pytest.mark.parametrize("n_ctx,batch,heads,top_k,n_classes", [
    (8193, 1, (8, 8), 300, 1), (9000, 1, (16, 8), 500, 7), (9001, 3, (3, 3), 500, 300), (20000, 1, (8, 8), 1500, 40)])
def test_tied_scores(fb, n_ctx, batch, heads, top_k, n_classes):  # noqa: F811
    w = _workload(n_ctx, batch, heads)
    x = _tied_inputs(w, n_classes, seed=3)
    print("calibration odd, ties", n_ctx, batch, heads, top_k, n_classes, flush=True)
    np.testing.assert_array_equal(_one_launch(fb, w, x, top_k), _exact_counts(fb, w, x, [x["q"]], top_k))


@pytest.mark.parametrize("n_ctx,batch,heads,top_k,n_odd,sign", [
    (9000, 1, (8, 8), 500, 8900, -1), (12001, 3, (6, 3), 4000, 7000, -1), (9000, 1, (16, 8), 500, 300, 1), (16384, 1, (8, 8), 1000, 2500, 1)])
def test_infinite_scores(fb, n_ctx, batch, heads, top_k, n_odd, sign):  # noqa: F811
    w = _workload(n_ctx, batch, heads)
    x = _inputs(w, n_odd, sign, 0)
    print("calibration odd, infinite", n_ctx, batch, heads, top_k, n_odd, sign, flush=True)
    np.testing.assert_array_equal(_one_launch(fb, w, x, top_k), _exact_counts(fb, w, x, [x["q"]], top_k))


@pytest.mark.parametrize("n_ctx,heads,top_k,n_odd", [(9000, (8, 8), 8999, 8000), (9000, (8, 8), 500, 9000), (20001, (16, 8), 2000, 600)])
def test_nan_scores_end(fb, n_ctx, heads, top_k, n_odd):  # noqa: F811
    w = _workload(n_ctx, 1, heads)
    x = _inputs(w, n_odd, 1, -1)
    print("calibration odd, NaNs", n_ctx, heads, top_k, n_odd, flush=True)
    cnt = _one_launch(fb, w, x, top_k)
    assert cnt.min() >= max(0, 2 * top_k - n_ctx) and cnt.max() <= top_k


@pytest.mark.parametrize("n_ctx,batch,heads,top_k", [(32768, 1, (8, 8), 5000), (20000, 1, (8, 8), 8000), (8200, 3, (3, 3), 8199), (8193, 1, (8, 8), 1)])
def test_large_budgets(fb, n_ctx, batch, heads, top_k):  # noqa: F811
    w = _workload(n_ctx, batch, heads)
    x = W.make_inputs(w, n_cap=(n_ctx + 63) // 64 * 64)
    print("calibration odd, budgets", n_ctx, batch, heads, top_k, flush=True)
    np.testing.assert_array_equal(_one_launch(fb, w, x, top_k), _exact_counts(fb, w, x, [x["q"]], top_k))


@pytest.mark.parametrize("n_ctx,batch,heads,top_k", [(8201, 1, (32, 8), 700), (12000, 9, (1, 1), 900)])
def test_interleaved_storage(fb, n_ctx, batch, heads, top_k):  # noqa: F811
    w = _workload(n_ctx, batch, heads)
    x = W.as_interleaved(W.make_inputs(w, n_cap=(n_ctx + 63) // 64 * 64))
    print("calibration odd, interleaved", n_ctx, batch, heads, top_k, flush=True)
    np.testing.assert_array_equal(_one_launch(fb, w, x, top_k, "interleaved"), _exact_counts(fb, w, x, [x["q"]], top_k, "interleaved"))


@pytest.mark.parametrize("n_ctx,batch,heads,top_k", [(12000, 1, (8, 8), 900), (32768, 1, (8, 8), 2048)])
def test_a_full_head_that_comes_late(fb, n_ctx, batch, heads, top_k):  # noqa: F811
    """The full head's scores are all equal: FCs cancel in pairs, in numbers that float32 holds exactly."""
    w = _workload(n_ctx, batch, heads)
    x = W.make_inputs(w, n_cap=(n_ctx + 63) // 64 * 64)
    rng = np.random.default_rng(n_ctx)
    k = rng.integers(-128, 128, size=(batch, heads[1], x["n_cap"], 2, 32)).astype(np.float64)      # [lo or hi][pair of FCs]
    K = np.stack([k, -k], axis=-1).reshape(batch, heads[1], x["n_cap"], 128)                       # FC 2j: lo, hi; FC 2j + 1: -lo, -hi
    q = np.concatenate([np.ones((batch, heads[0], 64)), np.full((batch, heads[0], 64), 2.0 ** -7)], axis=-1)
    x["K"][:, :, :x["n_cap"]] = W.to_storage(K, w.dtype)
    x["q"] = W.to_storage(q, w.dtype)
    print("calibration odd, late", n_ctx, batch, heads, top_k, flush=True)
    np.testing.assert_array_equal(_one_launch(fb, w, x, top_k), _exact_counts(fb, w, x, [x["q"]], top_k))
