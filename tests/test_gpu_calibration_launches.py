"""Calibration in one launch (rows that score the full head's slices, find its set and stream the FCs side by side): rows on both sides of its lines in tokens and
in rows, slices with one token, lists that the threads hold and longer ones, rows whose best lie together, several queries one after
the other on one workspace.  The bar is exact."""
import numpy as np
import pytest

from paper_2602_03152_amd import workload as W
from tests.test_gpu_calibration import _calibrate, _exact_counts, fb  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_ctx,batch,heads,top_k,rise", [
    (8192, 1, (8, 8), 300, 0.0), (8193, 1, (8, 8), 300, 0.0), (8193, 1, (8, 8), 300, 0.3), (16384, 1, (7, 7), 900, 0.0), (16384, 3, (3, 3), 900, 0.0),
    (9217, 1, (16, 8), 4000, 0.0), (10241, 2, (8, 4), 1, 0.0), (12000, 5, (4, 2), 700, 0.3), (12001, 1, (8, 8), 700, 0.0), (32768, 1, (8, 8), 3500, 0.3),
    (32768, 1, (8, 8), 2048, 0.0), (32700, 1, (8, 8), 4400, 0.0), (32769, 1, (2, 2), 1000, 0.0)])
def test_counts_exact(fb, n_ctx, batch, heads, top_k, rise):  # noqa: F811
    w = W.WORKLOADS[1].scaled(budget=1, n_ctx=n_ctx, batch=batch, n_q_heads=heads[0], n_kv_heads=heads[1])
    x = W.make_inputs(w, n_cap=(n_ctx + 63) // 64 * 64)
    if rise:      # later keys lean towards the queries
        K = W.storage_to_f64(x["K"])
        lean = W.storage_to_f64(x["q"]).reshape(batch, heads[1], -1, 128).mean(axis=2)
        K[:, :, :n_ctx] += (rise * np.arange(n_ctx) / n_ctx)[None, None, :, None] * lean[:, :, None, :]
        x["K"] = W.to_storage(K, w.dtype)
    queries = [x["q"], x["q"][:, ::-1].copy()]                # (the second adds to the first)
    print("calibration launches", n_ctx, batch, heads, top_k, rise, flush=True)
    fb.fasa_profile_reset()
    fb.fasa_profile_enable(True)
    try:
        got = _calibrate(fb, w, x, queries, top_k)
        names = set(fb.profile_summary())
    finally:
        fb.fasa_profile_enable(False)
        fb.fasa_profile_reset()
    one = 8192 < n_ctx <= 32768 and batch * heads[1] >= 8
    assert ("fasa_calib_clear" in names) == one and ("fasa_calib_full" in names) != one, names
    np.testing.assert_array_equal(np.rint(got * top_k).astype(int), _exact_counts(fb, w, x, queries, top_k))
