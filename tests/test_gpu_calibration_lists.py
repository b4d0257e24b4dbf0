"""The full head's set out of its segments' lists: rows whose best lie together (the lists are of no use there), budgets on both sides of the line from which no lists are
made, and rows that one and two workgroups of 1024 and three of 512 share a compute unit for.  The bar is exact."""
import numpy as np
import pytest

from paper_2602_03152_amd import workload as W
from tests.test_gpu_calibration import _calibrate, _exact_counts, fb  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_ctx,batch,heads,top_k,rise", [
    (8193, 1, (8, 2), 500, 0.0), (8193, 1, (8, 2), 500, 0.3), (9000, 2, (8, 4), 800, 0.3), (12289, 1, (14, 2), 2900, 0.0), (12289, 1, (4, 2), 4200, 0.0),
    (20011, 1, (2, 1), 64, 0.3), (33000, 1, (2, 1), 1500, 0.0), (33000, 1, (2, 1), 1500, 0.3)])
def test_counts_exact(fb, n_ctx, batch, heads, top_k, rise):  # noqa: F811
    w = W.WORKLOADS[1].scaled(budget=1, n_ctx=n_ctx, batch=batch, n_q_heads=heads[0], n_kv_heads=heads[1])
    x = W.make_inputs(w, n_cap=(n_ctx + 63) // 64 * 64)
    if rise:      # later keys lean towards the queries
        K = W.storage_to_f64(x["K"])
        lean = W.storage_to_f64(x["q"]).reshape(batch, heads[1], -1, 128).mean(axis=2)
        K[:, :, :n_ctx] += (rise * np.arange(n_ctx) / n_ctx)[None, None, :, None] * lean[:, :, None, :]
        x["K"] = W.to_storage(K, w.dtype)
    print("calibration lists", n_ctx, batch, heads, top_k, rise, flush=True)
    got = _calibrate(fb, w, x, [x["q"]], top_k)
    np.testing.assert_array_equal(np.rint(got * top_k).astype(int), _exact_counts(fb, w, x, [x["q"]], top_k))
