"""The calibration's sets (31 tokens a word) and the launch that makes the full head's beside the FCs': lengths at the ends of
words, one workgroup per row up to more workgroups than fit at once (the later ones find the full head's set ready), several
queries one after the other on one workspace; lists near their room.  The bar is exact."""
import numpy as np
import pytest

from paper_2602_03152_amd import workload as W
from tests.test_gpu_calibration import _calibrate, _exact_counts, fb  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cid,n_ctx,batch,heads,top_k", [
    (1, 31, 1, (1, 1), 30), (1, 62, 1, (2, 2), 7), (1, 63, 1, (8, 1), 31), (1, 310, 7, (12, 6), 45), (1, 1000, 40, (8, 8), 100),
    (1, 8184, 1, (8, 2), 500), (1, 8215, 3, (7, 7), 300), (1, 32767, 1, (4, 2), 2048), (1, 32768, 2, (16, 4), 1000),
    (1, 32768, 1, (4, 1), 4096), (1, 40000, 1, (2, 1), 6000), (1, 65537, 1, (2, 2), 3000), (0, 1500, 20, (4, 4), 150), (0, 8215, 2, (4, 2), 400)])
def test_counts_exact(fb, cid, n_ctx, batch, heads, top_k):  # noqa: F811
    w = W.WORKLOADS[cid].scaled(budget=1, n_ctx=n_ctx, batch=batch, n_q_heads=heads[0], n_kv_heads=heads[1])
    x = W.make_inputs(w, n_cap=(n_ctx + 63) // 64 * 64)
    print("calibration sets", cid, n_ctx, batch, heads, top_k, flush=True)
    queries = [x["q"], x["q"][:, ::-1].copy()]                # (the second adds to the first)
    got = _calibrate(fb, w, x, queries, top_k)
    want = _exact_counts(fb, w, x, queries, top_k)
    np.testing.assert_array_equal(np.rint(got * top_k).astype(int), want)
