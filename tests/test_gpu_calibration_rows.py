"""The calibration's per-row selection at the sizes where it changes form: rows in flight in one stretch or
several, the switch between workgroup sizes, lists that overflow (large K, tied scores).  The bar is exact: the
oracle's ranking on the device's own scores."""
import numpy as np
import pytest

from paper_2602_03152_amd import workload as W
from tests.test_gpu_calibration import _calibrate, _exact_counts, fb  # noqa: F401
from tests.test_gpu_decode_step import _tied_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw,top_k,n_classes", [
    (dict(cid=1, n_ctx=1, n_kv_heads=1, n_q_heads=4), 1, 0),
    (dict(cid=1, n_ctx=4096, n_kv_heads=1, n_q_heads=2), 1, 0),
    (dict(cid=1, n_ctx=4097, n_kv_heads=1, n_q_heads=2), 4096, 0),      # all but one: the list overflows
    (dict(cid=1, n_ctx=8192, n_kv_heads=1, n_q_heads=8), 700, 0),
    (dict(cid=1, n_ctx=8193, n_kv_heads=1, n_q_heads=1), 700, 0),
    (dict(cid=1, n_ctx=16385, n_kv_heads=1, n_q_heads=7), 2100, 0),
    (dict(cid=1, n_ctx=32769, n_kv_heads=1, n_q_heads=4), 4000, 0),
    (dict(cid=0, n_ctx=2049), 200, 0),
    (dict(cid=0, n_ctx=9001), 1500, 0),
    (dict(cid=1, n_ctx=5000, n_kv_heads=1, n_q_heads=4), 300, 1),       # every score equal
    (dict(cid=1, n_ctx=9000, n_kv_heads=1, n_q_heads=4), 500, 7),
    (dict(cid=1, n_ctx=9000, n_kv_heads=1, n_q_heads=4), 500, 300),
], ids=str)
def test_counts_exact_at_the_edges(fb, kw, top_k, n_classes):  # noqa: F811
    kw = dict(kw); cid = kw.pop("cid")
    w = W.WORKLOADS[cid].scaled(budget=1, **kw)
    x = _tied_inputs(w, n_classes, seed=3) if n_classes else W.make_inputs(w, n_cap=(w.n_ctx + 63) // 64 * 64)
    print("calibration rows", kw, top_k, flush=True)
    got = _calibrate(fb, w, x, [x["q"]], top_k)
    kk = min(top_k, w.n_ctx)
    np.testing.assert_array_equal(np.rint(got * kk).astype(int), _exact_counts(fb, w, x, [x["q"]], top_k))
