"""Scores that are not ordinary numbers in the calibration.  Finite queries and keys reach them: products that
overflow, and the sum of two that overflow in opposite directions.  Infinite scores rank like any others, so
the counts are exact, also where the K-th score is one of many -inf; where NaNs rank is unspecified, but
every set has K tokens and the call ends."""
import numpy as np
import pytest

from paper_2602_03152_amd import workload as W
from tests.test_gpu_calibration import _calibrate, _exact_counts, fb  # noqa: F401

pytestmark = pytest.mark.gpu

FC, HALF, BIG = 5, 64, 1e20          # BIG * BIG overflows float32; the sum of 8 queries of BIG does not


def _inputs(w, n_odd, sign_lo, sign_hi):
    """Make n_odd tokens' products of FC's two dims overflow to sign * inf (sign 0: dims as drawn)."""
    x = W.make_inputs(w, n_cap=(w.n_ctx + 63) // 64 * 64)
    rng = np.random.default_rng(n_odd)
    big = W.to_storage(np.array([-BIG, 0.0, BIG]), w.dtype)
    for h in range(w.n_kv_heads):
        odd = rng.permutation(w.n_ctx)[:n_odd]
        for dim, sign in ((FC, sign_lo), (FC + HALF, sign_hi)):
            if sign:
                x["q"][:, h * w.group:(h + 1) * w.group, dim] = big[2]
                x["K"][:, h, odd, dim] = big[1 + sign]
    return x


@pytest.mark.parametrize("kw,top_k,n_odd,sign", [
    (dict(cid=1, n_ctx=4000, n_kv_heads=2, n_q_heads=8), 1200, 3000, -1),
    (dict(cid=1, n_ctx=4999, n_kv_heads=1, n_q_heads=1), 4998, 4999, -1),       # all but one of a row of equals
    (dict(cid=1, n_ctx=32768, n_kv_heads=1, n_q_heads=4), 2048, 31800, -1),
    (dict(cid=1, n_ctx=40001, n_kv_heads=1, n_q_heads=7), 5000, 36000, -1),     # several stretches per row
    (dict(cid=0, n_ctx=9001), 500, 8900, -1),
    (dict(cid=1, n_ctx=9000, n_kv_heads=1, n_q_heads=4), 500, 600, 1),
    (dict(cid=0, n_ctx=3000), 500, 100, 1),
], ids=str)
def test_infinite_scores_rank(fb, kw, top_k, n_odd, sign):  # noqa: F811
    kw = dict(kw); cid = kw.pop("cid")
    w = W.WORKLOADS[cid].scaled(budget=1, **kw)
    x = _inputs(w, n_odd, sign, 0)
    print("calibration, infinite scores", kw, top_k, n_odd, sign, flush=True)
    got = _calibrate(fb, w, x, [x["q"]], top_k)
    want = _exact_counts(fb, w, x, [x["q"]], top_k)
    np.testing.assert_array_equal(np.rint(got * top_k).astype(int), want)
    assert want[:, :, FC].max() > 0                       # the set of the FC in question is not empty


@pytest.mark.parametrize("kw,top_k,n_odd", [
    (dict(cid=1, n_ctx=4000, n_kv_heads=2, n_q_heads=8), 3999, 3000),           # fewer than K ordinary scores
    (dict(cid=1, n_ctx=40001, n_kv_heads=1, n_q_heads=4), 40000, 40001),        # none
    (dict(cid=0, n_ctx=9001), 500, 8800),
], ids=str)
def test_nan_scores_end(fb, kw, top_k, n_odd):  # noqa: F811
    kw = dict(kw); cid = kw.pop("cid")
    w = W.WORKLOADS[cid].scaled(budget=1, **kw)
    x = _inputs(w, n_odd, 1, -1)
    print("calibration, NaN scores", kw, top_k, n_odd, flush=True)
    got = _calibrate(fb, w, x, [x["q"]], top_k) * top_k
    cnt = np.rint(got).astype(int)
    assert np.abs(got - cnt).max() < 1e-3 and cnt.min() >= 0 and cnt.max() <= top_k
    # both sets have K of the N tokens (which says most where K is N - 1)
    assert cnt.min() >= 2 * top_k - w.n_ctx
