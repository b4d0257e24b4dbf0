"""Rows that one workgroup selects out of its registers, where the bin that the B-th score lies in is crowded: ties by the hundred, many scores next to nothing among others, masks
and infinities by the hundred, one score far from all others, in fasa_topk and in the one-launch step, whose threads hold one, two and four pieces of the row.  Exact
against the oracle on the same float32 scores."""
import zlib

import numpy as np
import pytest

from paper_2602_03152_amd import workload as W
from tests.test_gpu_decode_step import _tied_inputs, compare_step, run_step
from tests.test_gpu_stages import _check_topk_exact, fb  # noqa: F401

pytestmark = pytest.mark.gpu


def _scores(kind, rows, n, rng):
    s = rng.normal(0, 20, size=rows + (n,))
    half = n // 2
    if kind == "next_to_nothing":      # half of the row within a bin's width
        s[..., half:] *= 1e-4
    elif kind == "equal":
        s[:] = 7.0
    elif kind == "two":
        s = np.where(s > 0, 3.0, -3.0)
    elif kind == "zeros":              # of both signs, equal to each other
        s[..., :half] = np.where(s[..., :half] > 0, 0.0, -0.0)
    elif kind == "masked":             # a stretch at the type's lowest value
        s[..., half:] = np.finfo(np.float32).min
    elif kind == "minus_inf":
        s[..., 1::2] = -np.inf
    elif kind == "plus_inf":
        s[..., ::3] = np.inf
    elif kind == "far":
        s[..., n // 3] = 1e12
        s[..., n // 7] = -1e12
    elif kind == "ties_in_a_cluster":
        s[..., half:] = np.round(s[..., half:] / 10) * 1e-4
    return s.astype(np.float32)


@pytest.mark.parametrize("kind", ["next_to_nothing", "equal", "two", "zeros", "masked", "minus_inf", "plus_inf", "far", "ties_in_a_cluster"])
@pytest.mark.parametrize("n,b", [(130, 65), (257, 128), (300, 299), (1000, 256), (1000, 500), (1531, 192), (2048, 1000), (2048, 1400), (2047, 33)])
def test_topk_of_crowded_bins(fb, n, b, kind):  # noqa: F811
    print("crowded", n, b, kind, flush=True)
    rng = np.random.default_rng(zlib.crc32(repr((n, b, kind)).encode()))
    s = np.full((2, 3, (n + 63) // 64 * 64), 1e38, dtype=np.float32)      # what lies beyond the row must not count
    s[..., :n] = _scores(kind, (2, 3), n, rng)
    _check_topk_exact(fb, s, n, b)


def _one_launch(fb, w, x):  # noqa: F811
    fb.fasa_profile_reset()
    fb.fasa_profile_enable(True)
    try:
        d = run_step(fb, w, x)
        assert set(fb.profile_summary()) & {"fasa_step", "fasa_list", "fasa_select_attend"} == {"fasa_step"}
    finally:
        fb.fasa_profile_enable(False)
        fb.fasa_profile_reset()
    compare_step(w, x["q"], x["K"], x["V"], x["fc_idx"], d, w.n_ctx, w.budget, rows=[0, w.batch - 1])


STEPS = [dict(cid=1, n_ctx=2048, budget=700), dict(cid=1, n_ctx=1531, budget=192), dict(cid=1, n_ctx=4000, budget=256), dict(cid=1, batch=8, n_ctx=8192, budget=320),
         dict(cid=0, n_ctx=1001, budget=300), dict(cid=0, n_ctx=4096, budget=500), dict(cid=0, n_ctx=8192, budget=300)]


@pytest.mark.parametrize("n_classes", [1, 3, 20])
@pytest.mark.parametrize("kw", STEPS, ids=str)
def test_step_of_tied_scores(fb, kw, n_classes):  # noqa: F811
    kw = dict(kw); cid = kw.pop("cid")
    w = W.WORKLOADS[cid].scaled(**kw)
    print("crowded step, ties", kw, n_classes, flush=True)
    _one_launch(fb, w, _tied_inputs(w, n_classes, seed=5))


@pytest.mark.parametrize("kind", ["far", "zero_keys"])
@pytest.mark.parametrize("kw", STEPS, ids=str)
def test_step_of_odd_keys(fb, kw, kind):  # noqa: F811
    kw = dict(kw); cid = kw.pop("cid")
    w = W.WORKLOADS[cid].scaled(**kw)
    x = W.make_inputs(w, n_cap=(w.n_ctx + 63) // 64 * 64)
    K = W.storage_to_f64(x["K"])
    if kind == "far":
        K[:, :, w.n_ctx // 3] *= 1e6                          # one key, of either sign for the queries
    else:
        K[:, :, w.n_ctx // 4:3 * w.n_ctx // 4] = 0.0          # padding: scores that are all equal
    x["K"] = W.to_storage(K, w.dtype)
    print("crowded step", kw, kind, flush=True)
    _one_launch(fb, w, x)
