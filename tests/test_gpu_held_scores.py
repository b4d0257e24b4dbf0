"""Rows that one workgroup selects out of its registers (fasa_topk up to 2048 tokens, the one-launch step): lengths and budgets on both
sides of where the first range begins at the threads' largest scores, scores that take a second and a third pass, and ones that take more
than there are.  Exact against the oracle on the same float32 scores."""
import zlib

import numpy as np
import pytest

from paper_2602_03152_amd import workload as W
from tests.test_gpu_decode_step import compare_step, run_step
from tests.test_gpu_stages import _check_topk_exact, fb  # noqa: F401

pytestmark = pytest.mark.gpu


def _scores(kind, rows, n, rng):
    s = rng.normal(0, 20, size=rows + (n,))
    if kind == "far":                 # one score far above, one far below: all others in one bin
        s[..., n // 3] = 1e30
        s[..., n // 5] = -1e30
    elif kind == "nested":            # every range leaves most scores in one bin of the next
        for i, x in enumerate((1e30, 1e24, 1e18, 1e12, 1e6)):
            s[..., i::17] = x * (1 + i / 8)
        s[..., n // 7] = -3.4e38
    elif kind == "lowest":            # a mask of the type's lowest value
        s[..., 1::2] = np.finfo(np.float32).min
    elif kind == "tied":
        s = np.round(s / 40)
    elif kind == "rising":            # a thread's scores next to each other
        s = np.sort(s, axis=-1)
    return s.astype(np.float32)


@pytest.mark.parametrize("kind", ["plain", "far", "nested", "lowest", "tied", "rising"])
@pytest.mark.parametrize("n,b", [(2, 1), (63, 15), (64, 16), (65, 17), (256, 64), (257, 255), (1531, 192), (1531, 383), (2047, 512), (2048, 511),
                                 (2048, 512), (2048, 513), (2048, 2047)])
def test_topk_of_held_scores(fb, n, b, kind):  # noqa: F811
    print("held", n, b, kind, flush=True)
    rng = np.random.default_rng(zlib.crc32(repr((n, b, kind)).encode()))
    s = np.full((2, 3, (n + 63) // 64 * 64), 1e38, dtype=np.float32)      # what lies beyond the row must not count
    s[..., :n] = _scores(kind, (2, 3), n, rng)
    _check_topk_exact(fb, s, n, b)


@pytest.mark.parametrize("kw", [
    dict(cid=1, n_ctx=2048, budget=512), dict(cid=1, n_ctx=2048, budget=513), dict(cid=1, n_ctx=2049, budget=320), dict(cid=1, n_ctx=4096, budget=256),
    dict(cid=1, n_ctx=4097, budget=256), dict(cid=1, n_ctx=6144, budget=1), dict(cid=1, batch=8, n_ctx=8192, budget=320), dict(cid=0, n_ctx=1024, budget=256),
    dict(cid=0, n_ctx=1025, budget=257), dict(cid=0, n_ctx=4096, budget=512), dict(cid=0, n_ctx=4097, budget=512)], ids=str)
def test_step_of_held_scores(fb, kw):  # noqa: F811
    kw = dict(kw); cid = kw.pop("cid")
    w = W.WORKLOADS[cid].scaled(**kw)
    x = W.make_inputs(w, n_cap=(w.n_ctx + 63) // 64 * 64)
    print("held step", kw, flush=True)
    fb.fasa_profile_reset()
    fb.fasa_profile_enable(True)
    try:
        d = run_step(fb, w, x)
        assert set(fb.profile_summary()) & {"fasa_step", "fasa_list", "fasa_select_attend"} == {"fasa_step"}
    finally:
        fb.fasa_profile_enable(False)
        fb.fasa_profile_reset()
    compare_step(w, x["q"], x["K"], x["V"], x["fc_idx"], d, w.n_ctx, w.budget, rows=[0, w.batch - 1])
