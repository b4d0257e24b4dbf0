"""fasa_topk in one launch (lists by the cut of a sample, selected by the workgroup that comes last): segments of 2048 tokens
and their edges, and what misleads the sample or hides from it.  Exact against the oracle on the same float32 scores."""
import zlib

import numpy as np
import pytest

from tests.test_gpu_stages import _check_topk_exact, fb  # noqa: F401

pytestmark = pytest.mark.gpu


def _sampled(n):
    """The tokens of the sample (topk_kernel)."""
    t = np.arange(256, dtype=np.uint64)
    return (((t << np.uint64(16)) | ((t * np.uint64(40503)) & np.uint64(0xffff))) * np.uint64(n) >> np.uint64(24)).astype(int)


def _scores(kind, rows, n, b, rng):
    s = rng.normal(0, 20, size=rows + (n,)).astype(np.float32)
    if kind == "sampled_high":        # fewer than B reach the cut
        s[..., _sampled(n)] += 500
    elif kind == "sampled_low":       # nearly all do
        s[..., _sampled(n)] -= 500
    elif kind == "half_masked":
        s[..., ::2] = -np.inf
    elif kind == "few_finite":        # fewer finite scores than selected ones
        s[..., max(1, b // 2):] = -np.inf
    elif kind == "infinite":
        s[..., ::5] = np.inf
        s[..., 1::7] = -np.inf
    elif kind == "crowded":           # all winners in the last tokens
        s[..., -min(n, b + 3):] += 300
    elif kind == "offset":            # a spread of a few units in the last place
        s = (s / 20000 + 4096).astype(np.float32)
    return s


@pytest.mark.parametrize("rows,n,b", [((1, 1), 257, 8), ((1, 3), 2047, 2046), ((2, 2), 2048, 300), ((1, 2), 2049, 1), ((1, 8), 4096, 700),
                                      ((1, 1), 4097, 3000), ((3, 3), 20011, 1250), ((1, 1), 70000, 40)])
@pytest.mark.parametrize("kind", ["plain", "sampled_high", "sampled_low", "half_masked", "few_finite", "infinite", "crowded", "offset"])
def test_topk_lists(fb, rows, n, b, kind):  # noqa: F811
    print("topk lists", rows, n, b, kind, flush=True)
    rng = np.random.default_rng(zlib.crc32(repr((rows, n, b, kind)).encode()))
    n_cap = (n + 63) // 64 * 64
    s = np.full(rows + (n_cap,), 1e30, dtype=np.float32)          # what lies beyond the row must not count
    s[..., :n] = _scores(kind, rows, n, b, rng)
    _check_topk_exact(fb, s, n, b)


@pytest.mark.parametrize("rows,n,b", [((1, 2), 2047, 300), ((1, 2), 4097, 300), ((3, 3), 20011, 1250), ((1, 1), 70000, 40)])
def test_nan_scores_end(fb, rows, n, b):  # noqa: F811
    """Where NaNs rank is unspecified, but a set has B tokens: finite scores at the sampled places only, so that the list is short,
    and one far above the others, so that the search for the threshold starts below zero."""
    import torch
    print("topk lists, NaN", rows, n, b, flush=True)
    rng = np.random.default_rng(n)
    n_cap = (n + 63) // 64 * 64
    s = np.full(rows + (n_cap,), np.nan, dtype=np.float32)
    s[..., _sampled(n)] = rng.normal(0, 1, size=rows + (256,))
    s[..., _sampled(n)[7]] = 100.0
    shape = fb.make_shape(rows[0], rows[1], rows[1], 128, 16, n, n_cap, b, "bf16")
    ws = torch.empty(fb.fasa_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    fb.fasa_workspace_init(shape, ws, ws.numel())
    T = torch.full(rows + (b,), -1, dtype=torch.int32, device="cuda")
    fb.fasa_topk(shape, torch.from_numpy(s).cuda(), T, ws, ws.numel())
    torch.cuda.synchronize()
    for t in T.reshape(-1, b):
        assert t.min() >= 0 and t.max() < n and t.unique().numel() == b
