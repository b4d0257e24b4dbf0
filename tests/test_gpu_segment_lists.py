"""Lists of segments of 256 tokens (csrc/row_list.h) at their edges: rows that end a token before, at and behind a segment,
room for all of a segment's scores and for eight, the fewest there are, scores that leave the first bins of a cut empty, rows whose best
lie in few segments, beyond the 512th among them, segments of NaNs, and more of the best in places that were not listed than LDS
has room for.  Two listed dims make the scores, so that hardly any two
are equal.  The bar is exact: the set is TopK-I of the device's own float32 scores."""
import numpy as np
import pytest
import torch

from oracle import fasa_oracle as O
from paper_2602_03152_amd import workload as W
from tests.test_gpu_list_cuts import ROW, fb, how_selected, step_of  # noqa: F401

pytestmark = pytest.mark.gpu

D = 128


def _scores(kind, rows, n, budget):
    rng = np.random.default_rng(n + 3 * budget)
    x = rng.standard_normal((rows, n))
    if kind == "sinks":                              # some segments' best far above all others, twice over
        x[:, 5::512] = 1e4
        x[:, 6::512] = 1e8
    elif kind == "rising":                           # all of the best in the last segments, and nearly as good ones ahead of them
        x = 0.02 * x + np.linspace(-3, 3, n)
    elif kind == "blocks":                           # every 7th segment holds more of the best than it has room for
        x += 6.0 * ((np.arange(n) // 256) % 7 == 3)
    elif kind == "masked":
        x[:, ::3] = -np.inf
    elif kind == "late":                             # all of the best in segments whose neighbours in the threads' registers are far away
        x[:, n * 5 // 6:n * 5 // 6 + 2 * budget] += 9.0
    return x


def _run(fb, scores, budget, lens=None, budgets=None, nan=None):  # noqa: F811
    rows, n = scores.shape
    cap = (n + 63) // 64 * 64
    x = np.zeros((rows, 8, cap, 2), dtype=np.uint16)
    finite = np.where(np.isfinite(scores), scores, 0.0)
    hi = W.to_storage(scores, "bf16")
    x[:, 0, :n, 0] = np.where(np.isnan(scores), nan, hi) if nan else hi
    x[:, 1, :n, 0] = W.to_storage(np.where(np.isfinite(scores), finite - W.storage_to_f64(W.to_storage(finite, "bf16")), 0.0), "bf16")
    q = torch.zeros(rows, 1, D, dtype=torch.bfloat16, device="cuda")
    q[:, :, :2] = 1.0
    K = torch.zeros(cap, D, dtype=torch.bfloat16, device="cuda")             # one K and V for all rows
    V = torch.randn(cap, D, generator=torch.Generator(device="cuda").manual_seed(n), device="cuda").bfloat16()
    fc = torch.arange(8, dtype=torch.int32, device="cuda")
    shape = fb.make_shape(rows, 1, 1, D, 8, n, cap, budget, "bf16", kv_stride_b=0, kv_stride_h=0, kv_stride_n=D)
    ws = torch.empty(fb.fasa_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    fb.fasa_workspace_init(shape, ws, ws.numel())
    S = torch.zeros(rows, 1, cap, device="cuda")
    Kp = torch.from_numpy(x.view(np.int16)).cuda()
    names = set()
    for i in range(2):                               # the workspace is left as it has to be
        fb.fasa_profile_enable(i == 0)
        T = torch.full((rows, 1, min(budget, n)), -1, dtype=torch.int32, device="cuda")
        out = torch.full((rows, 1, D), float("nan"), device="cuda")
        if lens is None:
            fb.fasa_decode_step(shape, q, K, V, Kp, fc, None, None, S, T, out, ws, ws.numel())
        else:
            fb.fasa_decode_step_ragged(shape, q, K, V, Kp, fc, None, None, lens, budgets, S, T, out, ws, ws.numel())
        torch.cuda.synchronize()
        names |= set(fb.profile_summary()) if i == 0 else set()
    fb.fasa_profile_enable(False)
    fb.fasa_profile_reset()
    assert {"fasa_score_list", "fasa_list"} <= names, names
    return S[:, 0].cpu().numpy(), T[:, 0].cpu().numpy(), out[:, 0].cpu().double(), V.cpu().double()


def _check(S, T, out, V, r, n, b):
    got = np.sort(T[r, :b])
    np.testing.assert_array_equal(got, O.topk(S[r][None, None, :n], b, n)[0, 0])
    # K is 0: every selected token weighs the same; float32 sums of at most 1e4 terms of at most about 5
    assert (out[r] - V[torch.from_numpy(got).long()].mean(0)).abs().max().item() <= 1e-4


@pytest.mark.parametrize("kind", ["plain", "sinks", "rising", "blocks", "masked"])
@pytest.mark.parametrize("rows,n_ctx,budget", [
    (8, 8191, 1), (8, 2304, 2303), (8, 2305, 1150),               # room for eight, for all, for a third
    (33, 9983, 300), (8, 9985, 2048), (8, 32767, 2048), (3, 40001, 7000), (8, 131073, 1500), (2, 524288, 600)])
def test_segments(fb, kind, rows, n_ctx, budget):  # noqa: F811
    print("segments", kind, rows, n_ctx, budget, flush=True)
    S, T, out, V = _run(fb, _scores(kind, rows, n_ctx, budget), budget)
    for r in sorted({0, rows // 2, rows - 1}):
        _check(S, T, out, V, r, n_ctx, budget)


@pytest.mark.parametrize("rows,n_ctx,budget", [(8, 131073, 1500), (4, 200001, 3000), (2, 524288, 600)])
def test_best_beyond_the_segments_of_the_threads(fb, rows, n_ctx, budget):  # noqa: F811
    """More segments than threads: what a thread knows of its segments is then the highest of several."""
    print("late", rows, n_ctx, budget, flush=True)
    S, T, out, V = _run(fb, _scores("late", rows, n_ctx, budget), budget)
    for r in range(rows):
        _check(S, T, out, V, r, n_ctx, budget)


@pytest.mark.parametrize("n_ctx,budget,first", [(42000, 9900, 30000), (42000, 9900, 0), (65536, 8192, 20000)])
def test_more_than_lds_holds(fb, n_ctx, budget, first):  # noqa: F811
    """All of the best in one stretch of two values: what is not listed of it has no room in LDS, and all of the row's scores are read, from a
    key on that is known by then."""
    rows = 3
    x = _scores("plain", rows, n_ctx, budget)
    x[:, first:first + 12000] = 8.0 + np.random.default_rng(budget).integers(0, 2, (rows, 12000))
    print("more than LDS holds", n_ctx, budget, first, flush=True)
    run, S, T, out, V, ws = step_of(fb, x, budget)
    for again in range(2):
        T.fill_(-1)
        run()
        torch.cuda.synchronize()
        for r in range(rows):
            _check(S[:, 0].cpu().numpy(), T[:, 0].cpu().numpy(), out[:, 0].cpu().double(), V.cpu().double(), r, n_ctx, budget)
        assert (how_selected(ws, rows)[1] == ROW).all()


@pytest.mark.parametrize("nan", [0x7fc0, 0xffc0], ids=hex)
def test_segments_of_nans_but_one(fb, nan):  # noqa: F811
    """Where NaNs rank is unspecified, but a set has B tokens: B of the finite scores if there are no more."""
    rows, n, budget = 8, 20000, 700
    x = np.full((rows, n), -np.inf)
    x[:, :budget] = _scores("plain", rows, n, budget)[:, :budget]
    x[:, 4096:8192] = np.nan
    x[:, 4096 + 77:8192:256] = 1.0
    print("segments of NaNs", hex(nan), flush=True)
    S, T, out, V = _run(fb, x, budget, nan=nan)
    for r in range(rows):
        assert T[r].min() >= 0 and T[r].max() < n and np.unique(T[r]).size == budget
        assert (out[r] - V[torch.from_numpy(T[r].astype(np.int64))].mean(0)).abs().max().item() <= 1e-4


@pytest.mark.parametrize("kind", ["plain", "blocks"])
def test_sequences_with_less_room_than_they_ask_for(fb, kind):  # noqa: F811
    """The places the selecting threads hold follow from the bounds; a sequence's budget may ask for more of them."""
    rows, n, budget = 8, 30000, 3000
    lens = [n, n - 255, 15001, 4097, 3000, 2999, 257, 1]
    budgets = [3000, 2999, 3000, 3000, 2999, 3000, 256, 1]
    dev = lambda a: torch.tensor(a, dtype=torch.int32, device="cuda")   # noqa: E731
    print("ragged segments", kind, flush=True)
    S, T, out, V = _run(fb, _scores(kind, rows, n, budget), budget, dev(lens), dev(budgets))
    for r in range(rows):
        _check(S, T, out, V, r, lens[r], min(budgets[r], lens[r]))
