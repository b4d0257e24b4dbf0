"""The lists that the scoring launch of a bf16 step makes (csrc/row_list.h) where a row's best scores lie together, as those of
attention do: rows of an autoregression, rows that rise, rows with all of their best in a few neighbouring segments of 256
tokens.  Such a segment has more of the best than it has places for.  Its scores are then read again, which is exact too but
costs every workgroup of the row some round trips, and has to stay the exception for scores that are independent; all of the
row's scores are read where nothing else is left, which no finite scores but ties need."""
import numpy as np
import pytest
import torch

from oracle import fasa_oracle as O
from paper_2602_03152_amd import workload as W

pytestmark = pytest.mark.gpu

D, HIST_BYTES, CTL_BYTES, CUT_WORD = 128, 4096 * 4, 128, 6     # of a row: histogram, counters, its cut and how it was selected (csrc/fasa_internal.h)
ALONE, REREAD, ROW = 1, 2, 3                     # out of its list, with scores read again, out of all of its scores


@pytest.fixture(scope="module")
def fb():
    from paper_2602_03152_amd import binding
    return binding


def make_scores(kind, rows, n, budget):
    rng = np.random.default_rng(n + budget)
    x = rng.standard_normal((rows, n)).astype(np.float32)
    if kind.startswith("ar"):
        rho = np.float32(kind[2:])
        x[:, 1:] *= np.sqrt(1 - rho * rho)
        for i in range(1, n):
            x[:, i] += rho * x[:, i - 1]
    elif kind == "rising":
        x = 0.01 * x + np.linspace(-3, 3, n, dtype=np.float32)
    elif kind == "recent":                           # a window of the last tokens
        x[:, n - min(1000, n // 8):] += 8.0
    elif kind == "together":                         # as many as fit, then some, in one place of every row
        for r in range(rows):
            at = rng.integers(0, n - min(n, 2 * budget) + 1)
            x[r, at:at + 2 * budget] += 8.0
    elif kind == "one_segment_infinite":
        x[:, 1024:2048] = np.inf
    elif kind == "outliers":                         # one score far above the rest in every segment, or far below
        x[:, 7::1024] = 3e4
        x[:, 9::1024] = -3e30
    elif kind == "levels":                           # ties in their thousands
        x = np.round(x * 2) / 2
    return x


def step_of(fb, scores, budget, lens=None, budgets=None, planes=None):
    """One step over rows of these scores (one KV head each; K is 0 beside them, so every selected token weighs the same)."""
    rows, n = scores.shape
    cap = (n + 63) // 64 * 64
    x = np.zeros((rows, 8, cap, 2), dtype=np.uint16)
    x[:, 0, :n, 0] = W.to_storage(scores, "bf16")
    if planes:
        planes(x)
    Kp = torch.from_numpy(x.view(np.int16)).cuda()
    q = torch.zeros(rows, 1, D, dtype=torch.bfloat16, device="cuda")
    q[:, :, 0] = 1.0
    K = torch.zeros(cap, D, dtype=torch.bfloat16, device="cuda")             # one K and V for all rows
    V = torch.randn(cap, D, generator=torch.Generator(device="cuda").manual_seed(n), device="cuda").bfloat16()
    fc = torch.arange(8, dtype=torch.int32, device="cuda")
    shape = fb.make_shape(rows, 1, 1, D, 8, n, cap, budget, "bf16", kv_stride_b=0, kv_stride_h=0, kv_stride_n=D)
    ws = torch.empty(fb.fasa_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    fb.fasa_workspace_init(shape, ws, ws.numel())
    S = torch.zeros(rows, 1, cap, device="cuda")
    T = torch.full((rows, 1, budget), -1, dtype=torch.int32, device="cuda")
    out = torch.zeros(rows, 1, D, device="cuda")

    def run():
        if lens is None:
            fb.fasa_decode_step(shape, q, K, V, Kp, fc, None, None, S, T, out, ws, ws.numel())
        else:
            fb.fasa_decode_step_ragged(shape, q, K, V, Kp, fc, None, None, lens, budgets, S, T, out, ws, ws.numel())
    return run, S, T, out, V, ws


@pytest.mark.parametrize("kind", ["ar0.9", "ar0.98", "rising", "together", "one_segment_infinite", "outliers", "levels"])
@pytest.mark.parametrize("rows,n_ctx,budget", [(128, 16384, 256), (9, 16385, 1023), (8, 32768, 2048), (4, 32905, 6219), (3, 3001, 650),
                                               (5, 50001, 70)])
def test_best_that_lie_together(fb, kind, rows, n_ctx, budget):
    print("lists", kind, rows, n_ctx, budget, flush=True)
    run, S, T, out, V, _ = step_of(fb, make_scores(kind, rows, n_ctx, budget), budget)
    for again in range(2):                           # the workspace is left as it has to be
        T.fill_(-1)
        out.fill_(float("nan"))
        run()
        torch.cuda.synchronize()
        some = sorted({0, 1, rows // 2, rows - 1})
        got = np.sort(T[some].cpu().numpy(), -1)
        np.testing.assert_array_equal(got, O.topk(S[some, :, :n_ctx].cpu().numpy(), budget, n_ctx))
        want = V.double()[torch.from_numpy(got[:, 0]).long().cuda()].mean(1)
        # float32 sums of 1e4 terms of at most about 5: well below 1e-4
        assert (out[some, 0].double() - want).abs().max().item() <= 1e-4


def test_ragged_rows_whose_best_lie_together(fb):
    rows, n, budget = 16, 20000, 1500
    lens = [n - 1201 * i for i in range(rows)]
    budgets = [max(1, budget * x // n) if i % 3 else budget for i, x in enumerate(lens)]
    dev = lambda a: torch.tensor(a, dtype=torch.int32, device="cuda")   # noqa: E731
    run, S, T, out, V, _ = step_of(fb, make_scores("ar0.98", rows, n, budget), budget, dev(lens), dev(budgets))
    print("ragged lists", flush=True)
    run()
    torch.cuda.synchronize()
    for r in range(rows):
        b = min(budgets[r], lens[r])
        got = np.sort(T[r, 0, :b].cpu().numpy())
        np.testing.assert_array_equal(got, O.topk(S[r:r + 1, :, :lens[r]].cpu().numpy(), b, lens[r])[0, 0])


def how_selected(ws, rows):
    """Per row: the key from which on its scores were looked at, how it was selected, counts of its list, waits for scores read again."""
    ctl = ws[rows * HIST_BYTES:rows * (HIST_BYTES + CTL_BYTES)].cpu().numpy().view(np.uint32).reshape(rows, -1)
    how = ctl[:, CUT_WORD + 1]
    return ctl[:, CUT_WORD], how & 3, how >> 8 & 255, how >> 16


@pytest.mark.parametrize("rho", [0.0, 0.9, 0.98])
@pytest.mark.parametrize("rows,n_ctx,budget", [(256, 16384, 256), (256, 16383, 1100), (64, 32905, 6219), (64, 50001, 700)])
def test_few_lists_are_short(fb, rows, n_ctx, budget, rho):
    """Lists hold the best of independent scores (one segment in 10^6 has more of them than places); those of rows whose neighbours
    are alike do with their segments' scores read again."""
    print("short lists", rows, n_ctx, budget, rho, flush=True)
    run, S, T, out, V, ws = step_of(fb, make_scores("ar%g" % rho, rows, n_ctx, budget), budget)
    run()
    torch.cuda.synchronize()
    key, way, counts, waits = how_selected(ws, rows)
    cut = np.where(key >> 31, key & 0x7fffffff, ~key).astype(np.uint32).view(np.float32)
    reach = (S[:, 0, :n_ctx].cpu().numpy() >= cut[:, None]).sum(-1)
    print("scores looked at / B: least %.2f, mean %.2f, most %.2f; rows that read again: %d, all: %d; counts %d, waits %d" % (
        reach.min() / budget, reach.mean() / budget, reach.max() / budget, (way == REREAD).sum(), (way == ROW).sum(), counts.max(),
        waits.max()), flush=True)
    assert (reach >= budget).all()
    assert (way == ALONE).all() if rho == 0.0 else (way != ROW).all()


@pytest.mark.parametrize("kind", ["ar0.98", "ar0.998", "rising", "recent"])
@pytest.mark.parametrize("rows,n_ctx,budget", [(8, 32768, 2048), (16, 32905, 6219), (16, 16384, 256), (8, 131072, 1024)])
def test_scores_are_read_again_once(fb, kind, rows, n_ctx, budget):
    """Where segments have more of the best than places, the list is counted three times - from the key that all lists are complete
    from, from the lowest such, and with the scores read again from a key on that B of them should reach - and few segments are read: 32 a
    wait, and those of more than one wait twice."""
    print("read again", kind, rows, n_ctx, budget, flush=True)
    run, S, T, out, V, ws = step_of(fb, make_scores(kind, rows, n_ctx, budget), budget)
    run()
    torch.cuda.synchronize()
    key, way, counts, waits = how_selected(ws, rows)
    print("ways %s, counts %s, waits %s" % (np.bincount(way, minlength=4)[1:], counts, waits), flush=True)
    got = np.sort(T[:2].cpu().numpy(), -1)
    np.testing.assert_array_equal(got, O.topk(S[:2, :, :n_ctx].cpu().numpy(), budget, n_ctx))
    assert (way == REREAD).all()
    assert counts.max() <= 4                         # (one more where the threshold's bin is wide)
    assert waits.max() <= 4


@pytest.mark.parametrize("equal", [False, True])
@pytest.mark.parametrize("lens,n_ctx,budget", [
    ([2049, 2300, 2305, 4096, 8000, 10752, 10753, 20001, 32768], 32768, 2048), ([1500, 6219, 6220, 12001, 17100, 32905, 257, 1], 32905, 6219),
    ([1025, 1200, 8192, 21760, 50001, 99999, 131071, 1], 131072, 1024), ([2049, 5001, 9000, 16383, 16384], 16384, 256)])
def test_short_sequences_of_one_budget(fb, lens, n_ctx, budget, equal):
    """Sequences of other lengths with the budget of the longest: independent scores of each are selected out of its list alone."""
    rows = len(lens)
    dev = lambda a: torch.tensor(a, dtype=torch.int32, device="cuda")   # noqa: E731
    run, S, T, out, V, ws = step_of(fb, make_scores("plain", rows, n_ctx, budget), budget, dev(lens), dev([budget] * rows) if equal else None)
    print("one budget", n_ctx, budget, equal, flush=True)
    for again in range(2):
        T.fill_(-1)
        out.fill_(float("nan"))
        run()
        torch.cuda.synchronize()
        for r, n in enumerate(lens):
            b = min(budget, n)
            got = np.sort(T[r, 0, :b].cpu().numpy())
            np.testing.assert_array_equal(got, O.topk(S[r:r + 1, :, :n].cpu().numpy(), b, n)[0, 0])
            want = V.double()[torch.from_numpy(got).long().cuda()].mean(0)
            assert (out[r, 0].double() - want).abs().max().item() <= 1e-4          # as in test_best_that_lie_together
    way = how_selected(ws, rows)[1]
    assert (way == ALONE).all(), dict(zip(lens, way))


# Where NaN scores rank is unspecified, but a set has B tokens and every call ends: fewer than B finite scores are listed here, in segments
# of NaNs, and the search for the threshold starts at a key below zero, from which bins are wide.  (csrc/abi_host_check.cpp goes through
# the ranges.)
@pytest.mark.parametrize("nan", [0x7fc0, 0xffc0, 0x7fff], ids=hex)
@pytest.mark.parametrize("n_ctx,budget", [(9001, 200), (16384, 700), (20000, 3000)])
def test_nan_scores_end(fb, n_ctx, budget, nan):
    rows = 8
    print("lists, NaN", n_ctx, budget, hex(nan), flush=True)
    scores = np.zeros((rows, n_ctx), dtype=np.float32)
    run, S, T, out, V, ws = step_of(fb, scores, budget, planes=lambda x: _nan_beside_clusters(x, n_ctx, nan))
    for again in range(2):
        T.fill_(-1)
        run()
        torch.cuda.synchronize()
        for r in range(rows):
            t = T[r, 0].long()
            assert t.min() >= 0 and t.max() < n_ctx and t.unique().numel() == budget
            want = V.double()[t].mean(0)
            assert (out[r, 0].double() - want).abs().max().item() <= 1e-4


def _nan_beside_clusters(x, n, nan):
    """Scores of 16 clusters of 16 neighbours, evenly spaced: ordinary, one of a row far above; else NaN."""
    rng = np.random.default_rng(n)
    x[:, 0, :n, 0] = nan
    at = np.concatenate([((n * (2 * c + 1) // 32) & ~15) + np.arange(16) for c in range(16)])
    for r in range(x.shape[0]):
        s = rng.standard_normal(256)
        s[rng.integers(256)] = 100.0
        x[r, 0, at, 0] = W.to_storage(s, "bf16")
