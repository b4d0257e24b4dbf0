"""The split form of the step (a scoring launch with a histogram, then one kernel that selects and attends by token ranges) on
bf16 caches: the shapes whose lists of large scores are too long, or whose workgroups' shares of the set are.  Every
instance by tokens per workgroup, group sizes, an appended row, paged and ragged caches, ties and infinite scores; which
kernels ran is asserted each time."""
import numpy as np
import pytest
import torch

from oracle import fasa_oracle as O
from paper_2602_03152_amd import workload as W
from tests.test_gpu_decode_step import _tied_inputs, compare_step, fb, run_step  # noqa: F401
from tests.test_gpu_paged import PagedDevice
from tests.test_gpu_ragged import compare_ragged, i32_dev
from tests.test_gpu_row_form import _inputs

pytestmark = pytest.mark.gpu


def recorded(fb, f):  # noqa: F811
    """f(), with the split form's kernels and no other selecting ones."""
    fb.fasa_profile_reset()
    fb.fasa_profile_enable(True)
    try:
        out = f()
        torch.cuda.synchronize()
        names = set(fb.profile_summary())
    finally:
        fb.fasa_profile_enable(False)
        fb.fasa_profile_reset()
    assert {"fasa_score_hist", "fasa_select_attend"} <= names and not names & {"fasa_list", "fasa_score_list", "fasa_sparse_attend"}, names
    return out


# (batch, query heads, KV heads, tokens, budget): long lists (slices of 1008 tokens: the 1024-token instance), then shares of more
# than 2048 with slices of 1264, 2256 and 3104 (the 2048-, 3072- and 4096-token instances)
@pytest.mark.parametrize("append", [False, True], ids=["", "append"])
@pytest.mark.parametrize("batch,hq,hkv,n_ctx,budget", [
    (1, 1, 1, 20000, 9000), (1, 8, 2, 20001, 9000), (1, 7, 1, 19999, 9001), (2, 8, 1, 20011, 9500),
    (16, 32, 8, 5000, 4100), (64, 4, 2, 5003, 4097), (32, 12, 4, 9000, 4200), (16, 40, 8, 12400, 4200)], ids=str)
def test_every_instance(fb, batch, hq, hkv, n_ctx, budget, append):  # noqa: F811
    w = W.WORKLOADS[1].scaled(batch=batch, n_q_heads=hq, n_kv_heads=hkv, n_ctx=n_ctx, budget=budget)
    x = _inputs(w)
    print("split", batch, hq, hkv, n_ctx, budget, append, flush=True)
    new = dict(k_new=x["K"][:, :, 5].copy(), v_new=x["V"][:, :, 7].copy()) if append else {}
    d = recorded(fb, lambda: run_step(fb, w, x, **new))
    if append:
        x["K"][:, :, n_ctx - 1], x["V"][:, :, n_ctx - 1] = new["k_new"], new["v_new"]
    compare_step(w, x["q"], x["K"], x["V"], x["fc_idx"], d, n_ctx, budget, rows=sorted({0, batch // 2, batch - 1}))


@pytest.mark.parametrize("n_classes", [1, 8, 300])
def test_ties(fb, n_classes):  # noqa: F811
    w = W.WORKLOADS[1].scaled(batch=1, n_q_heads=4, n_kv_heads=1, n_ctx=20000, budget=9000)
    x = _tied_inputs(w, n_classes, seed=n_classes)
    print("split, ties", n_classes, flush=True)
    d = recorded(fb, lambda: run_step(fb, w, x))
    compare_step(w, x["q"], x["K"], x["V"], x["fc_idx"], d, w.n_ctx, w.budget)


@pytest.mark.parametrize("n_pos,n_neg", [(40, 40), (9500, 10), (0, 11500)])
def test_infinite_scores(fb, n_pos, n_neg):  # noqa: F811
    from tests.gpu_util import to_host
    w = W.WORKLOADS[1].scaled(batch=1, n_q_heads=8, n_kv_heads=2, n_ctx=20000, budget=9000)
    x = W.make_inputs(w, n_cap=20032)
    neg, pos = W.to_storage(np.array([-1e20, 1e20]), w.dtype)
    odd = np.random.default_rng(n_pos).permutation(w.n_ctx)[:n_pos + n_neg]
    for h in range(2):
        dim = x["fc_idx"][h, 0]
        x["q"][:, 4 * h:4 * h + 4, dim] = pos                 # (products overflow, the sum of the group's queries does not)
        x["K"][:, h, odd[:n_pos], dim] = pos
        x["K"][:, h, odd[n_pos:], dim] = neg
    print("split, infinite scores", n_pos, n_neg, flush=True)
    d = recorded(fb, lambda: run_step(fb, w, x))
    S = to_host(d.S)[:, :, :w.n_ctx]
    assert np.isposinf(S).any() == (n_pos > 0) and np.isneginf(S).any()
    np.testing.assert_array_equal(np.sort(to_host(d.T), -1), O.topk(S, w.budget, w.n_ctx))


@pytest.mark.parametrize("page", [0, 16, 64])
def test_ragged_and_paged(fb, page):  # noqa: F811
    from tests.gpu_util import Device
    lens, budgets = [20000, 300, 15001], [9000, 9000, 33]
    w = W.WORKLOADS[1].scaled(batch=3, n_q_heads=4, n_kv_heads=1, n_ctx=20000, budget=9000)
    x = W.make_inputs(w, n_cap=20032)
    print("split, ragged", page, flush=True)
    if page:
        d = PagedDevice(fb, w, x, page, "token_major")
        fb.fasa_pack_kcache_paged(d.shape, d.paging, d.K, d.fc_idx, d.Kp, 0, w.n_ctx)
        recorded(fb, lambda: fb.fasa_decode_step_paged(d.shape, d.paging, d.q, d.K, d.V, d.Kp, d.fc_idx, None, None, i32_dev(lens),
                                                       i32_dev(budgets), d.S, d.T, d.O, d.ws, d.ws_bytes))
    else:
        d = Device(w, x)
        d.pack()
        recorded(fb, lambda: fb.fasa_decode_step_ragged(d.shape, d.q, d.K, d.V, d.Kp, d.fc_idx, None, None, i32_dev(lens), i32_dev(budgets),
                                                        d.S, d.T, d.O, d.ws, d.ws_bytes))
    compare_ragged(w, x["q"], x["K"], x["V"], x["fc_idx"], d, lens, budgets, 9000)
