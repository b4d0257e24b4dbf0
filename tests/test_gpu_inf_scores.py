"""Infinite scores (finite queries and keys whose products overflow) rank like any others in every form of the decode
step and in the stand-alone selection: the set is the top-B set of the device's own float32 scores, ties to
the lower index.  Among ordinary scores, and among scores that are all equal, where the bins of the adaptive
histogram have no width to go by.  (The attention over an infinite logit is not a number and is not looked at.)"""
import numpy as np
import pytest
import torch

from oracle import fasa_oracle as O
from paper_2602_03152_amd import workload as W
from tests.test_gpu_decode_step import fb, run_step  # noqa: F401

pytestmark = pytest.mark.gpu

BIG = 1e20                      # BIG * BIG overflows float32; the sum of 8 queries of BIG does not


@pytest.mark.parametrize("equal", [False, True], ids=["ordinary", "equal"])
@pytest.mark.parametrize("n_pos,n_neg", [(40, 40), (2000, 10), (0, 1800)])
@pytest.mark.parametrize("kw", [
    dict(cid=1, n_ctx=2011, budget=300), dict(cid=1, n_ctx=7001, budget=300), dict(cid=2, batch=16, n_ctx=8201, budget=300),
    dict(cid=1, n_ctx=9001, budget=700), dict(cid=0, n_ctx=9001, budget=700)], ids=str)
def test_infinite_scores_rank_in_every_form(fb, kw, n_pos, n_neg, equal):  # noqa: F811
    from tests.gpu_util import to_host
    kw = dict(kw); cid = kw.pop("cid")
    w = W.WORKLOADS[cid].scaled(**kw)
    x = W.make_inputs(w, n_cap=(w.n_ctx + 63) // 64 * 64)
    rng = np.random.default_rng(n_pos + n_neg)
    zero, neg, pos = W.to_storage(np.array([0.0, -BIG, BIG]), w.dtype)
    if equal:
        x["K"][:, :, :w.n_ctx] = x["K"][:, :, :1]
    for h in range(w.n_kv_heads):
        dim = x["fc_idx"][h, 0]
        x["q"][:, h * w.group:(h + 1) * w.group, dim] = pos
        if equal:
            x["K"][:, h, :, dim] = zero
        # not among the first tokens of a quarter of the row, which the adaptive histogram samples
        free = np.array([n for n in range(w.n_ctx) if n % max(1, (w.n_ctx >> 2) & ~15) >= 16])
        odd = rng.permutation(free)[:n_pos + n_neg]
        x["K"][:, h, odd[:n_pos], dim] = pos
        x["K"][:, h, odd[n_pos:], dim] = neg
    print("infinite scores", kw, n_pos, n_neg, equal, flush=True)
    d = run_step(fb, w, x)
    S = to_host(d.S)[:, :, :w.n_ctx]
    assert np.isposinf(S).any() == (n_pos > 0) and np.isneginf(S).any() == (len(odd) > n_pos)
    want = O.topk(S, w.budget, w.n_ctx)
    np.testing.assert_array_equal(np.sort(to_host(d.T), -1), want)
    d.T.fill_(-1)
    fb.fasa_topk(d.shape, d.S, d.T, d.ws, d.ws_bytes)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(np.sort(to_host(d.T), -1), want)


@pytest.mark.parametrize("append", [False, True], ids=["", "append"])
@pytest.mark.parametrize("n_fc", [4, 7, 12, 13, 20])
@pytest.mark.parametrize("n_ctx", [2011, 9001], ids=["one_launch", "lists"])
def test_infinite_keys_of_the_last_listed_pair(fb, n_ctx, n_fc, append):  # noqa: F811
    """List lengths that are no multiple of the planes in flight: an infinite key makes an infinite score, and no NaN."""
    from tests.gpu_util import to_host
    w = W.WORKLOADS[1].scaled(n_ctx=n_ctx, budget=300, n_fc=n_fc)
    x = W.make_inputs(w, n_cap=(n_ctx + 63) // 64 * 64)
    rng = np.random.default_rng(n_fc)
    one, neg, pos = W.to_storage(np.array([1.0, -np.inf, np.inf]), w.dtype)
    odd = rng.permutation(n_ctx - 1)[:90]
    for h in range(w.n_kv_heads):
        dim = x["fc_idx"][h, n_fc - 1]
        x["q"][:, h * w.group:(h + 1) * w.group, dim] = one
        x["K"][:, h, odd[:40], dim] = pos
        x["K"][:, h, odd[40:], dim] = neg
    new = {k: x[k[0].upper()][:, :, n_ctx - 1].copy() for k in ("k_new", "v_new")} if append else {}
    print("infinite keys", n_ctx, n_fc, append, flush=True)
    d = run_step(fb, w, x, **new)
    S = to_host(d.S)[:, :, :n_ctx]
    assert np.isposinf(S[:, :, odd[:40]]).all() and np.isneginf(S[:, :, odd[40:]]).all()
    assert not np.isnan(S).any()
    np.testing.assert_array_equal(np.sort(to_host(d.T), -1), O.topk(S, w.budget, n_ctx))
