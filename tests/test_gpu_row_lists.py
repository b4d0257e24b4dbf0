"""The decode step whose second launch selects out of the lists that the scoring launch makes (bf16): lengths around its
workgroups' 1024 tokens and their segments of 256, budgets around its workgroups' shares, every number of entries per thread it is built
for; winners that crowd a few segments (their scores are read again), or a few places of many, and sequences of a token to a few
segments.  The parity bar is the step's."""
import numpy as np
import pytest
import torch

from paper_2602_03152_amd import workload as W
from tests.test_gpu_decode_step import compare_step, fb, run_step  # noqa: F401

pytestmark = pytest.mark.gpu

EDGES = [
    dict(n_ctx=2049, budget=2048), dict(n_ctx=2050, budget=1025), dict(n_ctx=3072, budget=321), dict(n_ctx=4097, budget=63),
    dict(n_ctx=5120, budget=256), dict(n_ctx=5121, budget=257), dict(n_ctx=8191, budget=1), dict(n_ctx=8193, budget=4097),
    dict(n_ctx=9216, budget=2048), dict(n_ctx=12289, budget=6000), dict(n_ctx=20011, budget=64),
    # F without an instance of its own, one with 32 planes, other groups, row counts that are no multiple of 8
    dict(n_ctx=7001, budget=900, n_fc=12), dict(n_ctx=7001, budget=900, n_fc=45), dict(n_ctx=7001, budget=900, n_fc=32),
    dict(n_ctx=6143, budget=700, n_kv_heads=3, n_q_heads=3), dict(n_ctx=6145, budget=511, n_kv_heads=2, n_q_heads=16, batch=3),
    # one workgroup per row, and a few of a batch's rows each
    dict(n_ctx=5121, budget=300, batch=9), dict(n_ctx=6000, budget=700, batch=33), dict(n_ctx=9000, budget=200, batch=5),
]


def _inputs(w):
    return W.make_inputs(w, n_cap=(w.n_ctx + 63) // 64 * 64)


def _rows(w):
    return None if w.batch <= 3 else [0, w.batch - 1]


@pytest.mark.parametrize("kw", EDGES, ids=lambda kw: "_".join("%s%s" % i for i in kw.items()))
def test_lists_at_their_edges(fb, kw):  # noqa: F811
    w = W.WORKLOADS[1].scaled(**kw)
    x = _inputs(w)
    print("lists", kw, flush=True)
    app = W.make_append(w, x["fc_idx"], 1, w.n_ctx - 1)
    d = run_step(fb, w, x, k_new=app["k_new"], v_new=app["v_new"], q=app["q"])
    K, V = x["K"].copy(), x["V"].copy()
    K[:, :, w.n_ctx - 1], V[:, :, w.n_ctx - 1] = app["k_new"], app["v_new"]
    compare_step(w, app["q"], K, V, x["fc_idx"], d, w.n_ctx, w.budget, rows=_rows(w))


def _raise_scores(w, x, tokens):
    """Adds the group's mean query to the keys at `tokens`: they score far above the rest."""
    q = W.storage_to_f64(x["q"]).reshape(w.batch, w.n_kv_heads, w.group, w.head_dim).mean(axis=2)
    K = W.storage_to_f64(x["K"])
    K[:, :, tokens] += 0.7 * q[:, :, None, :]
    x["K"] = W.to_storage(K, w.dtype)


@pytest.mark.parametrize("n_ctx,budget,first,last", [(9000, 900, 7800, 9000), (9000, 900, 0, 1000), (30000, 250, 2048, 2400),
                                                     (16384, 4000, 9000, 13300)])
def test_winners_in_few_segments(fb, n_ctx, budget, first, last):  # noqa: F811
    w = W.WORKLOADS[1].scaled(n_ctx=n_ctx, budget=budget)
    x = _inputs(w)
    _raise_scores(w, x, np.arange(first, last))
    print("crowded", n_ctx, budget, first, last, flush=True)
    d = run_step(fb, w, x)
    compare_step(w, x["q"], x["K"], x["V"], x["fc_idx"], d, w.n_ctx, w.budget)


@pytest.mark.parametrize("n_ctx,budget,batch", [(9000, 700, 1), (9000, 200, 1), (20000, 3000, 1), (6000, 700, 33)])
def test_clusters_above_all_others(fb, n_ctx, budget, batch):  # noqa: F811
    """16 clusters of 16 neighbours, evenly spaced, score above all others: the cut of a segment lies far below its best."""
    w = W.WORKLOADS[1].scaled(n_ctx=n_ctx, budget=budget, batch=batch)
    x = _inputs(w)
    starts = [(n_ctx * (2 * c + 1) // 32) & ~15 for c in range(16)]
    _raise_scores(w, x, np.concatenate([np.arange(s, s + 16) for s in starts]))
    print("clusters", n_ctx, budget, batch, flush=True)
    d = run_step(fb, w, x)
    compare_step(w, x["q"], x["K"], x["V"], x["fc_idx"], d, w.n_ctx, w.budget, rows=_rows(w))


def test_sequences_of_any_length(fb):  # noqa: F811
    from tests.gpu_util import Device
    from tests.test_gpu_ragged import compare_ragged, i32_dev
    lens, budgets = [9001, 1, 130, 1024, 1023, 5000, 2048], [700, 5, 129, 1000, 1, 4999, 2048]
    w = W.WORKLOADS[1].scaled(batch=len(lens), n_ctx=max(lens), budget=5000)
    x = _inputs(w)
    d = Device(w, x)
    d.pack()
    shape = d.make_shape()
    print("ragged lists", flush=True)
    for _ in range(2):                                            # the second call on what the first one left
        fb.fasa_decode_step_ragged(shape, d.q, d.K, d.V, d.Kp, d.fc_idx, None, None, i32_dev(lens), i32_dev(budgets), d.S, d.T,
                                   d.O, d.ws, d.ws_bytes)
    torch.cuda.synchronize()
    compare_ragged(w, x["q"], x["K"], x["V"], x["fc_idx"], d, lens, budgets, 5000)
