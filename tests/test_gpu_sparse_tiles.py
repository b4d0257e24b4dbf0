"""Attention over a list long enough to be split more than 40 ways (bf16: eight waves per workgroup): lists that end inside a
tile, at a split's edge and past it, waves with no tile, one and two; pool slots of a paged cache; sequences of a batch that
leave whole splits empty."""
import numpy as np
import pytest
import torch

from oracle import fasa_oracle as O
from paper_2602_03152_amd import workload as W
from tests.test_gpu_decode_step import compare_step, fb  # noqa: F401
from tests.test_gpu_paged import PagedDevice
from tests.test_gpu_ragged import i32_dev

pytestmark = pytest.mark.gpu


def _inputs(w):
    return W.make_inputs(w, n_cap=(w.n_ctx + 63) // 64 * 64)


@pytest.mark.parametrize("heads", [(1, 1), (4, 1), (7, 1), (10, 2), (8, 1)])
@pytest.mark.parametrize("budget", [2560, 2561, 2625, 9000, 20001, 33000])
def test_list_at_the_edges_of_the_tiles(fb, heads, budget):  # noqa: F811
    from tests.gpu_util import Device, to_host
    w = W.WORKLOADS[1].scaled(batch=1, n_ctx=33017, budget=budget, n_q_heads=heads[0], n_kv_heads=heads[1])
    x = _inputs(w)
    rng = np.random.default_rng(budget)
    T = np.stack([rng.permutation(w.n_ctx)[:budget] for _ in range(heads[1])])[None].astype(np.int32)
    print("sparse", heads, budget, flush=True)
    d = Device(w, x)
    d.T.copy_(torch.from_numpy(T))
    fb.fasa_sparse_attend(d.shape, d.q, d.K, d.V, d.T, d.O, d.ws, d.ws_bytes)
    torch.cuda.synchronize()
    ref = O.sparse_attend(x["q"], x["K"], x["V"], T)
    assert np.abs(to_host(d.O) - ref).max() <= 2e-3


@pytest.mark.parametrize("page,layout", [(16, "token_major"), (64, "head_major")])
def test_list_of_pool_slots(fb, page, layout):  # noqa: F811
    w = W.WORKLOADS[1].scaled(batch=1, n_ctx=9001, budget=9001, n_q_heads=8, n_kv_heads=2)
    x = _inputs(w)
    print("slots", page, layout, flush=True)
    d = PagedDevice(fb, w, x, page, layout)
    fb.fasa_pack_kcache_paged(d.shape, d.paging, d.K, d.fc_idx, d.Kp, 0, w.n_ctx)
    fb.fasa_decode_step_paged(d.shape, d.paging, d.q, d.K, d.V, d.Kp, d.fc_idx, None, None, None, None,
                              d.S, d.T, d.O, d.ws, d.ws_bytes)
    torch.cuda.synchronize()
    compare_step(w, x["q"], x["K"], x["V"], x["fc_idx"], d, w.n_ctx, w.budget)


def test_list_with_empty_splits(fb):  # noqa: F811
    """Rows of more than 2^20 tokens run the stages one after another; a short second sequence leaves most of its splits empty.
    (Drawn on the GPU, one K and V for both sequences: the reference is float64 torch.)"""
    D, n, B, lens, budgets = 128, (1 << 20) + 1, 9000, [(1 << 20) + 1, 40000], [9000, 300]
    cap = (n + 63) // 64 * 64
    print("empty splits", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(11)
    rnd = lambda *s: torch.randn(*s, generator=gen, device="cuda").bfloat16()   # noqa: E731
    q, K, V, Kp = rnd(2, 4, D), rnd(cap, D), rnd(cap, D), rnd(2, 1, 8, cap, 2)
    fc = torch.arange(8, dtype=torch.int32, device="cuda")
    shape = fb.make_shape(2, 4, 1, D, 8, n, cap, B, "bf16", kv_stride_b=0, kv_stride_h=0, kv_stride_n=D)
    ws = torch.empty(fb.fasa_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    fb.fasa_workspace_init(shape, ws, ws.numel())
    S = torch.zeros(2, 1, cap, device="cuda")
    T = torch.full((2, 1, B), -1, dtype=torch.int32, device="cuda")
    out = torch.full((2, 4, D), float("nan"), device="cuda")
    fb.fasa_profile_reset()
    fb.fasa_profile_enable(True)
    try:
        for _ in range(2):                            # the workspace is left as it has to be
            fb.fasa_decode_step_ragged(shape, q, K, V, Kp, fc, None, None, i32_dev(lens), i32_dev(budgets), S, T, out, ws, ws.numel())
        torch.cuda.synchronize()
        names = set(fb.profile_summary())
    finally:
        fb.fasa_profile_enable(False)
        fb.fasa_profile_reset()
    assert "fasa_sparse_attend" in names and "fasa_select_attend" not in names and "fasa_list" not in names, names
    for b in range(2):
        t = T[b, 0, :budgets[b]].long()
        assert t.min() >= 0 and t.max() < lens[b] and t.unique().numel() == budgets[b]
        best = S[b, 0, :lens[b]].topk(budgets[b]).values
        assert torch.equal(S[b, 0, t].sort(descending=True).values, best)
        p = torch.softmax(q[b].double() @ K[t].double().T / D ** 0.5, -1)
        assert (out[b].double() - p @ V[t].double()).abs().max().item() <= 2e-3
