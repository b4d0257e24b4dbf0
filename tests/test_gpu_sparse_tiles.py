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
from tests.test_gpu_ragged import compare_ragged, i32_dev

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
    from tests.gpu_util import Device
    lens, budgets = [524289, 40000], [9000, 300]     # (too long for the step's two-launch forms)
    w = W.WORKLOADS[1].scaled(batch=2, n_ctx=524289, budget=9000, n_q_heads=4, n_kv_heads=1)
    x = _inputs(w)
    print("empty splits", flush=True)
    d = Device(w, x)
    d.pack()
    fb.fasa_decode_step_ragged(d.shape, d.q, d.K, d.V, d.Kp, d.fc_idx, None, None, i32_dev(lens), i32_dev(budgets),
                               d.S, d.T, d.O, d.ws, d.ws_bytes)
    torch.cuda.synchronize()
    compare_ragged(w, x["q"], x["K"], x["V"], x["fc_idx"], d, lens, budgets, 9000)
