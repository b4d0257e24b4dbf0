"""The memory-optimised step's one-kernel gather + attention at the edges of its tiles and splits, with the
step's append: list lengths around whole tiles, list parts without work for every wave, every storage unit of the
non-dominant dims (F a multiple of 4 or not, none left), both ends of the group size."""
import numpy as np
import pytest
import torch

from oracle import fasa_oracle as O
from paper_2602_03152_amd import workload as W
from tests.test_gpu_offload import OUT_ATOL, _pinned

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def fb():
    from paper_2602_03152_amd import binding
    return binding


@pytest.mark.parametrize("budget", [1, 15, 17, 64, 65, 700])
@pytest.mark.parametrize("kv,group,f", [(1, 1, 16), (3, 8, 6), (8, 4, 63), (2, 2, 64), (1, 4, 1)])
def test_offload_append_at_tile_edges(fb, budget, kv, group, f):
    from tests.gpu_util import Device, to_dev, to_host
    w = W.WORKLOADS[1].scaled(n_ctx=720, budget=budget, n_fc=f, n_kv_heads=kv, n_q_heads=kv * group)
    x = W.make_inputs(w, n_cap=768)
    K, V = x["K"].copy(), x["V"].copy()
    d = Device(w, x)
    nd = w.head_dim - 2 * f
    Knd = _pinned((1, kv, 768, max(nd, 1)), d.st)
    Vh = _pinned(x["V"].shape, d.st)
    Vh.copy_(torch.from_numpy(x["V"].view(np.int16)))
    fb.fasa_offload_split_kcache(d.shape, d.K, d.fc_idx, d.Kp, Knd, 0, w.n_ctx)
    n = w.n_ctx + 1
    shape = d.make_shape(n_ctx=n, budget=budget)
    a = W.make_append(w, x["fc_idx"], step=1, n_before=w.n_ctx)
    # a key along the group's summed query: the new token is always selected, so its row is read back
    qs = a["q"].view(np.uint16).astype(np.uint32) << 16
    qs = qs.view(np.float32).reshape(1, kv, group, -1).sum(2)
    a["k_new"] = (qs.view(np.uint32) >> 16).astype(np.uint16)
    K[:, :, w.n_ctx] = a["k_new"]
    V[:, :, w.n_ctx] = a["v_new"]
    ws_bytes = fb.fasa_workspace_bytes(shape)
    ws = torch.full((ws_bytes,), 0x77, dtype=torch.uint8, device="cuda")
    fb.fasa_workspace_init(shape, ws, ws_bytes)
    stage_bytes = fb.fasa_offload_stage_bytes(shape)
    stage = torch.zeros((stage_bytes,), dtype=torch.uint8, device="cuda")
    T = torch.full((1, kv, budget), -1, dtype=torch.int32, device="cuda")
    for _ in range(2):      # the second call appends the same row again: the workspace was left clean
        d.O.fill_(float("nan"))
        fb.fasa_offload_decode_step(shape, to_dev(a["q"]), d.Kp, d.fc_idx, Knd, Vh, to_dev(a["k_new"]), to_dev(a["v_new"]),
                                    d.S, T, d.O, ws, ws_bytes, stage, stage_bytes)
        torch.cuda.synchronize()
        Kp_ref, Knd_ref = O.split_kcache(K, x["fc_idx"], n)
        np.testing.assert_array_equal(to_host(d.Kp, np.uint16)[:, :, :, :n], Kp_ref)
        if nd:
            np.testing.assert_array_equal(Knd.numpy().view(np.uint16)[:, :, :n], Knd_ref)
        np.testing.assert_array_equal(Vh.numpy().view(np.uint16)[:, :, :n], V[:, :, :n])
        Th = to_host(T)
        np.testing.assert_array_equal(np.sort(Th, -1), O.topk(to_host(d.S)[:, :, :n], budget, n))
        rows = stage.cpu().numpy().view(np.uint16)[: 2 * kv * budget * 128].reshape(2, kv, budget, 128)
        for h in range(kv):
            np.testing.assert_array_equal(rows[0, h], K[0, h][Th[0, h]])
            np.testing.assert_array_equal(rows[1, h], V[0, h][Th[0, h]])
        assert np.abs(to_host(d.O) - O.sparse_attend(a["q"], K, V, Th)).max() <= OUT_ATOL
