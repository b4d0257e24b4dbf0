"""Full-KV attention at the edges of its tile loop: lists that end inside a tile, at one, and one past it, for waves with no
tile, one, two and several, and logits that grow so that the running maximum moves in every tile."""
import numpy as np
import pytest
import torch

from oracle import fasa_oracle as O
from paper_2602_03152_amd import workload as W
from tests.test_gpu_decode_step import fb  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cid,heads", [(1, (8, 2)), (3, (7, 1)), (1, (8, 8)), (0, (8, 2)), (0, (2, 2))])
@pytest.mark.parametrize("n_ctx", [1, 16, 17, 63, 65, 1023, 1025, 16384, 20011])
def test_dense_at_the_edges_of_the_tiles(fb, cid, heads, n_ctx):  # noqa: F811
    from tests.gpu_util import Device, to_host
    w = W.WORKLOADS[cid].scaled(batch=1, n_ctx=n_ctx, budget=1, n_q_heads=heads[0], n_kv_heads=heads[1])
    x = W.make_inputs(w, n_cap=(n_ctx + 63) // 64 * 64)
    # later keys lean further towards the queries: the maximum is met late, and moves all the way
    K = W.storage_to_f64(x["K"])
    lean = W.storage_to_f64(x["q"]).reshape(1, heads[1], -1, 128).mean(axis=2)
    K[:, :, :n_ctx] += (0.05 * np.arange(n_ctx) / n_ctx)[None, None, :, None] * lean[:, :, None, :]
    x["K"] = W.to_storage(K, w.dtype)
    print("dense", cid, heads, n_ctx, flush=True)
    d = Device(w, x)
    shape = d.make_shape(budget=n_ctx)
    ws = torch.empty((fb.fasa_workspace_bytes(shape),), dtype=torch.uint8, device="cuda")
    fb.fasa_workspace_init(shape, ws, ws.numel())
    fb.fasa_dense_attend(shape, d.q, d.K, d.V, d.O, ws, ws.numel())
    torch.cuda.synchronize()
    ref = O.dense_attend(x["q"], x["K"], x["V"], n_ctx)
    assert np.abs(to_host(d.O) - ref).max() <= 2e-3
