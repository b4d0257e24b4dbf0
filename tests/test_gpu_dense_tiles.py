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


@pytest.mark.parametrize("batch,heads,n_ctx", [(17, (32, 8), 1300), (33, (16, 8), 1040), (129, (7, 1), 2050), (20, (8, 8), 777)])
def test_dense_rows_around_the_compute_units(fb, batch, heads, n_ctx):  # noqa: F811
    """129 to 264 rows: several workgroups a row where one would leave half of the compute units idle."""
    from tests.gpu_util import Device, to_host
    w = W.WORKLOADS[1].scaled(batch=1, n_ctx=n_ctx, budget=n_ctx, n_q_heads=heads[0], n_kv_heads=heads[1])
    x = W.make_inputs(w, n_cap=(n_ctx + 63) // 64 * 64)
    # one sequence, its tokens in another rotation for every entry of the batch: the same attention
    for name in ("K", "V"):
        x[name] = np.stack([np.concatenate([np.roll(x[name][0][:, :n_ctx], 13 * b, axis=1), x[name][0][:, n_ctx:]], axis=1)
                            for b in range(batch)])
    ref = O.dense_attend(x["q"], x["K"][:1], x["V"][:1], n_ctx)
    x["q"] = np.repeat(x["q"], batch, axis=0)
    print("dense rows", batch, heads, n_ctx, flush=True)
    d = Device(w.scaled(batch=batch), x)
    fb.fasa_dense_attend(d.shape, d.q, d.K, d.V, d.O, d.ws, d.ws_bytes)
    torch.cuda.synchronize()
    assert np.abs(to_host(d.O) - ref).max() <= 2e-3


# full KV of few splits: which kernel is told by its partials' number, so both sides of each line are compared with the oracle
@pytest.mark.parametrize("batch,heads,n_ctx", [
    (1, (10, 2), 1024), (1, (10, 2), 1025), (1, (32, 8), 1024), (1, (32, 8), 1025), (4, (8, 4), 1024), (4, (8, 4), 1025), (4, (20, 5), 832)])
def test_dense_at_the_lines_of_short_rows(fb, batch, heads, n_ctx):  # noqa: F811
    from tests.gpu_util import Device, to_host
    w = W.WORKLOADS[1].scaled(batch=batch, n_ctx=n_ctx, budget=n_ctx, n_q_heads=heads[0], n_kv_heads=heads[1])
    x = W.make_inputs(w, n_cap=(n_ctx + 63) // 64 * 64)
    print("dense lines", batch, heads, n_ctx, flush=True)
    d = Device(w, x)
    fb.fasa_dense_attend(d.shape, d.q, d.K, d.V, d.O, d.ws, d.ws_bytes)
    torch.cuda.synchronize()
    assert np.abs(to_host(d.O) - O.dense_attend(x["q"], x["K"], x["V"], n_ctx)).max() <= 2e-3
