"""GPU parity of the forms the decode step takes by size - one launch (one or several slices per row), one
workgroup per row after the scoring launch, and the split selection and attention - at the edges where one
goes over into the next, with an appended row, and with tied scores in each."""
import numpy as np
import pytest

from paper_2602_03152_amd import workload as W
from tests.test_gpu_decode_step import _tied_inputs, compare_step, fb, run_step  # noqa: F401

pytestmark = pytest.mark.gpu

EDGES = [
    # one slice: first and last tokens of a wave, of the slice, and one past it
    dict(cid=1, n_ctx=2, budget=1), dict(cid=1, n_ctx=63, budget=17), dict(cid=1, n_ctx=257, budget=16),
    dict(cid=1, n_ctx=2047, budget=128), dict(cid=1, n_ctx=2048, budget=1024), dict(cid=1, n_ctx=2049, budget=129),
    # several slices, up to the budget and length where the split form takes over
    dict(cid=1, n_ctx=4097, budget=320), dict(cid=1, n_ctx=4097, budget=321), dict(cid=1, n_ctx=8192, budget=15),
    dict(cid=1, n_ctx=8193, budget=15), dict(cid=3, batch=1, n_ctx=6001, budget=255),
    dict(cid=0, n_ctx=1024, budget=512), dict(cid=0, n_ctx=1025, budget=513), dict(cid=0, n_ctx=8192, budget=33),
    dict(cid=0, n_ctx=3000, budget=64, n_kv_heads=2, n_q_heads=10),
    # one workgroup per row: 128 rows, lengths around its register stretch of 16384 and the largest budget
    dict(cid=2, n_ctx=8192, budget=1024), dict(cid=2, batch=32, n_kv_heads=4, n_q_heads=4, n_ctx=16385, budget=257),
    dict(cid=2, batch=64, n_kv_heads=2, n_q_heads=14, n_ctx=8200, budget=1025),
    dict(cid=0, batch=128, n_ctx=2111, budget=40), dict(cid=0, batch=64, n_kv_heads=2, n_q_heads=16, n_ctx=1500, budget=65),
]


def _id(kw):
    return "_".join("%s%s" % (k, v) for k, v in kw.items())


def _sample(w):
    return list(range(w.batch)) if w.batch <= 2 else [0, w.batch // 2, w.batch - 1]


@pytest.mark.parametrize("kw", EDGES, ids=_id)
def test_step_at_the_edges_of_the_forms(fb, kw):  # noqa: F811
    from tests.gpu_util import to_host
    kw = dict(kw); cid = kw.pop("cid")
    w = W.WORKLOADS[cid].scaled(**kw)
    x = W.make_inputs(w, n_cap=(w.n_ctx + 63) // 64 * 64)
    print("edge", kw, flush=True)
    app = W.make_append(w, x["fc_idx"], 1, w.n_ctx - 1)
    d = run_step(fb, w, x, k_new=app["k_new"], v_new=app["v_new"], q=app["q"])
    K, V = x["K"].copy(), x["V"].copy()
    K[:, :, w.n_ctx - 1] = app["k_new"]
    V[:, :, w.n_ctx - 1] = app["v_new"]
    assert np.array_equal(to_host(d.K, K.dtype), K) and np.array_equal(to_host(d.V, V.dtype), V)
    compare_step(w, app["q"], K, V, x["fc_idx"], d, w.n_ctx, w.budget, rows=_sample(w))


@pytest.mark.parametrize("n_classes", [1, 8, 40, 300])
@pytest.mark.parametrize("kw", [
    dict(cid=1, n_ctx=1900, budget=300), dict(cid=1, n_ctx=7000, budget=300), dict(cid=0, n_ctx=5000, budget=400),
    dict(cid=2, batch=16, n_ctx=8200, budget=500), dict(cid=1, n_ctx=9000, budget=700),
    dict(cid=3, batch=1, n_ctx=5000, budget=900)], ids=_id)
def test_tied_scores_in_every_form(fb, kw, n_classes):  # noqa: F811
    kw = dict(kw); cid = kw.pop("cid")
    w = W.WORKLOADS[cid].scaled(**kw)
    x = _tied_inputs(w, n_classes, seed=n_classes)
    print("tied", kw, n_classes, flush=True)
    d = run_step(fb, w, x)
    compare_step(w, x["q"], x["K"], x["V"], x["fc_idx"], d, w.n_ctx, w.budget, rows=_sample(w))


def test_new_row_is_selected_from_where_it_is_handed_in(fb):  # noqa: F811
    """The appended row scores highest, so every head attends to it: its K and V have to come through
    whatever the caches held there before (another row's values are planted in its place)."""
    from tests.gpu_util import to_host
    for n_ctx, budget in [(1000, 40), (5003, 100)]:
        w = W.WORKLOADS[1].scaled(n_ctx=n_ctx, budget=budget)
        x = W.make_inputs(w, n_cap=(w.n_ctx + 63) // 64 * 64)
        q = W.storage_to_f64(x["q"]).reshape(1, w.n_kv_heads, w.group, w.head_dim)
        k_new = W.to_storage(q.sum(axis=2), w.dtype)
        v_new = x["V"][:, :, 7].copy()
        d = run_step(fb, w, x, k_new=k_new, v_new=v_new)
        T = to_host(d.T).reshape(w.n_kv_heads, budget)
        assert all(n_ctx - 1 in T[h] for h in range(w.n_kv_heads))
        K, V = x["K"].copy(), x["V"].copy()
        K[:, :, n_ctx - 1], V[:, :, n_ctx - 1] = k_new, v_new
        compare_step(w, x["q"], K, V, x["fc_idx"], d, n_ctx, budget)
