"""Scoring with eight planes in flight (list lengths without an instance of their own, and 32 planes on a grid of
more than one workgroup per CU): remainders of the eight planes, the appended token in every place of a thread's
tokens, against the oracle, and the step built on it."""
import numpy as np
import pytest
import torch

from oracle import fasa_oracle as O
from paper_2602_03152_amd import workload as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("f,n,kv", [(1, 1030, 2), (7, 2049, 2), (9, 9002, 1), (12, 9003, 1), (17, 9004, 1), (40, 9001, 1),
                                    (64, 2050, 2), (32, 32770, 8)])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_any_number_of_planes(f, n, kv, dtype):
    from paper_2602_03152_amd import binding as fb
    from tests.gpu_util import Device, to_dev, to_host
    w = W.WORKLOADS[1].scaled(n_ctx=n, budget=max(8, n // 20), n_fc=f, n_kv_heads=kv, n_q_heads=4 * kv, dtype=dtype)
    x = W.make_inputs(w, n_cap=(n + 64) // 64 * 64)
    d = Device(w, x)
    fb.fasa_pack_kcache(d.shape, d.K, d.fc_idx, d.Kp, 0, n)
    fb.fasa_score(d.shape, d.q, d.Kp, d.fc_idx, d.S)
    torch.cuda.synchronize()
    S = to_host(d.S)[:, :, :n].copy()
    S_ref, D_ref = O.score(x["q"], x["K"], x["fc_idx"], n)
    assert np.all(np.abs(S - S_ref) <= 1e-5 * np.maximum(np.abs(S_ref), D_ref))
    # the step appends the last token again, into planes that do not hold it: the same scores bit for bit
    k_new, v_new = x["K"][:, :, n - 1].copy(), x["V"][:, :, n - 1].copy()
    d.Kp[:, :, :, n - 1].zero_()
    d.S.fill_(float("nan"))
    fb.fasa_decode_step(d.shape, d.q, d.K, d.V, d.Kp, d.fc_idx, to_dev(k_new), to_dev(v_new), d.S, d.T, d.O, d.ws, d.ws_bytes)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(to_host(d.S)[:, :, :n], S)
    T = to_host(d.T)
    np.testing.assert_array_equal(np.sort(T, -1), O.topk(S, w.budget, n))
    assert np.abs(to_host(d.O) - O.sparse_attend(x["q"], x["K"], x["V"], T)).max() <= 2e-3
