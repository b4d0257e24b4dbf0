"""Calls that read 90 MiB and more read their planes, their gathered values or their full KV non-temporal: odd lengths on that side of the lines, every
list length with an instance of its own, against torch (scores and attention in float64; the set by the scores the device itself wrote)."""
import pytest
import torch

pytestmark = pytest.mark.gpu

D = 128


def _tensors(batch, hq, hkv, f, n, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    cap = (n + 63) // 64 * 64
    rnd = lambda *s: torch.randn(*s, generator=gen, device="cuda").bfloat16()   # noqa: E731
    fc = torch.rand(hkv, D // 2, generator=gen, device="cuda").argsort(dim=-1)[:, :f].to(torch.int32).contiguous()
    return rnd(batch, hq, D), rnd(batch, hkv, cap, D), rnd(batch, hkv, cap, D), fc, cap


def _attention(q, K, V):
    """q [G][D], K, V [n][D] -> [G][D] in float64"""
    p = torch.softmax(q.double() @ K.double().T / D ** 0.5, dim=-1)
    return p @ V.double()


# 2^-16 of a weight is dropped where the matrix cores take it, against values of about 5 at most; logits of a few tens in float32
TOL = 2e-4


@pytest.mark.parametrize("batch,hq,hkv,f,n,budget,append", [
    (32, 16, 8, 8, 10001, 64, True), (24, 8, 4, 12, 20011, 300, True), (12, 32, 8, 16, 16383, 1000, False),
    (16, 14, 2, 24, 33001, 2500, True), (4, 8, 8, 32, 24577, 500, True), (8, 28, 4, 16, 32905, 6219, True), (8, 8, 4, 16, 20000, 7000, False)])
def test_step(batch, hq, hkv, f, n, budget, append):
    from paper_2602_03152_amd import binding as fb
    q, K, V, fc, cap = _tensors(batch, hq, hkv, f, n, 7)
    rows, G = batch * hkv, hq // hkv
    assert rows * (n * (4 * f + 4) + budget * 512) >= 90 << 20
    shape = fb.make_shape(batch, hq, hkv, D, f, n, cap, budget, "bf16")
    Kp = torch.zeros(batch, hkv, f, cap, 2, dtype=torch.bfloat16, device="cuda")
    S = torch.full((batch, hkv, cap), float("nan"), device="cuda")
    T = torch.full((batch, hkv, budget), -1, dtype=torch.int32, device="cuda")
    out = torch.full((batch, hq, D), float("nan"), device="cuda")
    k_new, v_new = (torch.randn(batch, hkv, D, device="cuda").bfloat16() for _ in range(2)) if append else (None, None)
    ws = torch.empty(fb.fasa_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    fb.fasa_workspace_init(shape, ws, ws.numel())
    fb.fasa_pack_kcache(shape, K, fc, Kp, 0, n)
    print("stream step", batch, hq, hkv, f, n, budget, append, flush=True)
    fb.fasa_decode_step(shape, q, K, V, Kp, fc, k_new, v_new, S, T, out, ws, ws.numel())
    torch.cuda.synchronize()
    if append:
        assert torch.equal(K[:, :, n - 1], k_new) and torch.equal(V[:, :, n - 1], v_new)
    for b in range(batch):
        for h in range(hkv):
            i = fc[h].long()
            dims = torch.cat([i, i + D // 2])
            qs = q[b, h * G:(h + 1) * G].double().sum(0)[dims]
            k = K[b, h, :n][:, dims].double()
            s = S[b, h, :n]
            assert ((s.double() - k @ qs).abs() <= 1e-5 * (k.abs() @ qs.abs())).all(), (b, h)
            t = T[b, h].long()
            inside = torch.zeros(n, dtype=torch.bool, device="cuda")
            inside[t] = True
            assert int(inside.sum()) == budget and float(s[inside].min()) >= float(s[~inside].max()), (b, h)
            ref = _attention(q[b, h * G:(h + 1) * G], K[b, h][t], V[b, h][t])
            assert float((out[b, h * G:(h + 1) * G] - ref).abs().max()) <= TOL, (b, h)


@pytest.mark.parametrize("batch,hq,hkv,n", [(1, 32, 8, 23041), (3, 7, 1, 100003), (4, 8, 4, 12345), (1, 16, 8, 46081), (40, 8, 8, 1201)])
def test_full_kv(batch, hq, hkv, n):
    from paper_2602_03152_amd import binding as fb
    q, K, V, _, cap = _tensors(batch, hq, hkv, 1, n, 9)
    assert batch * hkv * n * 512 >= 90 << 20
    G = hq // hkv
    shape = fb.make_shape(batch, hq, hkv, D, 1, n, cap, n, "bf16")
    out = torch.full((batch, hq, D), float("nan"), device="cuda")
    ws = torch.empty(fb.fasa_workspace_bytes(shape), dtype=torch.uint8, device="cuda")
    fb.fasa_workspace_init(shape, ws, ws.numel())
    print("stream dense", batch, hq, hkv, n, flush=True)
    fb.fasa_dense_attend(shape, q, K, V, out, ws, ws.numel())
    torch.cuda.synchronize()
    for b in range(batch):
        for h in range(hkv):
            ref = _attention(q[b, h * G:(h + 1) * G], K[b, h, :n], V[b, h, :n])
            assert float((out[b, h * G:(h + 1) * G] - ref).abs().max()) <= TOL, (b, h)
