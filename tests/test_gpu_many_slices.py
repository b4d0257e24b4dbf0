"""Quotients by multiplication (fast_div) are exact up to a bound that a launch's largest quotient is tested against on the host; beyond it the
kernels divide.  Rows of eight million tokens, 8191 and 8192 workgroups each, lie on both sides of it: every score against float32 torch."""
import pytest
import torch

pytestmark = pytest.mark.gpu

D, F = 128, 2


@pytest.mark.parametrize("n_ctx,beyond", [(8191 * 1024, False), (8191 * 1024 + 1, True)])
def test_scores_of_very_long_rows(n_ctx, beyond):
    from paper_2602_03152_amd import binding as fb
    batch, kv, group = 4, 8, 2
    slices = (n_ctx + 1023) // 1024
    assert (batch * kv * slices * slices >= 1 << 31) == beyond          # div_magic's bound
    cap = (n_ctx + 63) // 64 * 64
    gen = torch.Generator(device="cuda").manual_seed(5)
    q = torch.randn(batch, kv * group, D, generator=gen, device="cuda").bfloat16()
    fc = torch.tensor([[h, 63 - h] for h in range(kv)], dtype=torch.int32, device="cuda")
    Kp = torch.empty(batch, kv, F, cap, 2, dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    S = torch.full((batch, kv, cap), float("nan"), device="cuda")
    shape = fb.make_shape(batch, kv * group, kv, D, F, n_ctx, cap, 64, "bf16", kv_stride_b=0, kv_stride_h=0, kv_stride_n=D)
    print("many slices", n_ctx, slices, flush=True)
    fb.fasa_score(shape, q, Kp, fc, S)
    torch.cuda.synchronize()
    qs = q.float().reshape(batch, kv, group, D).sum(2)
    for b in range(batch):
        for h in range(kv):
            want, scale = torch.zeros(n_ctx, device="cuda"), torch.zeros(n_ctx, device="cuda")
            for f in range(F):
                i = int(fc[h, f])
                for part, dim in ((0, i), (1, i + D // 2)):
                    term = Kp[b, h, f, :n_ctx, part].float() * qs[b, h, dim]
                    want += term
                    scale += term.abs()
            # four products and sums in float32, in another order
            assert ((S[b, h, :n_ctx] - want).abs() <= 1e-6 * scale + 1e-30).all(), (b, h)
