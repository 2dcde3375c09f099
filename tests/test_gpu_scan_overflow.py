"""Intra-chunk weights past the range of float32 in the default bf16 causal scans.
Constant inputs whose features (ReLU, W = 1) are 2^55 in the first half of the rows
and 2^66 in the second: q-hat . k-hat is at most 2^118 among the first and past 2^128
among the second, while every feature, aggregate and value stays finite. A row of the numerator Q' K'^T V of
positive values is then +Inf where a product overflows and finite elsewhere, never
NaN; likewise dV for a positive output gradient."""
import pytest

pytestmark = pytest.mark.gpu


def _inputs(M, L):
    import torch
    q = torch.full((1, 2, L, 64), 2.0 ** 52, device="cuda", dtype=torch.bfloat16)
    q[:, :, L // 2:] = 2.0 ** 63
    v = 1.0 + torch.rand((1, 2, L, 64), device="cuda", generator=torch.Generator(
        device="cuda").manual_seed(3)).to(torch.bfloat16)
    W = torch.ones((2, M, 64), device="cuda")
    b = torch.zeros((2, M), device="cuda")
    # a feature is 64 x scale / sqrt(M) = 8 x
    return q, v, W, b, M ** 0.5 / 8.0


@pytest.mark.parametrize("M", [64, 128, 256])
@pytest.mark.parametrize("L", [256, 400])
def test_numerator_overflows_to_inf(M, L):
    import torch
    fv = __import__("paper_2006_03555_amd")
    q, v, W, b, s = _inputs(M, L)
    kw = dict(kernel=fv.KERNEL_RELU, kernel_eps=0.0, renormalize=False, segment=64,
              out_dtype=torch.float32)
    out = fv.attn_causal(q, q, v, W, b, s, **kw)
    named = fv.attn_causal(q, q, v, W, b, s, chunk=64, **kw)
    big = q[0, 0, :, 0] == 2.0 ** 63
    assert not torch.isnan(out).any()
    assert torch.isposinf(out[:, :, big]).all()
    assert torch.isfinite(out[:, :, ~big]).all()
    assert torch.equal(torch.isinf(named), torch.isinf(out))


@pytest.mark.parametrize("M", [64, 128, 256])
def test_dv_overflows_to_inf(M):
    import torch
    fv = __import__("paper_2006_03555_amd")
    q, v, W, b, s = _inputs(M, 256)
    do = torch.ones_like(v)
    _, _, dV = fv.attn_causal_backward(q, q, v, W, b, s, do, kernel=fv.KERNEL_RELU,
                                       kernel_eps=0.0, renormalize=False)
    assert not torch.isnan(dV).any()
    assert torch.isposinf(dV[:, :, 128:]).all()
