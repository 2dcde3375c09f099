"""The bf16 causal gradient scans (features split over the waves) at the sizes
where they can go wrong: one row, chunk and segment edges, every padded feature
count, both feature kinds, the paths with and without renormalisation and
stabiliser (g~ . q-hat is zero up to the stabiliser where renormalised), a carried
state with a state gradient, saved and recomputed statistics. Gate as in
test_gpu_backward."""
import numpy as np
import pytest

import workloads as wl
from helpers import TOL, to_dev, to_host
from oracle import favor
from test_gpu_backward import _check_all, _host_grads, _oracle_grads, _oracle_w

pytestmark = pytest.mark.gpu

S64 = 64 ** -0.25
KINDS = {"softmax": dict(kernel=favor.KERNEL_SOFTMAX, renormalize=True, denom_eps=0.0),
         "softmax_eps": dict(kernel=favor.KERNEL_SOFTMAX, renormalize=True, denom_eps=0.3),
         "softmax_numerator": dict(kernel=favor.KERNEL_SOFTMAX, renormalize=False, denom_eps=0.0),
         "relu_eps": dict(kernel=favor.KERNEL_RELU, renormalize=True, denom_eps=1e-3),
         "relu_numerator": dict(kernel=favor.KERNEL_RELU, renormalize=False, denom_eps=0.0)}


@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("M", [64, 80, 128, 144, 256])
@pytest.mark.parametrize("L", [1, 63, 64, 65, 193, 320])
def test_scan_edges(kind, M, L):
    import torch
    fv = __import__("paper_2006_03555_amd")
    B, H = 1, 2
    kw = KINDS[kind]
    rng = np.random.default_rng(100 * M + L)
    Q, K, V = wl.make_qkv(wl.Workload("t", "causal", B, H, L, 64, M, "bf16", M + L))
    dout = torch.from_numpy(rng.standard_normal((B, H, L, 64)).astype(np.float32))
    dout = dout.to(torch.bfloat16).float().numpy()
    W, b = favor.orf_draw(21, H, M, 64)
    W, b = W.astype(np.float32), b.astype(np.float32)
    Qe, Ke, Ve = wl.make_qkv(wl.Workload("t", "causal", B, H, 256, 64, M, "bf16", 9))
    _, S0 = favor.attn_causal(Qe, Ke, Ve, W, b, S64, kernel=kw["kernel"])
    S0 = S0.astype(np.float32)
    dS = rng.standard_normal(S0.shape).astype(np.float32) * 0.01
    q, k, v, do = (to_dev(x, "bf16") for x in (Q, K, V, dout))
    Wd, bd, s0, ds = to_dev(W), to_dev(b), to_dev(S0), to_dev(dS)
    saved = {}
    if kw["renormalize"] and L % 2:
        r = torch.empty((B, H, L), device="cuda")
        o = fv.attn_causal(q, k, v, Wd, bd, S64, state_in=s0, row_scale=r, **kw)
        saved = dict(out=o, row_scale=r)
    # gradients that start as NaN: every row has to be written
    g3 = [torch.full_like(q, float("nan")) for _ in range(3)]
    got = fv.attn_causal_backward(q, k, v, Wd, bd, S64, do, state_in=s0, dstate_out=ds,
                                  return_state_grad=True, dQ=g3[0], dK=g3[1], dV=g3[2], **kw,
                                  **saved)
    torch.cuda.synchronize()
    ref, scale, rS = _oracle_grads(Q, K, V, _oracle_w(W, M, "bf16", kw["kernel"]), b, dout, True,
                                   state_in=S0, dstate_out=dS, **kw)
    assert np.max(np.abs(to_host(got[3]) - rS)) <= TOL["bf16"] * np.max(np.abs(rS))
    _check_all(_host_grads(got), ref, "bf16", scale)
