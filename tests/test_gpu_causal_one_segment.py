"""Causal calls whose heads are one segment each (bf16): one launch that builds
W'' itself and carries the state. Against the oracle, with the state in place,
and with a backward call reading the workspace it leaves."""
import numpy as np
import pytest

import workloads as wl
from helpers import TOL, parity, to_dev, to_host
from oracle import favor

pytestmark = pytest.mark.gpu

S64 = 64 ** -0.25


# one chunk and less, whole and ragged chunks; one segment by length, by
# descriptor (segment >= L) or by head count (more heads than CUs; two of the
# combinations)
SIZES = ((1, 2, 1, 0), (2, 2, 63, 0), (1, 3, 128, 0), (1, 2, 191, 0), (1, 2, 700, 704),
         (33, 8, 300, 0))
FEATURES = ((64, 0), (112, 64), (128, 0), (208, 64), (256, 0), (256, 32))


@pytest.mark.parametrize("state,kernel,M,chunk,B,H,L,segment", [
    (state, kernel, *mc, *size) for state in (False, True) for kernel in ("softmax", "relu")
    for mc in FEATURES for size in SIZES
    if size[0] < 30 or (mc[0], state) in ((256, True), (112, False))])
def test_one_segment(B, H, L, segment, M, chunk, kernel, state):
    import torch
    fv = __import__("paper_2006_03555_amd")
    kn = favor.KERNEL_RELU if kernel == "relu" else favor.KERNEL_SOFTMAX
    Q, K, V = wl.make_qkv(wl.Workload("t", "causal", B, H, L, 64, M, "bf16", M + L))
    W, b = favor.orf_draw(23, H, M, 64)
    W, b = W.astype(np.float32), b.astype(np.float32)
    S0 = None
    if state:
        Qe, Ke, Ve = wl.make_qkv(wl.Workload("t", "causal", B, H, 256, 64, M, "bf16", 9))
        _, S0 = favor.attn_causal(Qe, Ke, Ve, W, b, S64, kernel=kn)
        S0 = S0.astype(np.float32)
    q, k, v = (to_dev(x, "bf16") for x in (Q, K, V))
    Wd, bd = to_dev(W), to_dev(b)
    s = to_dev(S0) if state else None
    kw = dict(kernel=kn, segment=segment, chunk=chunk)
    out, s1 = fv.attn_causal(q, k, v, Wd, bd, S64, state_in=s, return_state=True, **kw)
    heads = [(0, 0), (B - 1, H - 1)]
    stats = {}
    # cos features at M = 64: the first rows' denominators may cancel
    parity(to_host(out), Q, K, V, W, b, S64, True, "bf16", state_in=S0, heads=heads, kernel=kn,
           gate="cond" if M == 64 and kernel == "softmax" else "both", stats=stats)
    Kp = favor.features(K[-1:, -1:], W[-1:], b[-1:], S64, kn)
    C = np.concatenate([V[-1:, -1:], np.ones_like(V[-1:, -1:, :, :1])], -1).astype(np.float64)
    ref = np.swapaxes(Kp, -1, -2) @ C + (S0[-1, -1].astype(np.float64) if state else 0.0)
    got = to_host(s1)[-1:, -1:]
    assert np.max(np.abs(got - ref)) <= TOL["bf16"] * np.max(np.abs(ref))
    if state:   # the state updated in place
        out2, s2 = fv.attn_causal(q, k, v, Wd, bd, S64, state_in=s, state_out=s,
                                  return_state=True, **kw)
        assert torch.equal(out2, out) and torch.equal(s2, s1)


@pytest.mark.parametrize("M", [64, 112, 256])
def test_backward_reads_its_workspace(M):
    import torch
    fv = __import__("paper_2006_03555_amd")
    B, H, L = 2, 2, 150
    Q, K, V = wl.make_qkv(wl.Workload("t", "causal", B, H, L, 64, M, "bf16", 4))
    W, b = favor.orf_draw(24, H, M, 64)
    q, k, v = (to_dev(x, "bf16") for x in (Q, K, V))
    Wd, bd = to_dev(W), to_dev(b)
    do = to_dev(np.random.default_rng(1).standard_normal((B, H, L, 64)), "bf16")
    _, s0 = fv.attn_causal(k, q, v, Wd, bd, S64, return_state=True)
    g = fv.make_desc(B, H, L, 64, M, fv.BF16, fv.BF16, S64)
    ws = torch.full((fv.workspace_size(g, 1),), 255, dtype=torch.uint8, device="cuda")
    rs = torch.empty((B, H, L), device="cuda")
    out = fv.attn_causal(q, k, v, Wd, bd, S64, state_in=s0, workspace=ws, row_scale=rs)
    a = fv.attn_causal_backward(q, k, v, Wd, bd, S64, do, state_in=s0, return_state_grad=True,
                                out=out, row_scale=rs, forward_workspace=ws,
                                forward_call="causal")
    c = fv.attn_causal_backward(q, k, v, Wd, bd, S64, do, state_in=s0, return_state_grad=True,
                                out=out, row_scale=rs)
    assert all(torch.equal(x, y) for x, y in zip(a, c))


# the default chunk length, one segment by length and by head count
@pytest.mark.parametrize("B,H,L", [(2, 2, 150), (1, 2, 127), (65, 8, 200)])
@pytest.mark.parametrize("M", [64, 112, 256])
@pytest.mark.parametrize("kernel", ["softmax", "relu"])
def test_every_call_runs_the_same_scan(B, H, L, M, kernel):
    """The causal half of attn_both is bitwise what attn_causal returns, and a backward
    call that recomputes the output and the row scales returns the bits it returns when
    given those of the forward call."""
    import torch
    fv = __import__("paper_2006_03555_amd")
    kw = dict(kernel=favor.KERNEL_RELU if kernel == "relu" else favor.KERNEL_SOFTMAX)
    Q, K, V = wl.make_qkv(wl.Workload("t", "causal", B, H, L, 64, M, "bf16", 6))
    W, b = favor.orf_draw(25, H, M, 64)
    q, k, v = (to_dev(x, "bf16") for x in (Q, K, V))
    args = (q, k, v, to_dev(W), to_dev(b), S64)
    do, db = (to_dev(np.random.default_rng(i).standard_normal(Q.shape), "bf16") for i in (1, 2))
    rs, rb, rc = (torch.empty((B, H, L), device="cuda") for _ in range(3))
    _, s0 = fv.attn_causal(k, q, v, *args[3:], return_state=True, **kw)
    out = fv.attn_causal(*args, state_in=s0, row_scale=rs, **kw)
    ob, oc = fv.attn_both(*args, state_in=s0, row_scale_bidir=rb, row_scale_causal=rc, **kw)
    assert torch.equal(out, oc) and torch.equal(rs, rc)
    kw.update(state_in=s0, return_state_grad=True)
    saved = fv.attn_causal_backward(*args, do, out=out, row_scale=rs, **kw)
    fresh = fv.attn_causal_backward(*args, do, **kw)
    assert all(torch.equal(x, y) for x, y in zip(saved, fresh))
    saved = fv.attn_both_backward(*args, db, do, out_bidir=ob, row_scale_bidir=rb, out_causal=oc,
                                  row_scale_causal=rc, **kw)
    fresh = fv.attn_both_backward(*args, db, do, **kw)
    assert all(torch.equal(x, y) for x, y in zip(saved, fresh))
