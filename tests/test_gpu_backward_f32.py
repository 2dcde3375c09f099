"""The fp32 bidirectional gradients (features split over the waves) at the sizes
where they can go wrong: one row, 16-row block edges, more blocks than
workgroups with several heads in a workgroup's range, every padded feature
count, both feature kinds, with and without renormalisation and stabiliser.
Gate as in test_gpu_backward."""
import numpy as np
import pytest

import workloads as wl
from helpers import to_dev
from oracle import favor
from test_gpu_backward import _check_all, _host_grads, _oracle_grads, _oracle_w
from test_gpu_backward_scan import KINDS

pytestmark = pytest.mark.gpu

S64 = 64 ** -0.25


# the long case is run on three of the combinations
LONG = ((256, "softmax"), (64, "relu_eps"), (128, "softmax_eps"))


@pytest.mark.parametrize("kind,M,B,H,L", [
    (kind, M, B, H, L) for B, H, L in ((1, 1, 1), (1, 2, 16), (2, 1, 17), (1, 3, 100), (2, 3, 1100))
    for M in (64, 80, 128, 208, 256) for kind in KINDS if L < 1000 or (M, kind) in LONG])
def test_rows(kind, M, B, H, L):
    import torch
    fv = __import__("paper_2006_03555_amd")
    kw = KINDS[kind]
    Q, K, V = wl.make_qkv(wl.Workload("t", "bidir", B, H, L, 64, M, "f32", M + L))
    dout = np.random.default_rng(M + L).standard_normal((B, H, L, 64)).astype(np.float32)
    W, b = favor.orf_draw(22, H, M, 64)
    W, b = W.astype(np.float32), b.astype(np.float32)
    q, k, v, do = (to_dev(x) for x in (Q, K, V, dout))
    Wd, bd = to_dev(W), to_dev(b)
    g3 = [torch.full_like(q, float("nan")) for _ in range(3)]
    got = fv.attn_bidir_backward(q, k, v, Wd, bd, S64, do, dQ=g3[0], dK=g3[1], dV=g3[2], **kw)
    torch.cuda.synchronize()
    ref, scale, _ = _oracle_grads(Q, K, V, _oracle_w(W, M, "f32", kw["kernel"]), b, dout, False,
                                  **kw)
    _check_all(_host_grads(got), ref, "f32", scale)


# Gradients by 128-row tiles (dQ; at M = 64 dK and dV too): 256 tiles, the last of each
# head one row short or the tiles a tenth empty
@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("M,L", [(64, 2047), (80, 2047), (128, 2047), (128, 1850)])
def test_full_tiles(kind, M, L):
    import torch
    fv = __import__("paper_2006_03555_amd")
    kw = KINDS[kind]
    relu = kw["kernel"] == favor.KERNEL_RELU
    B, H = 2, 8
    gen = torch.Generator()
    gen.manual_seed(M + L)
    q, k, v, do = ((torch.randn((B, H, L, 64), generator=gen) * s).cuda()
                   for s in (S64, S64, 1.0, 1.0))
    W, b = fv.orf_draw(7, H, M)
    g3 = [torch.full_like(q, float("nan")) for _ in range(3)]
    got = fv.attn_bidir_backward(q, k, v, W, b, S64, do, dQ=g3[0], dK=g3[1], dV=g3[2], **kw)

    def phi(x):
        p = x * S64 @ W.double().transpose(-1, -2).contiguous()
        if relu:
            return p.clamp(min=0) / M ** 0.5 + 1e-3
        d = torch.exp(0.5 * (x * S64).square().sum(-1, keepdim=True))
        return d * (2.0 / M) ** 0.5 * torch.cos(p + b.double()[:, None, :])

    xs = [x.double().requires_grad_() for x in (q, k, v)]
    ones = torch.cat([xs[2], torch.ones_like(xs[2][..., :1])], -1)
    buf = phi(xs[0]) @ (phi(xs[1]).transpose(-1, -2).contiguous() @ ones)
    out = buf[..., :64]
    if kw.get("renormalize", True):
        out = out / (buf[..., 64:] + kw.get("denom_eps", 0.0))
    for x, ref in zip(got, torch.autograd.grad(out, xs, do.double())):
        # at most 1.2e-6 at the other sizes
        assert float((x - ref).norm() / ref.norm()) <= 5e-6
        # and no row is far off: a row's error against the larger of its own size and the
        # mean row's. Denominators that cancel amplify their rounding, so the worst rows
        # of cos features are looked at only for a wrong row (order 1)
        size = ref.norm(dim=-1).clamp(min=float(ref.norm(dim=-1).mean()))
        assert float(((x - ref).norm(dim=-1) / size).max()) <= (1e-4 if relu else 1e-2)
