"""Calls of few rows: the bidirectional query pass with its features split over
the waves, the key pass with one workgroup per 64 features and short row splits,
and the fp32 cosine."""
import math

import numpy as np
import pytest

import workloads as wl
from oracle import favor
from tests import helpers

pytestmark = pytest.mark.gpu

KERNELS = {"softmax": favor.KERNEL_SOFTMAX, "relu": favor.KERNEL_RELU}


# B * H * ceil(L / 16) is 1 .. 1024 row blocks (split form), then one more block
# per head (the persistent form); L below, at and past whole 16-row blocks and
# 64-row key tiles
@pytest.mark.parametrize("B,H,L", [(1, 1, 1), (1, 2, 15), (2, 1, 64), (1, 3, 65), (1, 1, 333),
                                   (1, 4, 4096), (1, 4, 4097), (3, 2, 1000)])
@pytest.mark.parametrize("dtype,M", [("f32", 128), ("f32", 208), ("bf16", 256), ("bf16", 112),
                                     ("f32", 64)])
@pytest.mark.parametrize("variant", ["softmax", "relu", "softmax_eps", "relu_numerator"])
def test_few_rows(B, H, L, dtype, M, variant):
    import paper_2006_03555_amd as fv
    kernel = variant.split("_")[0]
    renorm = "numerator" not in variant
    eps = 0.5 if "eps" in variant else 0.0
    w = wl.WORKLOADS["bidir_small"].with_(B=B, H=H, L=L, M=M, dtype=dtype, seed=L + M)
    Q, K, V = wl.make_qkv(w)
    W, b = favor.orf_draw(11, H, M, w.d)
    s = w.input_scale
    dev = [helpers.to_dev(x, dtype) for x in (Q, K, V)]
    Wd, bd = helpers.to_dev(W), helpers.to_dev(b)
    opts = dict(kernel=KERNELS[kernel], renormalize=renorm)
    out = fv.attn_bidir(*dev, Wd, bd, s, eps, **opts)
    W32, b32 = W.astype(np.float32), b.astype(np.float32)
    helpers.parity(helpers.to_host(out), Q, K, V, W32, b32, s, False, dtype, eps=eps,
                   kernel=KERNELS[kernel], renormalize=renorm,
                   gate="both" if renorm else "cond")
    if renorm:   # the saving form gives the same rows, and the rows' scales
        import torch
        rs = torch.full((B, H, L), float("nan"), dtype=torch.float32, device="cuda")
        again = fv.attn_bidir(*dev, Wd, bd, s, eps, row_scale=rs, **opts)
        assert torch.equal(again, out)
        assert bool(torch.isfinite(rs).all())


def test_fp32_cosine():
    """X' of rows with one non-zero entry, where the projection is one product:
    W'' = fl(W ws) with ws two roundings, the product and the sum with b'' = fl(b /
    2 pi) (constant and product rounded) put at most 6 half-ulps of |p| + |b''| into
    the phase; the cosine itself is within 1.4e-7, and D_X sqrt(2/M) and its
    product add a few roundings and expf's error (8 half-ulps)."""
    import torch

    import paper_2006_03555_amd as fv
    rng = np.random.default_rng(5)
    L, M = 512, 128
    s = 64.0 ** -0.25
    X = np.zeros((1, 1, L, 64), np.float32)
    X[0, 0, np.arange(L), np.arange(L) % 64] = rng.uniform(-1.5, 1.5, L)
    W = (rng.standard_normal((1, M, 64)) * 8).astype(np.float32)
    b = rng.uniform(0, 2 * np.pi, (1, M)).astype(np.float32)
    got = fv.feature_map(torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda(),
                         torch.from_numpy(b).cuda(), s).cpu().numpy()[0, 0].astype(np.float64)
    x64 = X[0, 0].astype(np.float64) * float(np.float32(s))
    th = x64 @ W[0].astype(np.float64).T
    D = np.exp(0.5 * (x64 ** 2).sum(1, keepdims=True)) * math.sqrt(2 / M)
    ref = D * np.cos(th + b[0].astype(np.float64))
    u = 2.0 ** -24
    bound = D * (6 * u * (np.abs(th) + b[0]) + 1.4e-7 + 8 * u)
    assert (np.abs(got - ref) <= bound).all(), float((np.abs(got - ref) / bound).max())
