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


@pytest.mark.parametrize("kind", list(KINDS))
@pytest.mark.parametrize("M", [64, 80, 128, 208, 256])
@pytest.mark.parametrize("B,H,L", [(1, 1, 1), (1, 2, 16), (2, 1, 17), (1, 3, 100), (2, 3, 1100)])
def test_rows(kind, M, B, H, L):
    import torch
    fv = __import__("paper_2006_03555_amd")
    if L > 1000 and (M, kind) not in ((256, "softmax"), (64, "relu_eps"), (128, "softmax_eps")):
        pytest.skip("the long case is run on three of the combinations")
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
