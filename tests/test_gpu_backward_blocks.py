"""The bidirectional bf16 gradient kernels (two 16-row blocks per wave in one pass
over the features) at the edges of a block, a wave's pair and a tile of 256 rows,
every padded feature count, with and without renormalisation and stabiliser. Gate
as in test_gpu_backward."""
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
@pytest.mark.parametrize("L", [1, 16, 17, 33, 255, 257])
def test_block_edges(kind, M, L):
    import torch
    fv = __import__("paper_2006_03555_amd")
    B, H = 1, 2
    kw = KINDS[kind]
    rng = np.random.default_rng(100 * M + L)
    Q, K, V = wl.make_qkv(wl.Workload("t", "bidir", B, H, L, 64, M, "bf16", M + L))
    dout = torch.from_numpy(rng.standard_normal((B, H, L, 64)).astype(np.float32))
    dout = dout.to(torch.bfloat16).float().numpy()
    W, b = favor.orf_draw(22, H, M, 64)
    W, b = W.astype(np.float32), b.astype(np.float32)
    q, k, v, do = (to_dev(x, "bf16") for x in (Q, K, V, dout))
    # gradients that start as NaN: every row has to be written
    g3 = [torch.full_like(q, float("nan")) for _ in range(3)]
    got = fv.attn_bidir_backward(q, k, v, to_dev(W), to_dev(b), S64, do, dQ=g3[0], dK=g3[1],
                                 dV=g3[2], **kw)
    ref, scale, _ = _oracle_grads(Q, K, V, _oracle_w(W, M, "bf16", kw["kernel"]), b, dout, False,
                                  **kw)
    _check_all(_host_grads(got), ref, "bf16", scale)
