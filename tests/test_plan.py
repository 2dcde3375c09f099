"""The split plan of the bidirectional key pass, read from the workspace size (host
code only; no GPU is needed). Splits shorter than 256 rows serve calls that leave
most CUs idle; the reduction walks a head's splits in series, so a long sequence
of few heads keeps 256-row splits: with 64-row ones (bf16, one head of 16384
tokens at M = 64: 256 splits) the call took 35.9 us against 18.5.
"""
import pytest

import paper_2006_03555_amd as fv

S64 = 64 ** -0.25


def _round(n):
    return (n + 255) // 256 * 256


def _splits(dtype, H, L, M):
    """Splits per head of a bidirectional call of H heads."""
    code, fb = (fv.BF16, 16) if dtype == "bf16" else (fv.F32, 32)
    P = 64 if M <= 64 else 128 if M <= 128 else 256
    total = fv.workspace_size(fv.make_desc(1, H, L, 64, M, code, code, S64), 0)
    rest = _round(H * 5 * (P // 32) * 64 * fb) + _round(H * P // 16 * 128 * fb) + _round(H * P * 4)
    unit = H * P * 65 * 4
    n = (total - rest) // unit
    assert _round(n * unit) + rest == total
    return n


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("M", [64, 112, 256])
@pytest.mark.parametrize("H", [1, 2, 3, 4, 8, 16, 32])
def test_short_splits_are_few(dtype, M, H):
    for L in (1, 64, 65, 255, 512, 1000, 1024, 2048, 4096, 4097, 6144, 8192, 12288, 16384, 24576,
              32768, 65536):
        n = _splits(dtype, H, L, M)
        assert 1 <= n <= -(-L // 64)
        if n > max(1, L // 256):   # shorter than 256 rows
            assert n <= (16 if dtype == "bf16" else 128), (L, n)
            assert H * n <= 256, (L, n)


@pytest.mark.parametrize("dtype,L,n", [("bf16", 512, 8), ("bf16", 2048, 16), ("bf16", 16384, 64),
                                       ("f32", 1024, 16), ("f32", 4096, 64), ("f32", 16384, 128),
                                       ("f32", 32768, 128)])
def test_one_head_m64(dtype, L, n):
    assert _splits(dtype, 1, L, 64) == n
