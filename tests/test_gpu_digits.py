"""GPU parity of the fp64 column statistic on integer digits (fl_digits.h) where its tiles and ranges end.

Keys within one fp32 ulp of the oracle's fp64 statistic rounded to fp32: the digits hold the dot products to better
than 2^-24 of an exponent, or the (batch, head) takes the fp64 products.  Lengths: around the 16-vector blocks, the
64-vector stages and both workgroup sizes.  Values: standard normal; elements far below the largest of their block
(digit 0) on either and on both sides; zero vectors; magnitudes whose exponents leave the digits' range, an infinity
and an outlier beside tiny elements (fp64 products); and a workspace that holds no digits.
"""
import ctypes

import numpy as np
import pytest
import torch

from gpu_util import assert_keys_close, down, say, up_bf16
from oracle import attention as att
from oracle.numerics import bf16_to_f64, f32_to_bf16

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    from paper_2609_29812_amd import flashloop
    flashloop.load()
    return flashloop


def _inputs(kind, B, N, H, d):
    rng = np.random.default_rng(N * 1000 + d + len(kind))
    q, k = (rng.standard_normal((B, N, H, d)).astype(np.float32) for _ in range(2))
    tiny = np.where(rng.random((B, N, H, d)) < 0.02, np.float32(2.0 ** -17), np.float32(0))
    if kind in ("tiny-q", "tiny-both"):
        q = np.where(tiny > 0, q * tiny, q)
    if kind in ("tiny-k", "tiny-both"):
        k = np.where(tiny > 0, k * tiny, k)
    if kind == "zeros":
        q[:, ::3], k[:, 1::2] = 0, 0
    if kind == "large":                       # exponents in the hundreds
        q, k = q * 12, k * 12
    if kind == "outlier":                     # elements that the digits of their block do not hold
        k[:, :, 0, 3] *= 5000
        q[:, :, 0, 3] *= 2.0 ** -20
    if kind == "wide":
        q = q * np.exp2(rng.integers(-30, 2, q.shape)).astype(np.float32)
        k = k * np.exp2(rng.integers(-30, 2, q.shape)).astype(np.float32)
    return f32_to_bf16(q), f32_to_bf16(k)


def _check(F, kind, B, N, H, d, got, q, k, heads):
    for b in range(B):
        for h in heads:
            q64, k64 = bf16_to_f64(q[b, :, h]), bf16_to_f64(k[b, :, h])
            _, _, cs = att.dense_loop(q64, k64, k64, 1 / np.sqrt(d))
            assert_keys_close(got[b, h], cs.astype(np.float32), f"{kind} b={b} h={h}")


@pytest.mark.parametrize("B,N,H,d", [(1, 1, 1, 64), (1, 15, 2, 128), (2, 16, 3, 64), (1, 17, 8, 128), (1, 63, 2, 64),
                                     (1, 64, 1, 128), (1, 65, 2, 128), (3, 129, 8, 64), (1, 257, 3, 128),
                                     (1, 513, 16, 64)])
def test_lengths(F, B, N, H, d):
    q, k = _inputs("normal", B, N, H, d)
    got = down(F.column_scores(up_bf16(q), up_bf16(k)))
    _check(F, "normal", B, N, H, d, got, q, k, range(H))


@pytest.mark.parametrize("d", [64, 128])
def test_two_blocks_per_wave(F, d):
    """128-vector workgroups (at least 512 of them), the last one partial."""
    B, N, H = 2, 2047, 16
    q, k = _inputs("normal", B, N, H, d)
    got = down(F.column_scores(up_bf16(q), up_bf16(k)))
    _check(F, "normal", B, N, H, d, got, q, k, (0, 9))


@pytest.mark.parametrize("kind", ["tiny-q", "tiny-k", "tiny-both", "zeros", "large", "outlier", "wide"])
@pytest.mark.parametrize("d", [64, 128])
def test_values(F, kind, d):
    B, N, H = 1, 300, 2
    q, k = _inputs(kind, B, N, H, d)
    got = down(F.column_scores(up_bf16(q), up_bf16(k)))
    _check(F, kind, B, N, H, d, got, q, k, range(H))


def test_not_finite_takes_fp64(F):
    """A head with an infinite key gives what the fp64 products give (NaN in the rows that see it), the other heads
    their own keys."""
    B, N, H, d = 1, 200, 2, 64
    q, k = _inputs("normal", B, N, H, d)
    k[0, 50, 1, 0] = 0x7F80
    got = down(F.column_scores(up_bf16(q), up_bf16(k)))
    _check(F, "finite head", B, N, H, d, got, q, k, (0,))
    assert np.isnan(got[0, 1, :]).any()
    assert np.array_equal(got[0, 1], _small_workspace(F, q, k)[0, 1], equal_nan=True)


def _small_workspace(F, q, k):
    """fl_column_scores with room for the rows' log-normalisers only (fp64 products for every head)."""
    B, N, H, d = q.shape
    dq, dk = up_bf16(q), up_bf16(k)
    ws = torch.empty(B * H * N * 8, dtype=torch.uint8, device="cuda")
    assert F.load().fl_column_scores_ws(B, N, H) > ws.numel()
    key = torch.empty(B, H, N, device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    rc = F.load().fl_column_scores(p(dq), p(dk), B, N, H, d, p(key), p(ws), ws.numel(),
                                   ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    torch.cuda.synchronize()
    return down(key)


def test_small_workspace(F):
    q, k = _inputs("normal", 2, 140, 3, 128)
    want = _small_workspace(F, q, k)
    _check(F, "fp64 products", 2, 140, 3, 128, want, q, k, range(3))
    got = down(F.column_scores(up_bf16(q), up_bf16(k)))
    say("digits against fp64 products")
    for b in range(2):
        for h in range(3):
            assert_keys_close(got[b, h], want[b, h], f"b={b} h={h}")
