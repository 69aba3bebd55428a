"""GPU parity of the dense source loop where its row tiles, column stages and both workgroup forms end.

Against the oracle's dense loop, with the attention tolerance of the parity tests (P is rounded to fp16): max-abs 1e-2
and relative Frobenius 2e-3 on the output and the log-normaliser.  64 rows per workgroup with split columns for few
workgroups, 128 rows for many (512 at d = 128, 1024 at d = 64).
"""
import numpy as np
import pytest
import torch

from gpu_util import assert_close, down, up_bf16
from oracle import attention as att
from oracle.numerics import bf16_to_f64, f32_to_bf16

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    from paper_2609_29812_amd import flashloop
    flashloop.load()
    return flashloop


def _check(F, B, N, H, d, heads, scale=1.0):
    rng = np.random.default_rng(N * 7 + d)
    q, k, v = (f32_to_bf16((rng.standard_normal((B, N, H, d)) * s).astype(np.float32)) for s in (scale, 1.0, 1.0))
    o, lse = (down(t) for t in F.dense_attn(up_bf16(q), up_bf16(k), up_bf16(v)))
    for b, h in heads:
        wo, wl, _ = att.dense_loop(bf16_to_f64(q[b, :, h]), bf16_to_f64(k[b, :, h]), bf16_to_f64(v[b, :, h]),
                                   1 / np.sqrt(d), want_colscore=False)
        assert_close(o[b, :, h], wo, f"o N={N} d={d} b={b} h={h}")
        assert_close(lse[b, :, h], wl, f"lse N={N} d={d} b={b} h={h}")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("N", [1, 31, 32, 33, 63, 64, 65, 95, 97, 127, 128, 129, 191, 193, 321])
def test_split_columns(F, N, d):
    _check(F, 1, N, 3, d, [(0, 0), (0, 2)])


@pytest.mark.parametrize("N", [33, 127, 129, 257])
@pytest.mark.parametrize("d,B,H", [(128, 8, 64), (64, 16, 64)])
def test_whole_rows(F, N, d, B, H):
    _check(F, B, N, H, d, [(0, 0), (B - 1, 5)])


def test_sharp_rows(F):
    """Logits that move the softmax reference many times."""
    _check(F, 1, 700, 2, 128, [(0, 0), (0, 1)], scale=8.0)


@pytest.mark.parametrize("d,B,H", [(128, 1, 3), (64, 1, 3), (128, 8, 64), (64, 16, 64)])   # split columns, whole rows
@pytest.mark.parametrize("j", [40, 70, 100, 127, 140])
def test_value_out_of_range(F, d, B, H, j):
    """A value that is not finite in fp16 reaches the 32-row group of its own position and the rows after, no earlier
    ones: those keep the bits of finite values."""
    N = 150
    g = torch.Generator(device="cuda").manual_seed(j)
    q, k, v = (torch.randn(B, N, H, d, device="cuda", generator=g).to(torch.bfloat16) for _ in range(3))
    want, want_lse = F.dense_attn(q, k, v)
    v[:, j] = torch.tensor([float("inf"), float("nan"), 1e6, -1e6], device="cuda").to(torch.bfloat16).repeat(d // 4)
    got, lse = F.dense_attn(q, k, v)
    lo = j // 32 * 32
    assert torch.equal(got[:, :lo], want[:, :lo])
    assert torch.equal(lse, want_lse)
