"""The codec's group metadata where its fp32 form ends, bit for bit against the oracle (fp64).

Groups whose minimum lies on, just above and just below fp16 values (normal, subnormal, zero), whose range is an exact
multiple of the grid or a neighbour of one, that saturate at +-65504 on either side, whose range is not exact in fp32
(a huge and a tiny bound), and constant groups; every bit width, both axes, every group size, against a reference and
without one.
"""
import numpy as np
import pytest
import torch

from gpu_util import down, down_bits16, f16_bits, up, up_bf16
from oracle import codec
from oracle.numerics import f32_to_bf16

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    from paper_2609_29812_amd import flashloop
    flashloop.load()
    return flashloop


def _values(rng, shape):
    """fp32 values in runs of 8 channels, each run of its own kind and scale."""
    B, N, H, d = shape
    n = B * N * H * d // 8
    kind = rng.integers(0, 7, n)
    scale = np.exp2(rng.integers(-26, 18, n)).astype(np.float64)
    x = rng.standard_normal((n, 8)) * scale[:, None]
    grid = rng.integers(-40, 40, (n, 8)) * scale[:, None]                    # multiples of a power of two
    x = np.where((kind == 1)[:, None], grid, x)
    x = np.where((kind == 2)[:, None], x[:, :1], x)                          # constant
    x = np.where((kind == 3)[:, None], 0.0, x)
    x = np.where((kind == 4)[:, None], np.abs(x) + 60000.0, x)               # around the saturation
    x = np.where((kind == 5)[:, None], -np.abs(x) * 4 - 60000.0, x)
    x = np.where((kind == 6)[:, None], rng.standard_normal((n, 8)) * 2.0 ** -25, x)   # below fp16's subnormals
    return x.reshape(shape).astype(np.float32)


@pytest.mark.parametrize("bits", [2, 4, 8])
@pytest.mark.parametrize("axis", [codec.AXIS_TOKEN, codec.AXIS_CHANNEL])
@pytest.mark.parametrize("group", [8, 16, 32, 64, 128])
def test_metadata(F, bits, axis, group):
    rng = np.random.default_rng(bits * 1000 + axis * 100 + group)
    B, N, H, d = 1, 300, 2, 128
    cur = f32_to_bf16(_values(rng, (B, N, H, d)))
    ref = f32_to_bf16(_values(rng, (B, N, H, d)))
    idx = np.sort(rng.choice(N, 181, replace=False))[None].astype(np.int32)
    for x_ref, rows in ((None, None), (ref, idx)):
        with np.errstate(over="ignore"):
            enc = codec.quantize(cur, x_ref, rows, bits, group, axis)
            _, new = codec.reconstruct(x_ref, cur, rows, enc, bits, group, axis)
        codes, scale, zero, out = F.kv_residual_quant(up_bf16(cur), None if x_ref is None else up_bf16(x_ref),
                                                      None if rows is None else up(rows), bits, group, axis)
        torch.cuda.synchronize()
        assert np.array_equal(down(zero).view(np.uint16), f16_bits(enc["zero"]))
        assert np.array_equal(down(scale).view(np.uint16), f16_bits(enc["scale"]))
        assert np.array_equal(down(codes), enc["codes"])
        assert np.array_equal(down_bits16(out), new)


@pytest.mark.parametrize("axis", [codec.AXIS_TOKEN, codec.AXIS_CHANNEL])
@pytest.mark.parametrize("kind", ["-0", "-0 and 0", "-0 - 0"])
def test_negative_zeros(F, axis, kind):
    """Groups of zeros of either sign, whose range may be -0: zero and scale are +0."""
    B, N, H, d, bits, group = 1, 72, 2, 64, 4, 8
    cur = np.full((B, N, H, d), 0x8000, np.uint16)
    if kind == "-0 and 0":
        cur[:, ::3, :, 5::7] = 0
    ref = np.zeros_like(cur) if kind == "-0 - 0" else None
    enc = codec.quantize(cur, ref, None, bits, group, axis)
    _, new = codec.reconstruct(ref, cur, None, enc, bits, group, axis)
    codes, scale, zero, out = F.kv_residual_quant(up_bf16(cur), None if ref is None else up_bf16(ref), None, bits, group, axis)
    torch.cuda.synchronize()
    assert np.array_equal(down(zero).view(np.uint16), f16_bits(enc["zero"]))
    assert np.array_equal(down(scale).view(np.uint16), f16_bits(enc["scale"]))
    assert np.array_equal(down(codes), enc["codes"])
    assert np.array_equal(down_bits16(out), new)
