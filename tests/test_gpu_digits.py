"""GPU parity of the fp64 column and list statistics on integer digits (fl_digits.h) where its tiles and ranges end.

Keys within one fp32 ulp of the oracle's fp64 statistic rounded to fp32: the digits hold an exponent to 2^-25, so a sum
of exponentials to 2^-24 of itself before it is rounded (in the worst case; typically some 2^-30), or the (batch, head)
takes the fp64 products.  Which of the two served is read off the workspace.  Lengths: around the 16-vector blocks, the
64-vector stages and both workgroup sizes, and several groups of pairs.  Values: normal of several deviations; channels
far from the others; elements far below the largest of their block (digit 0) on either and on both sides; zero vectors;
exponents close to the digits' bound and beyond it; an infinity and an outlier beside tiny elements (fp64 products); and
a workspace that holds no digits.
"""
import ctypes

import numpy as np
import pytest
import torch

from gpu_util import assert_keys_close, column_layout, down, say, up_bf16
from oracle import attention as att
from oracle import prune
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
    if kind[0] == "s" and kind[1:].isdigit():
        q, k = q * int(kind[1:]), k * int(kind[1:])
    if kind == "channel":
        k[..., 3] += 32
    if kind == "channels":
        k[..., 3] += 16
        q[..., 5] += 8
    if kind == "sharp":                       # exponents of 280 for rows and columns that are alike, of either sign
        k = q * rng.choice(np.float32([-1, 1]), (B, N, H, 1))
        q, k = (x * (np.sqrt(280.0 * np.sqrt(d)) / np.linalg.norm(x, axis=-1, keepdims=True)) for x in (q, k))
    if kind == "large":                       # exponents beyond the digits' bound
        q, k = q * 12, k * 12
    if kind == "outlier":                     # elements that the digits of their block do not hold
        k[:, :, 0, 3] *= 5000
        q[:, :, 0, 3] *= 2.0 ** -20
    if kind == "wide":
        q = q * np.exp2(rng.integers(-30, 2, q.shape)).astype(np.float32)
        k = k * np.exp2(rng.integers(-30, 2, q.shape)).astype(np.float32)
    return f32_to_bf16(q), f32_to_bf16(k)


def _scores(F, q, k, ws_bytes=None):
    """fl_column_scores with the workspace that the query asks for (or ws_bytes): the keys, and per (batch, head) of the
    last group of pairs whether the digits served it: they leave base-2 row normalisers at the workspace's start, the
    fp64 products natural ones."""
    B, N, H, d = q.shape
    n, need = column_layout(B, N, H, d)
    size = F.load().fl_column_scores_ws(B, N, H) if ws_bytes is None else ws_bytes
    ws = torch.zeros(size, dtype=torch.uint8, device="cuda")
    key = torch.empty(B, H, N, device="cuda")
    p = lambda t: ctypes.c_void_p(t.data_ptr())  # noqa: E731
    rc = F.load().fl_column_scores(p(q), p(k), B, N, H, d, p(key), p(ws), size,
                                   ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    assert rc == 0
    pairs = B * H
    first, stride = (pairs - 1) // n * n, -(-N // 16) * 16
    if size < need or (q.data_ptr() | k.data_ptr()) % 16:
        first, stride = 0, N
    lse = ws[:(pairs - first) * stride * 8].view(torch.float64).view(-1, stride)[:, :N]
    rows = torch.linspace(0, N - 1, min(N, 9), device="cuda").round().long()
    served = []
    for x in range(first, pairs):
        b, h = divmod(x, H)
        want = torch.stack([torch.logsumexp(k[b, :i + 1, h].double() @ q[b, i, h].double() / d ** 0.5, 0)
                            for i in rows.tolist()])
        got = lse[x - first, rows]
        by2 = bool(((got - want * 1.4426950408889634).abs() <= 1e-6 * (1 + want.abs())).all())
        assert by2 or bool(((got - want).abs() <= 1e-9 * (1 + want.abs())).all()) or not bool(want.isfinite().all())
        served.append(by2)
    return down(key), served


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
@pytest.mark.parametrize("N", [2047, 1936, 1970])     # 128, 121 and 124 blocks: upper halves whole, of one block, and absent
def test_two_blocks_per_wave(F, N, d):
    """128-vector workgroups (1024 of them)."""
    B, H = 4, 16
    q, k = _inputs("normal", B, N, H, d)
    got, served = _scores(F, up_bf16(q), up_bf16(k))
    assert all(served)
    _check(F, "normal", B, N, H, d, got, q, k, (0, 9))


def _assert_sums(key, N):
    """Each row's probabilities sum to 1: N in all, to the fp32 rounding of the keys."""
    total = key.astype(np.float64).sum(-1)
    assert np.all(np.abs(total - N) <= 2.0 ** -22 * N), total


@pytest.mark.parametrize("B,N,H,d,groups", [(1, 16400, 16, 64, 1),      # (two groups of 128-wide heads)
                                            (9, 8177, 9, 64, 2), (1, 16400, 17, 128, 3)])
def test_groups(F, B, N, H, d, groups):
    """Long prompts and batches, whose pairs take one group of the workspace or more, the last one smaller: with the
    workspace that the query asks for the digits serve all of them."""
    assert -(-B * H // column_layout(B, N, H, d)[0]) == groups
    g = torch.Generator(device="cuda").manual_seed(N)
    q, k = (torch.randn(B, N, H, d, device="cuda", generator=g).to(torch.bfloat16) for _ in range(2))
    key, served = _scores(F, q, k)
    assert all(served)
    _assert_sums(key, N)
    for b, h in ((0, 0), (B - 1, H - 1)):
        alone = down(F.column_scores(*(x[b:b + 1, :, h:h + 1].contiguous() for x in (q, k))))
        assert_keys_close(key[b, h], alone[0, 0], f"b={b} h={h}")


def test_many_heads(F):
    """More (batch, head) pairs than a grid's y extent; one position each, whose only probability is 1."""
    B, N, H, d = 35000, 1, 2, 64
    x = torch.randn(B, N, H, d, device="cuda").to(torch.bfloat16)
    assert bool((F.column_scores(x, x) == 1.0).all())


@pytest.mark.parametrize("kind,serves", [("normal", True), ("s2", True), ("s3", True), ("s4", True), ("channel", True),
                                         ("channels", True), ("tiny-q", True), ("tiny-k", True), ("tiny-both", True),
                                         ("zeros", True), ("sharp", True), ("large", False), ("outlier", False),
                                         ("wide", False)])
@pytest.mark.parametrize("d", [64, 128])
def test_values(F, kind, serves, d):
    B, N, H = 1, 300, 2
    q, k = _inputs(kind, B, N, H, d)
    got, served = _scores(F, up_bf16(q), up_bf16(k))
    assert served == [serves, serves or kind == "outlier"]      # (the outlier is in the first head)
    _check(F, kind, B, N, H, d, got, q, k, range(H))


@pytest.mark.parametrize("kind", ["s3", "s4", "channel"])
def test_values_of_a_long_prompt(F, kind):
    """Many vectors, with the rare elements that the digits round, in 128-vector workgroups: the digits serve them."""
    B, N, H, d = 1, 8192, 16, 128
    q, k = (up_bf16(x) for x in _inputs(kind, B, N, H, d))
    got, served = _scores(F, q, k)
    assert all(served)
    want, _ = _scores(F, q, k, 8 * B * N * H)
    for h in range(H):
        assert_keys_close(got[0, h], want[0, h], f"{kind} h={h}")


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
    key, served = _scores(F, up_bf16(q), up_bf16(k), B * H * N * 8)
    assert not any(served)
    return key


def test_small_workspace(F):
    q, k = _inputs("normal", 2, 140, 3, 128)
    want = _small_workspace(F, q, k)
    _check(F, "fp64 products", 2, 140, 3, 128, want, q, k, range(3))
    got = down(F.column_scores(up_bf16(q), up_bf16(k)))
    say("digits against fp64 products")
    for b in range(2):
        for h in range(3):
            assert_keys_close(got[b, h], want[b, h], f"b={b} h={h}")


def _misaligned(x):
    """The same tensor one element (2 bytes) past a 16-byte boundary."""
    y = torch.empty(x.numel() + 8, dtype=x.dtype, device="cuda")[1:1 + x.numel()].view(x.shape)
    assert y.data_ptr() % 16 == 2
    return y.copy_(x)


@pytest.mark.parametrize("d", [64, 128])
def test_misaligned(F, d):
    """Queries or keys off the 16-byte boundary take the fp64 products, in both statistics."""
    q, k, rows, cols, lse = _prune_state("normal", 2, 333, 3, d, 70, 290)
    q, k = up_bf16(q), up_bf16(k)
    rows, cols, lse = (torch.from_numpy(x).cuda() for x in (rows, cols, lse))
    want, served = _scores(F, q, k)
    list_want = down(F.prune_columns(q, k, rows, cols, lse, 4, 5)[1])
    assert all(served)
    for mq, mk in ((_misaligned(q), k), (q, _misaligned(k))):
        got, served = _scores(F, mq, mk, F.load().fl_column_scores_ws(2, 333, 3))
        assert not any(served)
        list_got = down(F.prune_columns(mq, mk, rows, cols, lse, 4, 5)[1])
        for b in range(2):
            for h in range(3):
                assert_keys_close(got[b, h], want[b, h], f"b={b} h={h}")
                assert_keys_close(list_got[b, h], list_want[b, h], f"list b={b} h={h}")


# ---- the list statistic -----------------------------------------------------------------------------------
def _check_prune(F, what, q, k, rows, cols, lse, ns, heads):
    B, N, H, d = q.shape
    _, got = F.prune_columns(up_bf16(q), up_bf16(k), torch.from_numpy(rows).cuda(), torch.from_numpy(cols).cuda(),
                             torch.from_numpy(lse).cuda(), ns, 5)
    got = down(got)
    for b in range(B):
        for h in heads:
            stat = prune.column_mass(cols[b, h], rows[b], bf16_to_f64(q[b, :, h]), bf16_to_f64(k[b, :, h]),
                                     lse[b, :, h].astype(np.float64), 1 / np.sqrt(d), ns)
            assert_keys_close(got[b, h], stat.astype(np.float32), f"{what} b={b} h={h}")


def _prune_state(kind, B, N, H, d, n_ent, k):
    rng = np.random.default_rng(N + d)
    q, kc = _inputs(kind, B, N, H, d)
    pick = lambda n: np.sort(rng.choice(N - 4, n, replace=False)).astype(np.int32) + 4  # noqa: E731
    rows = np.stack([pick(k) for _ in range(B)])
    cols = np.stack([np.stack([np.concatenate([np.arange(4, dtype=np.int32), pick(n_ent)]) for _ in range(H)])
                     for _ in range(B)])
    lse = rng.normal(5.0, 1.0, (B, N, H)).astype(np.float32)
    return q, kc, rows, cols, lse


@pytest.mark.parametrize("d", [64, 128])
def test_prune_two_blocks_per_wave(F, d):
    """128-entry workgroups (528 of them) with a partial last one, the last chunk of rows partial."""
    q, k, rows, cols, lse = _prune_state("normal", 2, 2400, 8, d, 1301, 700)
    _check_prune(F, "normal", q, k, rows, cols, lse, 4, (0, 5))


@pytest.mark.parametrize("kind", ["s4", "channel", "tiny-both", "zeros", "large", "outlier", "wide"])
def test_prune_values(F, kind):
    q, k, rows, cols, lse = _prune_state(kind, 1, 400, 2, 128, 70, 300)
    if kind == "large":
        lse += 640     # (the logits reach about 600: the keys stay finite)
    _check_prune(F, kind, q, k, rows, cols, lse, 4, range(2))


def test_prune_normaliser_out_of_range(F):
    """A log-normaliser beyond the digits' exponents sends its chunk of rows to the fp64 products."""
    q, k, rows, cols, lse = _prune_state("normal", 1, 400, 2, 64, 70, 300)
    lse[0, rows[0, 290]] = 400.0
    lse[0, rows[0, 10], 1] = -340.0
    _, got = F.prune_columns(up_bf16(q), up_bf16(k), torch.from_numpy(rows).cuda(), torch.from_numpy(cols).cuda(),
                             torch.from_numpy(lse).cuda(), 4, 5)
    assert np.isinf(down(got)[0, 1, 0])       # exp(340) is beyond fp32
    _check_prune(F, "normaliser", q, k, rows, cols, lse, 4, (0,))
