"""The radix top-k where its layouts end, and the decode step with several selecting workgroups, against the oracle.

Top-k (bit-exact): key counts around every thread count and register depth, two blocks of positions per thread, and
keys that are random, tied, mostly at the lowest value, infinite or signed.  Decode: shares of the selection that are
even, uneven and single, in both head dimensions, the selections identical and the sums within the decode tolerance.
"""
import numpy as np
import pytest
import torch

from gpu_util import down, say, up, up_bf16
from oracle import decode as odec
from oracle import select
from oracle.numerics import bf16_to_f64, f32_to_bf16

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def F():
    from paper_2609_29812_amd import flashloop
    flashloop.load()
    return flashloop


def _keys(kind, n, rng):
    if kind == "random":
        return rng.standard_normal(n).astype(np.float32)
    if kind == "tied":
        return rng.choice(np.float32([-2.0, -0.0, 0.0, 1e-30, 7.0]), n).astype(np.float32)
    if kind == "lowest":                      # most keys share the lowest value of their type
        return np.where(rng.random(n) < 0.9, np.float32(-np.inf), rng.standard_normal(n)).astype(np.float32)
    return np.where(rng.random(n) < 0.1, np.float32(np.inf), rng.random(n) * np.float32(1e-3)).astype(np.float32)


@pytest.mark.parametrize("n", [1, 63, 64, 255, 256, 257, 1023, 1024, 1025, 2048, 2049, 4096, 4097, 8192, 8193, 16385,
                               32768, 32769, 65536])
def test_topk_lengths(F, n):
    rng = np.random.default_rng(n)
    for kind in ("random", "tied", "lowest", "infinite"):
        keys = np.stack([_keys(kind, n, rng), _keys(kind, n, rng)])[None]
        for t in sorted({1, n // 20, n // 2, n - 1, n} - {0}):
            got = down(F.select_columns(up(keys), 0, t))[0]
            for h in range(2):
                # (descending, ties to the lower index)
                want = np.sort(np.argsort(-keys[0, h].astype(np.float64), kind="stable")[:t])
                assert np.array_equal(got[h], want), f"n={n} kind={kind} t={t} h={h}"
    say(f"top-k n={n} ok")


def test_topk_slots_and_candidates(F):
    """The slot map and candidate ids at a key count with a partial last thread."""
    rng = np.random.default_rng(3)
    B, N, D = 2, 3000, 64
    x = [f32_to_bf16(rng.standard_normal((B, N, D)).astype(np.float32)) for _ in range(4)]
    cand = np.stack([np.sort(rng.choice(N, 2111, replace=False)) for _ in range(B)]).astype(np.int32)
    k = 333
    idx, slot, key = F.select_tokens(*[up_bf16(a.reshape(B, N, 1, D)) for a in x], k, cand=up(cand))
    want_idx, want_slot = select.nested_topk(down(key), cand, k, N)
    assert np.array_equal(down(idx), want_idx)
    assert np.array_equal(down(slot), want_slot)


@pytest.mark.parametrize("B,H,d,T,c", [(1, 2, 128, 3000, 259), (1, 2, 128, 3000, 260), (1, 3, 64, 2500, 1001),
                                       (2, 20, 128, 1400, 1399), (1, 2, 64, 9000, 8200), (1, 1, 128, 33000, 2048)])
def test_decode_shares(F, B, H, d, T, c):
    rng = np.random.default_rng(T + c)
    q = f32_to_bf16(rng.standard_normal((B, H, d)).astype(np.float32))
    k, v = (f32_to_bf16(rng.standard_normal((B, T, H, d)).astype(np.float32)) for _ in range(2))
    o = torch.empty(B, H, d, device="cuda")
    lse = torch.empty(B, H, device="cuda")
    cols, mass, sub = F.decode_step(up_bf16(q), up_bf16(k), up_bf16(v), None, None, None, o, c, n_sink=4, window=16,
                                    lse=lse)
    cols, mass, sub, o, lse = (down(t) for t in (cols, mass, sub, o, lse))
    for b in range(B):
        for h in range(0, H, 7):
            wo, wc, wm, ws, wl = odec.decode_step(bf16_to_f64(q[b, h]), bf16_to_f64(k[b, :, h]), bf16_to_f64(v[b, :, h]),
                                                  None, None, None, None, 1 / np.sqrt(d), 4, 16, c)
            assert np.array_equal(cols[b, h], wc)
            # fp32 sums of at most T terms in any order: T 2^-24 of the sum of their magnitudes bounds the error, which
            # random signs leave at its square root
            bound = 8 * np.sqrt(T) * 2.0 ** -24
            for got, want, what in ((o[b, h], wo, "o"), (sub[b, h], ws, "sub")):
                assert np.max(np.abs(got - want)) <= bound, what
            assert abs(mass[b, h] - wm) <= 2.0 ** -22 and abs(lse[b, h] - wl) <= 2.0 ** -22 * max(1, abs(wl))
