"""The calls that a program serving a looped model makes of this package, as measurable cases.

Five kinds, each through the public entry points (paper_2609_29812_amd.driver and .flashloop):

  setup    driver.setup: the dense loop 1 of one layer (base codec, dense attention, column statistic, lists)
  dense    flashloop.dense_attn: the dense causal attention alone
  columns  flashloop.column_scores and select_columns: the column statistic and the lists alone
  codec    flashloop.kv_residual_quant_kv: K and V of every row quantized and rebuilt (the base of a prompt)
  layer    driver.sparse_step: the sparse loops 2..R of one layer (select, quantize and commit, attention)
  decode   flashloop.decode_step: the newest position, a dense loop and then sparse ones over its selection
  prune    flashloop.prune_columns: the lists cut to a smaller budget between two loops

States are drawn as the method meets them: loop-1 Q, K and V are standard normal in bf16, every later loop
adds a small change to each row and a large one to a nested set of hot rows.  What a step starts from (the
caches, the first loop's output and log-normalisers, the column lists) is made here in plain torch.
"""
import math
from types import SimpleNamespace

import torch

from paper_2609_29812_amd import driver
from paper_2609_29812_amd import flashloop as fl

SINK = 4       # leading columns every list keeps
BASE_BITS = 4  # bit width of the loop-1 base
COLD = 0.01    # change of a row between two loops; a hot row's is HOT
HOT = 0.5


def listed():
    return [
        # the dense first loop of a 4K prompt, one layer of 16 heads x 128: what each layer of a prefill begins with
        dict(name="setup_4k", kind="setup", B=1, N=4096, H=16, d=128, bits=4, group=64, t=508, tail=0),
        # its attention alone for a 16K prompt, and for a few short prompts of uneven length with 64-wide heads
        dict(name="dense_16k", kind="dense", B=1, N=16384, H=16, d=128),
        dict(name="dense_ragged", kind="dense", B=3, N=1009, H=8, d=64),
        # the column statistic and the lists of an 8K prompt
        dict(name="columns_8k", kind="columns", B=1, N=8192, H=16, d=128, t=1020),
        # the int4 base of a 32K prompt's keys and values
        dict(name="codec_32k", kind="codec", B=1, N=32768, H=16, d=128, bits=4, group=64),
        # the smallest layer: one sparse loop over 256 positions, where launches count
        dict(name="step_tiny", kind="layer", B=1, N=256, H=2, d=64, R=2, first=0.25, last=0.25, c=32, window=0,
             bits=4, group=32, tail=0),
        # one layer of a 4-loop model: a 4K prompt, and a 32K prompt with a local window and 2-bit residuals
        dict(name="layer_4k", kind="layer", B=1, N=4096, H=16, d=128, R=4, first=0.10, last=0.10, c=512, window=0,
             bits=4, group=64, tail=0),
        dict(name="layer_32k", kind="layer", B=1, N=32768, H=16, d=128, R=4, first=0.05, last=0.05, c=2048, window=512,
             bits=2, group=64, tail=0),
        # the first sparse loop of a batch of four 16K prompts, a fifth of the rows updated
        dict(name="step_b4_16k", kind="layer", B=4, N=16384, H=16, d=128, R=2, first=0.20, last=0.20, c=1024, window=0,
             bits=4, group=64, tail=0),
        # decoding: the dense loop over a 32K context, and the four loops of one position for a batch of eight
        dict(name="decode_32k", kind="decode", B=1, T=32768, H=16, d=128, R=1, c=2048, window=512),
        dict(name="decode_b8_8k", kind="decode", B=8, T=8192, H=16, d=128, R=4, c=1024, window=64),
        # the lists of the 32K layer halved after a loop
        dict(name="prune_32k", kind="prune", B=1, N=32768, H=16, d=128, k=1638, c=1536, t=766),
    ]


# ---- drawn cases: the ranges between and around the listed ones -------------------------------------------
def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """A case of the listed kinds: lengths 64..32768 (any, not only round ones), 1..8 sequences, 2..16 heads of
    64 or 128, groups of 32 or 64, 2-, 4- and 8-bit residuals, with and without a window and a bf16 tail."""
    kind = rng.choice(("setup", "dense", "columns", "codec", "layer", "layer", "layer", "decode", "decode", "prune"))
    H, d = rng.choice((2, 4, 5, 8, 12, 16)), rng.choice((64, 128))
    group = rng.choice((32, 64))
    if kind in ("setup", "dense", "columns"):
        most = {"setup": 4096, "dense": 16384, "columns": 8192}[kind]
        N = _log(rng, 64, most)
        B = rng.randint(1, max(1, min(4, (most * most) // (N * N))))
        t = rng.randint(1, max(1, (N - SINK) // 4))
        if kind == "setup":
            return dict(kind=kind, B=B, N=N, H=H, d=d, bits=rng.choice((4, 8)), group=group, t=t,
                        tail=rng.choice((0, 64)))
        return dict(kind=kind, B=B, N=N, H=H, d=d, **({"t": t} if kind == "columns" else {}))
    if kind == "codec":
        N = _log(rng, 128, 32768)
        return dict(kind=kind, B=rng.randint(1, max(1, min(4, 32768 // N))), N=N, H=H, d=d,
                    bits=rng.choice((2, 4, 8)), group=group)
    if kind == "layer":
        N = _log(rng, 256, 32768)
        B = rng.randint(1, max(1, min(4, 65536 // N)))
        first = rng.uniform(0.03, 0.20)
        window = rng.choice((0, 0, rng.randint(16, 512)))
        return dict(kind=kind, B=B, N=N, H=H, d=d, R=rng.randint(2, 4 if B == 1 else 2), first=first,
                    last=first * rng.uniform(0.3, 1.0), c=min(N // 2, window + SINK + _log(rng, 32, 1536)),
                    window=min(window, N // 4), bits=rng.choice((2, 4)), group=group, tail=rng.choice((0, 0, 64)))
    if kind == "decode":
        T = _log(rng, 256, 32768)
        return dict(kind=kind, B=rng.randint(1, max(1, min(8, 65536 // T))), T=T, H=H, d=d, R=rng.randint(1, 4),
                    c=min(T // 2, _log(rng, 32, 2048)), window=rng.choice((0, 16, 64)))
    N = _log(rng, 512, 32768)
    c = min(N // 2, _log(rng, 64, 1536))
    return dict(kind=kind, B=1, N=N, H=H, d=d, k=max(1, int(N * rng.uniform(0.02, 0.10))), c=c,
                t=max(1, int((c - SINK) * rng.uniform(0.3, 0.9))))


# ---- the states ------------------------------------------------------------------------------------------
def _normal(g, *shape):
    return torch.randn(shape, generator=g, device="cuda")


def _budget(case, r):
    """Rows updated in loop r (2..R): a geometric decay from `first` to `last`, never more than before."""
    n = case["N"]
    for rr in range(2, r + 1):
        f = case["first"] * (case["last"] / case["first"]) ** ((rr - 2) / max(1, case["R"] - 2))
        n = min(n, max(1, math.floor(f * case["N"] + 0.5)))
    return n


def _loop_states(case, g):
    """Q, K, V of loops 1..R as lists of bf16 [B, N, H, d]: the hot rows of a loop are among the last one's."""
    B, N, H, d = (case[x] for x in "BNHd")
    out = {n: [_normal(g, B, N, H, d).to(torch.bfloat16)] for n in "qkv"}
    hot = [torch.arange(N, device="cuda") for _ in range(B)]
    for r in range(2, case["R"] + 1):
        hot = [h[torch.randperm(h.numel(), generator=g, device="cuda")[:_budget(case, r)]].sort().values for h in hot]
        for n in "qkv":
            delta = _normal(g, B, N, H, d) * COLD
            for b in range(B):
                delta[b, hot[b]] = _normal(g, hot[b].numel(), H, d) * HOT
            out[n].append((out[n][-1].float() + delta).to(torch.bfloat16))
    return out


def _dense(q, k, v, dtype, stats=True, chunk=2048):
    """Dense causal attention in `dtype`: o [B, N, H, d], lse [B, N, H] and the column sums of the
    probabilities [B, H, N] (None without stats)."""
    B, N, H, d = q.shape
    o = torch.empty(B, N, H, d, dtype=dtype, device=q.device)
    lse = torch.empty(B, N, H, dtype=dtype, device=q.device)
    col = torch.zeros(B, H, N, dtype=dtype, device=q.device) if stats else None
    for b in range(B):
        for h in range(H):
            kk, vv = k[b, :, h].to(dtype), v[b, :, h].to(dtype)
            for i in range(0, N, chunk):
                e = min(N, i + chunk)
                s = (q[b, i:e, h].to(dtype) @ kk[:e].T) * (1.0 / math.sqrt(d))
                s[:, i:].masked_fill_(torch.ones(e - i, e - i, dtype=torch.bool, device=q.device).triu(1), -math.inf)
                lse[b, i:e, h] = torch.logsumexp(s, 1)
                s = s.sub_(lse[b, i:e, h, None]).exp_()
                o[b, i:e, h] = s @ vv[:e]
                if stats:
                    col[b, h, :e] += s.sum(0)
    return o, lse, col


def _half_towards(x, up):
    """The nearest float16 at or above (up) or at or below x (float64)."""
    h = x.clamp(-65504, 65504).to(torch.float16)

    def step(v, up):
        bits = v.view(torch.int16).to(torch.int32)
        key = torch.where(bits < 0, -(bits & 0x7FFF), bits) + (1 if up else -1)
        return torch.where(key < 0, (-key) | -0x8000, key).to(torch.int16).view(torch.float16)

    past = (lambda v: v.double() < x) if up else (lambda v: v.double() > x)
    h = torch.where(past(h), step(h, up), h)
    back = step(h, not up)
    return torch.where(past(back), h, back) + 0.0


def _rebuild(cur, ref, bits, group, token):
    """Rows [k, H, d] after the residual codec, as bf16: groups of `group` rows per channel (token) or of
    `group` channels per row."""
    ref = torch.zeros_like(cur) if ref is None else ref
    delta = cur.float() - ref.float()
    k, H, d = delta.shape
    if token:
        pad = -k % group
        x = torch.cat([delta, delta[-1:].expand(pad, H, d)]).reshape(-1, group, H, d)
        dim = 1
    else:
        x, dim = delta.reshape(k, H, d // group, group), 3
    z = _half_towards(x.amin(dim, keepdim=True).double(), False)
    s = _half_towards((x.amax(dim, keepdim=True).double() - z.double()) / (2 ** bits - 1), True).float()
    z = z.float()
    q = torch.where(s == 0, torch.zeros_like(x), torch.round((x - z) / s).clamp(0, 2 ** bits - 1))
    dq = (z + q * s).reshape(-1, H, d)[:k]
    return (ref.float() + dq).to(torch.bfloat16)


def _base(x, bits, group, token, tail):
    hat = torch.stack([_rebuild(x[b], None, bits, group, token) for b in range(x.shape[0])])
    if tail:
        hat[:, -tail:] = x[:, -tail:]
    return hat


def _lists(col_key, t):
    """Column lists [B, H, SINK + t]: the leading columns and the t others with the largest keys, ascending."""
    B, H, N = col_key.shape
    top = torch.sort(col_key[:, :, SINK:], dim=2, descending=True, stable=True).indices[:, :, :t] + SINK
    sink = torch.arange(SINK, device=col_key.device).expand(B, H, SINK)
    return torch.cat([sink, top], 2).sort(2).values.to(torch.int32)


def _generator(seed):
    return torch.Generator(device="cuda").manual_seed(seed)


def _prompt(case, g):
    """q, k, v of a loop 1 as bf16 [B, N, H, d]."""
    B, N, H, d = (case[x] for x in "BNHd")
    return [_normal(g, B, N, H, d).to(torch.bfloat16) for _ in range(3)]


def _layer(case, seed):
    """The loops' states and what loop 1 left: caches, output, log-normalisers and lists."""
    x = _loop_states(case, _generator(seed))
    k_hat = _base(x["k"][0], BASE_BITS, case["group"], True, case["tail"])
    v_hat = _base(x["v"][0], BASE_BITS, case["group"], False, case["tail"])
    o, lse, col = _dense(x["q"][0], k_hat, v_hat, torch.float32)
    t = max(1, min(case["c"] - SINK - case["window"], case["N"] - SINK))
    return x, driver.LayerState(k_hat, v_hat, o, lse, _lists(col.float(), t), None, case["window"], case["group"],
                                tail=case["tail"], v16=v_hat.half())


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("setup", "dense", "columns", "codec"):
        return SimpleNamespace(case=case, x=_prompt(case, _generator(seed)))
    if kind == "layer":
        x, st = _layer(case, seed)
        return SimpleNamespace(case=case, x=x, st=st, lse=st.lse.clone() if case["R"] > 2 else None, turn=0)
    if kind == "decode":
        return _decode_state(case, seed)
    q, k, _ = _prompt(case, _generator(seed))
    _, lse, col = _dense(q, k, k, torch.float32)
    g = _generator(seed + 1)
    rows = torch.randperm(case["N"], generator=g, device="cuda")[:case["k"]].sort().values
    return SimpleNamespace(case=case, q=q, k=k, lse=lse, rows=rows.to(torch.int32)[None].contiguous(),
                           cols=_lists(col, case["c"] - SINK))


def _decode_state(case, seed):
    """Caches of R loops over T positions and the newest position's queries; buffers kept between positions."""
    g = _generator(seed)
    B, T, H, d = (case[x] for x in "BTHd")
    k, v, q = [_normal(g, B, T, H, d)], [_normal(g, B, T, H, d)], [_normal(g, B, H, d)]
    for _ in range(case["R"] - 1):
        k.append(k[-1] + _normal(g, B, T, H, d) * 0.1)
        v.append(v[-1] + _normal(g, B, T, H, d) * 0.1)
        q.append(q[-1] + _normal(g, B, H, d) * 0.1)
    k, v, q = ([t.to(torch.bfloat16) for t in u] for u in (k, v, q))
    out = [(torch.empty(B, H, case["c"], dtype=torch.int32, device="cuda"), torch.empty(B, H, device="cuda"),
            torch.empty(B, H, d, device="cuda")) for _ in range(case["R"])]
    ws = max((fl.decode_ws(k[0], c, case["c"]) for c in (None, out[0][0])), key=lambda w: w.numel())
    return SimpleNamespace(case=case, q=q, k=k, v=v, o=torch.empty(B, H, d, device="cuda"),
                           lse=torch.empty(B, H, device="cuda"), out=out, ws=ws)


# ---- one pass ---------------------------------------------------------------------------------------------
def _fields(st):
    return dict(o=st.o, lse=st.lse, k_hat=st.k_hat, v_hat=st.v_hat, v16=st.v16, cols=st.cols)


def run(s):
    case = s.case
    kind = case["kind"]
    if kind == "setup":
        st = driver.setup(*s.x, case["bits"], case["group"], SINK, case["t"], 0, tail=case["tail"])
        return dict(_fields(st), **st.base)
    if kind == "dense":
        return fl.dense_attn(*s.x)
    if kind == "columns":
        key = fl.column_scores(s.x[0], s.x[1])
        return key, fl.select_columns(key, SINK, case["t"])
    if kind == "codec":
        return fl.kv_residual_quant_kv(s.x[1], None, s.x[2], None, None, case["bits"], case["group"])
    if kind == "layer":
        return _run_layer(s)
    if kind == "decode":
        cols = mass = sub = None
        for r in range(case["R"]):
            cols, mass, sub = fl.decode_step(s.q[r], s.k[r], s.v[r], cols, mass, sub, s.o, case["c"], n_sink=SINK,
                                             window=case["window"], lse=s.lse, out=s.out[r], ws=s.ws)
        return dict(o=s.o, lse=s.lse, cols=cols, mass=mass, sub=sub)
    return fl.prune_columns(s.q, s.k, s.rows, s.cols, s.lse, SINK, case["t"])


def _run_layer(s):
    """Loops 2..R of the layer.  A pass after the first runs on the state the last one left: two loops go back
    and forth between their states; of more, each pass begins with the log-normalisers of the set-up."""
    case, st, x = s.case, s.st, s.x
    st.cand = st.term = st.mass = st.slot_prev = None
    if case["R"] == 2:
        order = [1 - s.turn, s.turn]
        s.turn = 1 - s.turn
        order.reverse()
    else:
        st.lse.copy_(s.lse)
        order = list(range(case["R"]))
    kept = []
    for r in range(2, case["R"] + 1):
        p, c = order[r - 2], order[r - 1]
        kept.append(driver.sparse_step(st, x["q"][c], x["q"][p], x["k"][c], x["k"][p], x["v"][c], x["v"][p],
                                       _budget(case, r), case["bits"], keep=True))
    return dict(_fields(st), loops=kept, term=st.term, mass=st.mass)


# ---- what a pass cannot do without -------------------------------------------------------------------------
def work(case):
    """Bytes: each input read once and each output written once.  Flops: the products of the method."""
    kind, H, d = case["kind"], case["H"], case["d"]
    B = case["B"]
    if kind == "decode":
        T, c = case["T"], case["c"]
        columns = B * H * (T + (case["R"] - 1) * c)
        return {"bytes": columns * 4 * d + case["R"] * B * H * (2 * d + 8 * d + 4 * c), "flops": columns * 4 * d}
    N = case["N"]
    row, pairs = H * d, B * H * N * (N + 1) / 2
    if kind == "dense":
        return {"bytes": B * N * (10 * row + 4 * H), "flops": 4 * d * pairs}
    if kind == "columns":
        return {"bytes": B * N * (4 * row + 4 * H) + 4 * B * H * case["t"], "flops": 4 * d * pairs}
    if kind in ("setup", "codec"):
        coded = B * N * row * (4 + 4 + case["bits"] / 4 + 8 / case["group"])
        if kind == "codec":
            return {"bytes": coded, "flops": 0}
        return {"bytes": coded + B * N * row * (2 + 4 + 2) + B * N * H * 8, "flops": 8 * d * pairs}
    if kind == "prune":
        k, c = case["k"], case["c"]
        return {"bytes": B * H * ((k + c) * 2 * d + 8 * c + 4 * k), "flops": 2 * d * B * H * k * c}
    total = {"bytes": 0.0, "flops": 0.0}
    t, w, cand = case["c"] - case["window"], case["window"], N
    for r in range(2, case["R"] + 1):
        k = _budget(case, r)
        touched = min(N, t + (N * (1 - (1 - k / N) ** w) if w else 0))
        passes = 2 if r == 2 else 1
        total["bytes"] += B * (cand * 8 * row + k * row * (4 + 6 + case["bits"] / 4) + passes * touched * 4 * row
                               + k * row * (2 * passes + 8 + 8))
        total["flops"] += passes * 4 * d * B * H * k * min(N, t + w)
        cand = k
    return total


# ---- how far another correct implementation may be -----------------------------------------------------------
def tolerance(case):
    """The codec is defined to the bit.  Statistics and decode logits are 64-bit sums rounded to float32 (a list may
    swap two columns whose keys tie to the last bit); attention multiplies probabilities rounded to float16."""
    kind = case["kind"]
    if kind == "codec":
        return "exact"
    if kind in ("columns", "prune"):
        return {"rel": 1e-6, "max": 1e-5, "differ": 2e-3}
    if kind == "decode":
        return {"rel": 1e-5, "max": 1e-4, "differ": 2e-3}
    return {"rel": 1e-3, "max": 2e-2, "differ": 2e-3 if kind == "setup" else 0.0}


# ---- the same in 64 bits -------------------------------------------------------------------------------------
def exact(case, seed):
    kind = case["kind"]
    if kind == "codec":
        return None
    if kind == "layer":
        return _exact_layer(case, seed)
    if kind == "decode":
        return _exact_decode(_decode_state(case, seed))
    if kind == "prune":
        s = prepare(case, seed)
        key = torch.empty(1, case["H"], case["c"] - SINK, dtype=torch.float64, device="cuda")
        rows = s.rows[0].long()
        for h in range(case["H"]):
            js = s.cols[0, h, SINK:].long()
            p = torch.exp((s.q[0, rows, h].double() @ s.k[0, js, h].double().T) / math.sqrt(case["d"])
                          - s.lse[0, rows, h, None].double())
            key[0, h] = (p * (rows[:, None] >= js[None, :])).sum(0)
        return None, key
    q, k, v = _prompt(case, _generator(seed))
    if kind == "dense":
        return _dense(q, k, v, torch.float64, stats=False)[:2]
    if kind == "columns":
        return _dense(q, k, k, torch.float64)[2], None
    k_hat = _base(k, case["bits"], case["group"], True, case["tail"])
    v_hat = _base(v, case["bits"], case["group"], False, case["tail"])
    o, lse, col = _dense(q, k_hat, v_hat, torch.float64)
    return dict(o=o, lse=lse, col_key=col)


def _exact_layer(case, seed):
    """The first pass: selection, codec and the mass-corrected update of each loop, the update in 64 bits."""
    x, st = _layer(case, seed)
    B, N, H, d = (case[n] for n in "BNHd")
    o, lse, scale, w = st.o.double(), st.lse.double(), 1.0 / math.sqrt(d), case["window"]
    j = torch.arange(N, device="cuda")
    cand = [j] * B
    for r in range(2, case["R"] + 1):
        k = _budget(case, r)
        term = torch.zeros(B, k, H, d, dtype=torch.float64, device="cuda")
        mass = torch.zeros(B, k, H, dtype=torch.float64, device="cuda")
        old = st.k_hat.clone(), st.v_hat.clone()
        for b in range(B):
            num = den = 0.0
            for n in "kv":
                cur, prev = x[n][r - 1][b, cand[b]].float(), x[n][r - 2][b, cand[b]].float()
                num = num + (cur - prev).double().square().sum((1, 2))
                den = den + cur.double().square().sum((1, 2))
            key = (num.sqrt() / (den.sqrt() + 1e-6)).float()
            rows = cand[b] = cand[b][torch.sort(key, descending=True, stable=True).indices[:k].sort().values]
            for n, hat in (("k", st.k_hat), ("v", st.v_hat)):
                new = _rebuild(x[n][r - 1][b, rows], hat[b, rows], case["bits"], case["group"], n == "k")
                recent = rows >= N - case["tail"]
                hat[b, rows] = torch.where(recent[:, None, None], x[n][r - 1][b, rows], new)
            for h in range(H):
                listed_ = torch.zeros(N, dtype=torch.bool, device="cuda")
                listed_[st.cols[b, h].long()] = True
                seen = (listed_[None, :] | (j[None, :] > rows[:, None] - w)) & (j[None, :] <= rows[:, None])
                a = (x["q"][r - 2][b, rows, h].double() @ old[0][b, :, h].double().T) * scale - lse[b, rows, h, None]
                pp = torch.exp(a.masked_fill_(~seen, -math.inf))
                m = pp.sum(1)
                sub = pp @ old[1][b, :, h].double()
                a = (x["q"][r - 1][b, rows, h].double() @ st.k_hat[b, :, h].double().T) * scale
                L = torch.logsumexp(a.masked_fill_(~seen, -math.inf), 1)
                add = (torch.exp(a - L[:, None]) @ st.v_hat[b, :, h].double()) * m[:, None]
                o[b, rows, h] += add - sub
                lse[b, rows, h] = L - torch.log(m)
                term[b, :, h], mass[b, :, h] = add, m
    return dict(o=o, lse=lse, term=term, mass=mass)


def _exact_decode(s):
    case = s.case
    B, T, H, d = (case[x] for x in "BTHd")
    o, sub = (torch.zeros(B, H, d, dtype=torch.float64, device="cuda") for _ in range(2))
    lse, mass = (torch.zeros(B, H, dtype=torch.float64, device="cuda") for _ in range(2))
    for b in range(B):
        for h in range(H):
            cols = torch.arange(T, device="cuda")
            m = 1.0
            for r in range(case["R"]):
                v = s.v[r][b, cols, h].double()
                a = (s.k[r][b, cols, h].double() @ s.q[r][b, h].double()) / math.sqrt(d)
                lse[b, h] = torch.logsumexp(a, 0)
                p = torch.exp(a - lse[b, h]) * m
                o[b, h] = p @ v if r == 0 else o[b, h] - sub[b, h] + p @ v
                key = a.float().masked_fill((cols < SINK) | (cols >= T - case["window"]), math.inf)
                keep = torch.sort(key, descending=True, stable=True).indices[:case["c"]].sort().values
                cols, m = cols[keep], p[keep].sum()
                mass[b, h], sub[b, h] = m, p[keep] @ v[keep]
    return dict(o=o, lse=lse, mass=mass, sub=sub)
