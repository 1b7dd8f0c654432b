"""The calls this library is timed on: one generation step of an attention layer, through the public
entry points, over the range of layers, batches, contexts, caches and options that callers have.

A case is a plain dict:
  entry   which public call: decode | decode_static | xcache | block | vanilla_block
  B, H, d_k, T   sequences, heads, head width, rows of the cache (after the append, for a block)
  d       width of a cached row: H * d_k, or the layer input's width for an X-cache
  lo      0: every sequence has T rows; else the lengths spread from lo to T (a ragged batch)
  dtype   "bf16" | "f32": elements of the cache and the weights
  banded  the K-cache is stored in 32-row bands, head-major inside a band
  rope    the keys carry rotary positions

Values are random, on the scale that a trained layer has them: unit keys, values and inputs, weights of
variance 1 / fan-in, queries whose scores spread by one or two (so the softmax is neither flat nor one-hot).
"""
import math

import torch

from paper_2503_05840_amd import binding

_T = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(name, entry, B, H, d_k, T, d=0, lo=0, dtype="bf16", banded=False, rope=False):
    return {"name": name, "entry": entry, "B": B, "H": H, "d_k": d_k, "T": T, "d": d or H * d_k, "lo": lo,
            "dtype": dtype, "banded": banded, "rope": rope}


def listed():
    return [
        # the smallest layer in full precision: latency and launches are all there is
        _case("decode f32 tiny", "decode", 1, 8, 64, 256, dtype="f32"),
        # a full-precision cache in a small ragged batch: a model served as it was trained
        _case("decode f32 batch", "decode", 4, 16, 64, 1500, lo=300, dtype="f32"),
        # one chat turn on a 7B-shaped layer: short odd context, one sequence, the call that never allocates
        _case("decode short", "decode_static", 1, 32, 128, 777),
        # the same layer at its full context (CodeLlama-7B-shaped, 16k rows)
        _case("decode 16k", "decode", 1, 32, 128, 16384),
        # long ragged contexts in a batch (Phi-3-mini-shaped), the K-cache in its banded layout: the largest call
        _case("decode ragged long", "decode", 16, 32, 96, 32768, lo=8192, banded=True),
        # decoder cross-attention over 1500 encoder frames (Whisper-large-shaped), a full batch
        _case("decode cross", "decode", 64, 20, 64, 1500),
        # rotary keys, ragged contexts of a chat batch, row-major cache as other software writes it
        _case("decode rotary", "decode", 8, 32, 96, 5000, lo=600, rope=True),
        # a layer of more than 32 heads (a 13B-sized model's), two conversations of different length
        _case("decode 40 heads", "decode", 2, 40, 128, 4001, lo=2500),
        # wide projections over a shared encoder output (T5-11B-shaped): only X is cached
        _case("xcache wide", "xcache", 8, 128, 128, 4096, d=1024),
        # the encoder output as the only cache of square cross-attention layers (Whisper-large-shaped)
        _case("xcache encoder", "xcache", 24, 20, 64, 1500, d=1280),
        # one token through the whole attention block: projections, append, step, output projection; a
        # chat batch with rotary positions
        _case("block rotary", "block", 16, 32, 128, 2049, lo=300, rope=True),
        # the same block with K and V caches, which the others are compared with
        _case("block vanilla", "vanilla_block", 4, 32, 128, 4099),
    ]


def _rows(c):
    """Rows of every sequence: T, or spread over lo..T in a fixed order that is neither sorted nor periodic."""
    B, T, lo = c["B"], c["T"], c["lo"]
    if not lo:
        return [T] * B
    return [T] + [lo + int((T - lo) * (b * 0.6180339887498949 % 1.0)) for b in range(1, B)]


def _esize(c):
    return 2 if c["dtype"] == "bf16" else 4


def work(case):
    c = case
    n, e, d, B = sum(_rows(c)), c["H"] * c["d_k"], c["d"], c["B"]
    z = _esize(c)
    if c["entry"] == "xcache":          # X once, W_K and W_V; q~ = q W_K^T, scores and sums over whole rows
        return {"bytes": n * d * z + 2 * d * e * z + 2 * B * e * 4, "flops": 4 * n * c["H"] * d + 4 * B * d * e}
    if c["entry"] == "vanilla_block":   # K and V once, four weights
        return {"bytes": 2 * n * d * z + 4 * d * d * z + 2 * B * d * 4, "flops": 4 * n * d + 8 * B * d * d}
    nw = 4 if c["entry"] == "block" else 1
    return {"bytes": n * d * z + nw * d * d * z + 2 * B * d * 4, "flops": 2 * n * d + 2 * n * c["H"] * d + 2 * nw * B * d * d}


def tolerance(case):
    return {"rel": 1e-5} if case["dtype"] == "f32" else {"rel": 1e-2}


def draw(rng):
    """One more call from the same ranges: a listed kind with other sizes, odd ones among them."""
    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(["f32", "one", "batch", "batch", "cross", "rotary", "heads", "xcache", "encoder", "block", "vanilla"])
    if kind == "f32":
        H = rng.choice([4, 8, 12, 16])
        T = spread(100, 3000)
        return _drop(_case("", "decode", spread(1, 8), H, 64, T, lo=rng.choice([0, max(1, T // 5)]), dtype="f32"))
    if kind == "one":
        H, d_k = rng.choice([(32, 128), (32, 96), (32, 80), (20, 64), (16, 128)])
        return _drop(_case("", rng.choice(["decode", "decode_static"]), 1, H, d_k, spread(200, 16384)))
    if kind == "batch":
        H, d_k = rng.choice([(32, 96), (32, 128), (24, 128), (20, 64)])
        B, T = spread(2, 32), spread(500, 20000)
        T = min(T, 300_000 * 3072 // (B * H * d_k))
        banded = rng.random() < 0.5
        return _drop(_case("", "decode", B, H, d_k, (T + 31) // 32 * 32 if banded else T, lo=max(1, T // rng.randint(3, 8)), banded=banded))
    if kind == "cross":
        H = rng.choice([6, 8, 12, 16, 20])
        return _drop(_case("", "decode", spread(8, 96), H, 64, rng.choice([1500, 1500, 750, 448, 1000])))
    if kind == "rotary":
        H, d_k = rng.choice([(32, 96), (32, 128), (16, 128)])
        T = spread(300, 8000)
        return _drop(_case("", "decode", spread(1, 12), H, d_k, T, lo=max(1, T // 6), rope=True))
    if kind == "heads":
        H, d_k = rng.choice([(40, 128), (36, 64), (48, 128), (64, 128), (40, 96)])
        T = spread(400, 6000)
        return _drop(_case("", "decode", spread(1, 4), H, d_k, T, lo=rng.choice([0, T // 2])))
    if kind == "xcache":
        H, d = rng.choice([(32, 1024), (64, 1024), (128, 1024), (64, 768)])
        return _drop(_case("", "xcache", spread(1, 8), H, 128, spread(300, 4096), d=d, lo=rng.choice([0, 200])))
    if kind == "encoder":
        H = rng.choice([8, 12, 16, 20])
        return _drop(_case("", "xcache", spread(4, 64), H, 64, rng.choice([1500, 1500, 750, 1000]), d=64 * H))
    H, d_k = rng.choice([(32, 128), (32, 96), (20, 64)])
    T = spread(200, 5000)
    if kind == "block":
        return _drop(_case("", "block", spread(1, 24), H, d_k, T, lo=max(1, T // 6), rope=rng.random() < 0.5))
    return _drop(_case("", "vanilla_block", spread(1, 12), H, d_k, T, lo=rng.choice([0, max(1, T // 4)])))


def _drop(c):
    return {k: v for k, v in c.items() if k != "name"}


# ---- inputs -------------------------------------------------------------------------------------------

def _inputs(c, seed):
    """What the call is given, from the seed alone: the same tensors for the library and for exact()."""
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    B, H, d, T = c["B"], c["H"], c["d"], c["T"]
    e = H * c["d_k"]

    def rnd(*shape, std=1.0, dtype=None):
        t = torch.randn(shape, generator=g, device="cuda", dtype=dtype or _T[c["dtype"]])
        return t if std == 1.0 else t.mul_(std)

    s = {"lens": torch.tensor(_rows(c), dtype=torch.int32, device="cuda") if c["lo"] else None}
    if c["entry"] == "xcache":
        s["x"] = rnd(B, e, dtype=torch.float32)                   # the projected queries
        s["cache"] = rnd(B, T, d)
        s["W_K"], s["W_V"] = rnd(d, e, std=d ** -0.5), rnd(d, e, std=d ** -0.5)
        return s
    block = c["entry"] in ("block", "vanilla_block")
    s["x"] = rnd(B, d, std=1.0 if block else 2.0, dtype=torch.float32)     # block: the tokens' inputs; else projected queries
    s["cache"] = rnd(B, T, d)
    if c["entry"] == "vanilla_block":
        s["vcache"] = rnd(B, T, d)
        s["W_V"] = rnd(d, d, std=d ** -0.5)
    else:
        s["W_KV"] = rnd(d, d, std=d ** -0.5)
    if block:
        for k in ("W_Q", "W_K", "W_O"):
            s[k] = rnd(d, d, std=d ** -0.5)
    return s


def prepare(case, seed):
    """The caches and weights a serving process holds, a workspace of its own, and the outputs' buffers."""
    c = dict(case)
    s = _inputs(c, seed)
    s["case"] = c
    B, H, T, d, dt = c["B"], c["H"], c["T"], c["d"], c["dtype"]
    binding.slim_init()
    s["out"] = torch.empty((B, H * c["d_k"]), device="cuda", dtype=torch.float32)
    if c["entry"] != "decode_static":
        need = {"decode": lambda: binding.slim_workspace_bytes(B, H, T, d, dt),
                "xcache": lambda: binding.slim_workspace_bytes_xcache(B, H, T, d, c["d_k"], dt),
                "block": lambda: binding.slim_workspace_bytes_block(B, H, T, d, dt),
                "vanilla_block": lambda: binding.slim_workspace_bytes_block(B, H, T, d, dt)}[c["entry"]]()
        s["ws"] = torch.empty(need, dtype=torch.uint8, device="cuda")
    s["rope"] = torch.from_numpy(binding.slim_rope_table(T, c["d_k"])).cuda() if c["rope"] else None
    return s


def run(state):
    """One step: the call a serving loop makes for one layer and one new token per sequence."""
    s = state
    c = s["case"]
    B, H, T, d, dt, lens = c["B"], c["H"], c["T"], c["d"], c["dtype"], s["lens"]
    layout = binding.K_BANDED if c["banded"] else binding.K_ROWMAJOR
    if c["entry"] == "decode":
        binding.slim_decode(s["x"], s["cache"], s["W_KV"], s["out"], B, H, T, d, dtype=dt, seq_lens=lens, workspace=s["ws"],
                            rope_table=s["rope"], k_layout=layout)
        return s["out"]
    if c["entry"] == "decode_static":
        binding.slim_decode_static(s["x"], s["cache"], s["W_KV"], s["out"], B, H, T, d, dtype=dt, seq_lens=lens,
                                   rope_table=s["rope"], k_layout=layout)
        return s["out"]
    if c["entry"] == "xcache":
        binding.slim_decode_xcache(s["x"], s["cache"], s["W_K"], s["W_V"], s["out"], B, H, T, d, c["d_k"], dtype=dt,
                                   seq_lens=lens, workspace=s["ws"])
        return s["out"]
    if c["entry"] == "block":
        binding.slim_attention_block(s["x"], s["W_Q"], s["W_K"], s["W_KV"], s["W_O"], s["cache"], s["out"], B, H, T, d,
                                     dtype=dt, seq_lens=lens, workspace=s["ws"], rope_table=s["rope"], k_layout=layout)
        return {"y": s["out"], "K": s["cache"]}
    binding.vanilla_attention_block(s["x"], s["W_Q"], s["W_K"], s["W_V"], s["W_O"], s["cache"], s["vcache"], s["out"],
                                    B, H, T, d, dtype=dt, seq_lens=lens, workspace=s["ws"])
    return {"y": s["out"], "K": s["cache"], "V": s["vcache"]}


# ---- the same in 64 bits ------------------------------------------------------------------------------

def _turn(x, pos, H):
    """Rotary encoding of rows x (n, e) at positions pos, per head and adjacent pair."""
    n, e = x.shape
    d_k = e // H
    theta = 10000.0 ** (-2.0 * torch.arange(d_k // 2, device=x.device, dtype=torch.float64) / d_k)
    a = pos.to(torch.float64)[:, None] * theta
    c, s = a.cos()[:, None, :], a.sin()[:, None, :]
    p = x.view(n, H, d_k // 2, 2)
    return torch.stack((p[..., 0] * c + p[..., 1] * s, -p[..., 0] * s + p[..., 1] * c), dim=-1).reshape(n, e)


def _heads(full, H):
    """Row h of `full` (H, e) restricted to head h's columns, put together: (e,)."""
    return torch.cat([full[h].view(H, -1)[h] for h in range(H)])


def _softmax(q, K, H):
    """(H, n) weights of one query row (e,) against keys (n, e), one head at a time."""
    d_k = q.numel() // H
    s = torch.stack([K[:, h * d_k:(h + 1) * d_k] @ q[h * d_k:(h + 1) * d_k] for h in range(H)]) / math.sqrt(d_k)
    return torch.softmax(s, dim=1)


def exact(case, seed):
    c = dict(case)
    s = _inputs(c, seed)
    B, H, d, d_k = c["B"], c["H"], c["d"], c["d_k"]
    block = c["entry"] in ("block", "vanilla_block")
    f = {k: s[k].double() for k in ("x", "W_Q", "W_K", "W_V", "W_KV", "W_O") if k in s}
    q = f["x"] @ f["W_Q"] if block else f["x"]
    if block:
        knew = f["x"] @ f["W_K"]
        vnew = f["x"] @ f["W_V"] if "W_V" in f else None
    out = torch.empty((B, H * d_k), dtype=torch.float64, device="cuda")
    new_K, new_V = [], []
    for b, n in enumerate(_rows(c)):
        K = s["cache"][b]
        if c["banded"]:
            K = K.view(c["T"] // 32, H, 32, d_k).transpose(1, 2).reshape(c["T"], d)
        K = K[:n].double()
        if c["entry"] == "xcache":
            qt = torch.stack([f["W_K"][:, h * d_k:(h + 1) * d_k] @ q[b, h * d_k:(h + 1) * d_k] for h in range(H)])
            P = torch.softmax(qt @ K.T.contiguous() / math.sqrt(d_k), dim=1)
            C = P @ K
            out[b] = torch.cat([C[h] @ f["W_V"][:, h * d_k:(h + 1) * d_k] for h in range(H)])
            continue
        qb = q[b]
        if block:
            K[n - 1] = knew[b].to(_T[c["dtype"]]).double()        # the new row, as the cache stores it
            new_K.append(knew[b])
        if c["rope"]:
            pos = torch.arange(n, device="cuda")
            Kr = _turn(K, pos, H)
            if block:
                qb = _turn(qb[None], pos[-1:], H)[0]
        else:
            Kr = K
        P = _softmax(qb, Kr, H)
        if c["entry"] == "vanilla_block":
            V = s["vcache"][b, :n].double()
            V[n - 1] = vnew[b].to(_T[c["dtype"]]).double()
            new_V.append(vnew[b])
            out[b] = _heads(P @ V, H)
        else:
            C = P @ K
            out[b] = torch.cat([C[h] @ f["W_KV"][:, h * d_k:(h + 1) * d_k] for h in range(H)])
    if not block:
        return out
    y = {"y": out @ f["W_O"]}
    for name, src, rows in (("K", s["cache"], new_K), ("V", s.get("vcache"), new_V)):
        if rows:
            t = src.double()
            for b, n in enumerate(_rows(c)):
                t[b, n - 1] = rows[b]
            y[name] = t
    return y
