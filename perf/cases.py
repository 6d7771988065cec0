"""The workloads this framework's speed is judged by: what a serving loop has it do, called the way such a loop calls it.

A case is a dict of plain values.  `listed()` names twelve of them, `draw()` gives more from the same ranges; `prepare`
makes what the loop holds before the call (a pool filled with its conversations, the step's Q/K/V rows), `run` is one
pass through the public entry points, `exact` the same results in float64 from plain torch.

Kinds of case:
  conversation  one session from its first token: acquire, ingest the system prompt, then `turns` turns of `delta` new
                tokens, each appended and attended in one call, release
  step          one scheduler iteration over a batch of sessions: `chunks` sessions take a prefill chunk of `chunk`
                tokens, the others delta_lo..delta_hi new tokens; "fused" appends and attends in one call, "staged"
                attends the candidate rows first and then appends the accepted ones; the slots are rewound afterwards
  verify        greedy verification of speculated rows: argmax over the vocabulary, accepted count and next token
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2605_26289_amd import DevicePool
from paper_2605_26289_amd import binding as dk

PRODUCTION = {"hq": 32, "hkv": 8, "d": 128, "dtype": "bf16"}


def _step(name, **kw):
    case = {"kind": "step", **PRODUCTION, "slots": 1, "prefix": 0, "n_lo": 0, "n_hi": 0, "delta_lo": 1, "delta_hi": 1,
            "chunks": 0, "chunk": 0, "mode": "fused", "lse": False, "lens": 1}
    case.update(kw)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # A single fp32 session (validation runs and small models kept in fp32): 200 cached tokens, one 150-token turn.
        {"name": "conversation_f32", "kind": "conversation", "hq": 4, "hkv": 1, "d": 64, "dtype": "f32", "system": 200,
         "turns": 1, "delta": 150},
        # The five-turn agent conversation: a 200-token system prompt, then 150 tokens per turn (950 at the end).
        {"name": "conversation_5turn", "kind": "conversation", **PRODUCTION, "system": 200, "turns": 5, "delta": 150},
        # One user decoding token by token: the smallest call, latency and launches.
        _step("decode_one", n_lo=3000, n_hi=3000),
        # Speculative verification: 64 sessions, 1 + 8 candidate rows each, long prefixes; the accepted rows are appended.
        _step("spec_verify", slots=64, n_lo=4096, n_hi=16384, delta_lo=9, delta_hi=9, mode="staged", lens=5),
        # Plain decoding of a full house of sessions of very different age.
        _step("decode_many", slots=256, n_lo=512, n_hi=8192, lens=6),
        # Short tool results and user messages: a few dozen new tokens per session on a shared preamble.
        _step("tool_results", slots=16, prefix=2048, n_lo=1024, n_hi=8192, delta_lo=24, delta_hi=64, lens=7),
        # Interleaved agents on one shared 2048-token preamble, 64 to 512 new tokens each.
        _step("multi_agent", slots=16, prefix=2048, n_lo=1024, n_hi=8192, delta_lo=64, delta_hi=512, lens=8),
        # The last turn of a 35-turn coding conversation: one long session, one long turn; its log-sum-exp is kept.
        _step("coding_turn", n_lo=24581, n_hi=24581, delta_lo=761, delta_hi=761, lse=True),
        # A mixed scheduler iteration: four prefill chunks of 1024 among 60 decoding or verifying sessions.
        _step("mixed", slots=64, n_lo=4096, n_hi=16384, delta_lo=1, delta_hi=9, chunks=4, chunk=1024, lens=9),
        # Models with 64-wide heads: two prefill chunks among decoding and verifying sessions.
        _step("heads64", d=64, slots=16, n_lo=512, n_hi=4096, delta_lo=1, delta_hi=9, chunks=2, chunk=256, lens=10),
        # Three query heads to a KV head (a group that is no power of two): a few agents' turns.
        _step("group3", hq=24, slots=4, n_lo=256, n_hi=2048, delta_lo=1, delta_hi=200, lens=11),
        # The step after speculative verification: 64 sessions of nine rows over a 128 256-entry vocabulary.
        {"name": "verify_greedy", "kind": "verify", "seqs": 64, "rows": 9, "vocab": 128256, "dtype": "bf16"},
    ]


def _between(rng, lo, hi):
    """A whole number spread evenly over the logarithm of [lo, hi]."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def draw(rng):
    kind = rng.choice(["conversation", "decode", "decode", "short", "turns", "turns", "mixed", "heads", "f32", "verify"])
    lens = rng.randrange(1, 1 << 30)
    if kind == "conversation":
        return {"kind": "conversation", **PRODUCTION, "system": _between(rng, 20, 1000), "turns": rng.randint(1, 6),
                "delta": _between(rng, 30, 400)}
    if kind == "verify":
        return {"kind": "verify", "seqs": _between(rng, 1, 64), "rows": rng.randint(1, 9),
                "vocab": 8 * rng.randint(4000, 16032), "dtype": rng.choice(["bf16", "f32"])}
    if kind == "f32":
        hq, hkv, d = rng.choice([(4, 1, 64), (4, 2, 64), (8, 2, 64), (8, 2, 128), (16, 4, 128)])
        n = _between(rng, 30, 2000)
        return _step(None, hq=hq, hkv=hkv, d=d, dtype="f32", slots=rng.randint(1, 4), n_lo=max(1, n // 2), n_hi=n,
                     delta_lo=1, delta_hi=_between(rng, 1, 300), mode=rng.choice(["fused", "staged"]),
                     lse=rng.random() < 0.5, lens=lens)
    if kind == "heads":  # head widths and groups other than the usual one
        hq, hkv, d = rng.choice([(32, 8, 64), (16, 4, 64), (14, 2, 64), (24, 8, 128), (12, 2, 128), (28, 4, 128),
                                 (8, 8, 128), (16, 2, 128), (16, 1, 128)])
        n = _between(rng, 64, 8192)
        return _step(None, hq=hq, hkv=hkv, d=d, slots=_between(rng, 1, 16), n_lo=max(1, n // 4), n_hi=n, delta_lo=1,
                     delta_hi=_between(rng, 1, 256), mode=rng.choice(["fused", "staged"]), lse=rng.random() < 0.3,
                     lens=lens)
    if kind == "decode":  # decoding and verification
        slots = _between(rng, 1, 256)
        n = _between(rng, 200, min(32000, 1000000 // slots))
        k = rng.choice([0, 0, rng.randint(1, 8), rng.randint(9, 20)])
        return _step(None, slots=slots, n_lo=max(1, n // 4), n_hi=n, delta_lo=1 if rng.random() < 0.3 else 1 + k,
                     delta_hi=1 + k, mode=rng.choice(["fused", "staged"]), lens=lens)
    if kind == "short":
        return _step(None, slots=_between(rng, 1, 24), prefix=rng.choice([0, _between(rng, 100, 2048)]), n_lo=200,
                     n_hi=_between(rng, 400, 8192), delta_lo=10, delta_hi=rng.randint(20, 100), lens=lens)
    if kind == "turns":
        slots = _between(rng, 1, 12)
        return _step(None, slots=slots, prefix=rng.choice([0, _between(rng, 100, 2048)]), n_lo=1,
                     n_hi=_between(rng, 200, 30000 // slots), delta_lo=16, delta_hi=_between(rng, 64, 3000 // slots),
                     lse=rng.random() < 0.3, lens=lens)
    return _step(None, slots=_between(rng, 4, 48), n_lo=1000, n_hi=_between(rng, 2000, 12000), delta_lo=1,
                 delta_hi=rng.randint(1, 12), chunks=rng.randint(1, 3), chunk=_between(rng, 128, 1024), lens=lens)


# ---- inputs ----------------------------------------------------------------------------------------------------------
def _torch_type(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _lengths(case):
    """(private history, new tokens, accepted tokens) of every session of a step, by the case alone."""
    rng = random.Random(case["lens"])
    hist = [rng.randint(case["n_lo"], case["n_hi"]) for _ in range(case["slots"])]
    delta = [rng.randint(case["delta_lo"], case["delta_hi"]) for _ in range(case["slots"])]
    for i in rng.sample(range(case["slots"]), min(case["chunks"], case["slots"])):
        delta[i] = case["chunk"]
    # acceptance is all or nearly nothing
    accept = [d if rng.random() < 0.6 else min(d, 1 + rng.randint(0, 2)) for d in delta]
    return hist, delta, accept


def _tensors(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    dt = _torch_type(case)

    def normal(*shape):
        return torch.randn(shape, generator=gen, device="cuda", dtype=dt)

    hkv, hq, d = case["hkv"], case["hq"], case["d"]
    if case["kind"] == "conversation":
        total = case["system"] + case["turns"] * case["delta"]
        new = case["turns"] * case["delta"]
        return {"k": normal(total, hkv, d), "v": normal(total, hkv, d), "q": normal(new, hq, d)}
    hist, delta, _ = _lengths(case)
    return {"pk": normal(case["prefix"], hkv, d), "pv": normal(case["prefix"], hkv, d), "k": normal(sum(hist), hkv, d),
            "v": normal(sum(hist), hkv, d), "q": normal(sum(delta), hq, d), "k_new": normal(sum(delta), hkv, d),
            "v_new": normal(sum(delta), hkv, d)}


def _offsets(lengths):
    return np.concatenate([[0], np.cumsum(lengths)]).astype(np.int32)


def _logits(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))
    rows = case["seqs"] * case["rows"]
    logits = torch.randn((rows, case["vocab"]), generator=gen, device="cuda", dtype=_torch_type(case))
    tokens = torch.randint(0, case["vocab"], (rows,), generator=gen, device="cuda", dtype=torch.int32)
    right = torch.rand((rows,), generator=gen, device="cuda") < 0.8  # drafts the model agrees with
    if rows > 1:
        best = logits[:-1].float().argmax(dim=1).to(torch.int32)
        tokens[1:] = torch.where(right[1:], best, tokens[1:])
    return logits, tokens


def prepare(case, seed):
    if case["kind"] == "verify":
        logits, tokens = _logits(case, seed)
        rows, seqs = case["seqs"] * case["rows"], case["seqs"]
        code = dk.BF16 if case["dtype"] == "bf16" else dk.F32
        cu = torch.arange(0, rows + 1, case["rows"], dtype=torch.int32, device="cuda")
        ints = [torch.empty(n, dtype=torch.int32, device="cuda") for n in (seqs, seqs, rows)]
        ws = torch.empty(dk.verify_workspace_bytes(rows, case["vocab"], code), dtype=torch.uint8, device="cuda")
        return {"case": case, "logits": logits, "tokens": tokens, "cu": cu, "keep": ints[0], "next": ints[1],
                "argmax": ints[2], "ws": ws, "code": code}
    t = _tensors(case, seed)
    scale = 1.0 / math.sqrt(case["d"])
    if case["kind"] == "conversation":
        total = case["system"] + case["turns"] * case["delta"]
        pool = DevicePool(2, total + 1024, case["hq"], case["hkv"], case["d"], case["dtype"])
        s, step = case["system"], case["delta"]
        turns = []
        for i in range(case["turns"]):
            a, b = i * step, (i + 1) * step
            turns.append((t["q"][a:b], t["k"][s + a:s + b], t["v"][s + a:s + b]))
        return {"case": case, "pool": pool, "scale": scale, "system": (t["k"][:s], t["v"][:s]), "turns": turns,
                "cu_system": np.array([0, s], dtype=np.int32), "cu": np.array([0, step], dtype=np.int32)}
    hist, delta, accept = _lengths(case)
    n_slots, prefix = case["slots"], case["prefix"]
    pool = DevicePool(n_slots, prefix + sum(hist) + sum(delta) + 512 * (n_slots + 2), case["hq"], case["hkv"], case["d"],
                      case["dtype"])
    slots = np.array([pool.acquire() for _ in range(n_slots)], dtype=np.int32)
    if prefix:
        pool.append(slots[:1], [0, prefix], t["pk"], t["pv"])
        for s in slots[1:]:
            pool.alias(int(slots[0]), int(s), prefix)
    pool.append(slots, _offsets(hist), t["k"], t["v"])
    return {"case": case, "pool": pool, "scale": scale, "slots": slots, "cu": _offsets(delta), "q": t["q"],
            "k_new": t["k_new"], "v_new": t["v_new"], "n_past": np.array([prefix + h for h in hist], dtype=np.int64),
            "accept": np.array(accept, dtype=np.int32), "out": torch.empty_like(t["q"]),
            "lse": torch.empty((sum(delta), case["hq"]), dtype=torch.float32, device="cuda") if case["lse"] else None}


def run(state):
    case = state["case"]
    if case["kind"] == "verify":
        dk.verify_greedy(case["seqs"], case["seqs"] * case["rows"], state["cu"], state["logits"], state["code"],
                         case["vocab"], case["vocab"], state["tokens"], state["keep"], state["next"], state["ws"],
                         argmax_out=state["argmax"])
        return {"keep": state["keep"], "next": state["next"], "argmax": state["argmax"]}
    pool = state["pool"]
    if case["kind"] == "conversation":
        slot = pool.acquire()
        k, v = state["system"]
        pool.append([slot], state["cu_system"], k, v)
        outs = [pool.append_attend([slot], state["cu"], q, k, v, state["scale"]) for q, k, v in state["turns"]]
        pool.release(slot)
        return outs
    slots, cu = state["slots"], state["cu"]
    if case["mode"] == "fused":
        pool.append_attend(slots, cu, state["q"], state["k_new"], state["v_new"], state["scale"], out=state["out"],
                           lse=state["lse"])
    else:
        pool.attend(slots, cu, state["q"], state["scale"], state["k_new"], state["v_new"], out=state["out"],
                    lse=state["lse"])
        pool.append(slots, cu, state["k_new"], state["v_new"], state["accept"])
    pool.trim_batch(slots, state["n_past"])
    return [state["out"]] if state["lse"] is None else [state["out"], state["lse"]]


# ---- what a pass cannot do without -----------------------------------------------------------------------------------
def work(case):
    e = 2 if case["dtype"] == "bf16" else 4
    if case["kind"] == "verify":
        rows = case["seqs"] * case["rows"]
        return {"bytes": rows * case["vocab"] * e, "flops": 0}
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    row = hkv * d * e * 2  # K and V of one token

    def turn(n, new):  # the products of `new` tokens on n cached ones
        return 4 * hq * d * (new * n + new * (new + 1) // 2)

    if case["kind"] == "conversation":
        s, new = case["system"], case["delta"]
        nbytes, flops = 2 * s * row, 0
        for i in range(case["turns"]):
            n = s + i * new
            nbytes += n * row + 2 * new * row + 2 * new * hq * d * e
            flops += turn(n, new)
        return {"bytes": nbytes, "flops": flops}
    hist, delta, accept = _lengths(case)
    written = sum(accept if case["mode"] == "staged" else delta)
    nbytes = (case["prefix"] + sum(hist) + sum(delta) + written) * row + 2 * sum(delta) * hq * d * e
    if case["lse"]:
        nbytes += sum(delta) * hq * 4
    return {"bytes": nbytes, "flops": sum(turn(case["prefix"] + h, new) for h, new in zip(hist, delta))}


def tolerance(case):
    if case["kind"] == "verify":
        return "exact"
    if case["dtype"] == "f32":
        return {"rel": 1e-5, "max": 1e-3}
    return {"rel": 1e-2, "max": 1e-1}


# ---- the same results in 64 bits -------------------------------------------------------------------------------------
def _attend64(q, k, v, n):
    """Causal attention of q's rows (token i at position n + i) over k, v: (out, natural log-sum-exp)."""
    new, hq, d = q.shape
    hkv = k.shape[1]
    group = hq // hkv
    out = torch.empty((new, hq, d), dtype=torch.float64, device=q.device)
    lse = torch.empty((new, hq), dtype=torch.float64, device=q.device)
    pos = torch.arange(n + new, device=q.device)
    for g in range(hkv):
        kg, vg = k[:, g].double(), v[:, g].double()
        for lo in range(0, new, 512):
            hi = min(new, lo + 512)
            rows = q[lo:hi, g * group:(g + 1) * group].double().reshape(-1, d)
            s = (rows @ kg.t()) / math.sqrt(d)
            limit = torch.arange(n + lo, n + hi, device=q.device).repeat_interleave(group)
            s.masked_fill_(pos[None, :] > limit[:, None], float("-inf"))
            lse[lo:hi, g * group:(g + 1) * group] = torch.logsumexp(s, dim=1).reshape(hi - lo, group)
            out[lo:hi, g * group:(g + 1) * group] = (torch.softmax(s, dim=1) @ vg).reshape(hi - lo, group, d)
    return out, lse


def exact(case, seed):
    if case["kind"] == "verify":
        return None
    t = _tensors(case, seed)
    if case["kind"] == "conversation":
        outs, n = [], case["system"]
        for i in range(case["turns"]):
            end = n + case["delta"]
            q = t["q"][i * case["delta"]:(i + 1) * case["delta"]]
            outs.append(_attend64(q, t["k"][:end], t["v"][:end], n)[0])
            n = end
        return outs
    hist, delta, _ = _lengths(case)
    ch, cu = _offsets(hist), _offsets(delta)
    outs, lses = [], []
    for b in range(case["slots"]):
        new = slice(int(cu[b]), int(cu[b + 1]))
        old = slice(int(ch[b]), int(ch[b + 1]))
        k = torch.cat([t["pk"], t["k"][old], t["k_new"][new]])
        v = torch.cat([t["pv"], t["v"][old], t["v_new"][new]])
        out, lse = _attend64(t["q"][new], k, v, case["prefix"] + hist[b])
        outs.append(out)
        lses.append(lse)
    return [torch.cat(outs), torch.cat(lses)] if case["lse"] else [torch.cat(outs)]
