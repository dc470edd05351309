"""The measured work of the library: what a user of it has it do, through the
public entry points of ``paper_2406_14909_amd.moa``.

Kinds of cases:

``prompt``     a prompt enters: ``moa_prefill`` of all its tokens, then
               ``moa_kv_append`` of them into the per-head static caches.
``step``       one decode step of a batch whose sequences share one position:
               ``moa_kv_append`` of one token, then ``moa_decode``.
``ragged``     one decode step of a serving batch, every sequence at its own
               position: ``moa_kv_append_ragged``, then ``moa_decode_ragged``.
``influence``  one layer's profile in the rule search: ``moa_influence``.
``rules``      the loss of every candidate rule for every head:
               ``moa_rule_loss``.

Inputs are N(0, 1); queries share a component with the first four keys, as the
sink tokens of a trained model draw weight from every query.  The rule of each
KV head is drawn from the spans that the method searches and scaled so that
the mean window is ``mean`` of the length.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2406_14909_amd import moa, search

DEVICE = "cuda"
SINK_TOKENS = 4            # keys that every query leans to
SINK_SHIFT = 0.5           # shared component per dimension


def _prompt(name, b, hq, hkv, d, n, dtype="bf16", sink=64, mean=0.5, flags=0, rules=1):
    return dict(name=name, kind="prompt", b=b, hq=hq, hkv=hkv, d=d, n=n, dtype=dtype, sink=sink, mean=mean,
                flags=flags, rules=rules)


def _step(name, kind, b, hq, hkv, d, n, pos, dtype="bf16", sink=64, mean=0.5, rules=1):
    return dict(name=name, kind=kind, b=b, hq=hq, hkv=hkv, d=d, n=n, pos=pos, dtype=dtype, sink=sink, mean=mean,
                flags=0, rules=rules)


def listed():
    return [
        # a short chat prompt: few work-groups, launches and latency count
        _prompt("prompt-512", 1, 32, 32, 128, 512),
        # one prompt of a 4k model (32 heads of 128)
        _prompt("prompt-4k", 1, 32, 32, 128, 4096, rules=2),
        # one long prompt of a grouped-query model (4 query heads per KV head)
        _prompt("prompt-gqa4-16k", 1, 32, 8, 128, 16384, rules=3),
        # a full prefill batch; keys and values exceed every cache of the chip
        _prompt("prompt-b8-8k", 8, 32, 32, 128, 8192, rules=4),
        # odd length, small heads, the 64-token block band and spans that include the sinks
        _prompt("prompt-odd-d64-block", 3, 32, 8, 64, 1999, flags=3, rules=5),
        # a reference run in fp32, as a model is checked against its 16-bit form
        _prompt("prompt-f32-d64", 1, 8, 8, 64, 1501, dtype="f32", sink=4, rules=6),
        # interactive decode: one sequence
        _step("step-b1-4k", "step", 1, 32, 32, 128, 4096, 4100, rules=2),
        # batch decode of a grouped-query model at long context
        _step("step-gqa4-b16-16k", "step", 16, 32, 8, 128, 16384, 16400, rules=3),
        # the large decode batch: 2 GB of caches read per token
        _step("step-b32-8k", "step", 32, 32, 32, 128, 8192, 8200, rules=4),
        # continuous batching: 8 query heads per KV head, every sequence somewhere else, one slot idle
        _step("ragged-gqa8-b23-8k", "ragged", 23, 64, 8, 128, 8192, 9001, mean=0.25, rules=7),
        # rule search: the profile of one layer over two calibration items
        dict(name="influence-gqa4-4k", kind="influence", b=2, hq=32, hkv=8, d=128, n=4096),
        # rule search: 32 layers of 32 heads, 54 candidate rules
        dict(name="rules-1024h-8k", kind="rules", heads=1024, n=8192, sink=64, flags=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# (query heads, KV heads, head dim): the layers of the configurations, and smaller ones of each group size
_LAYERS = [(32, 32, 128), (32, 8, 128), (64, 8, 128), (16, 8, 128), (32, 8, 64), (16, 16, 64)]


def _cost(case):
    w = work(case)
    rate = 5e13 if case.get("dtype") == "f32" and case["kind"] == "prompt" else 8e14
    return max(w["bytes"] / 5e12, w["flops"] / rate)


def draw(rng):
    most = max(_cost(c) for c in listed())
    while True:
        kind = rng.choice(["prompt", "prompt", "prompt", "step", "step", "ragged", "influence", "rules"])
        hq, hkv, d = rng.choice(_LAYERS)
        rules = rng.randrange(100, 1000)
        if kind == "rules":
            case = dict(kind=kind, heads=_log_int(rng, 32, 1024), n=_log_int(rng, 1000, 16000),
                        sink=rng.choice([4, 64]), flags=rng.choice([0, 2, 3]))
        elif kind == "influence":
            case = dict(kind=kind, b=rng.randint(1, 4), hq=hq, hkv=hkv, d=d, n=_log_int(rng, 500, 8192))
        elif kind == "prompt":
            dtype = "f32" if rng.random() < 0.15 else "bf16"
            n = _log_int(rng, 200, 2048) if dtype == "f32" else _log_int(rng, 200, 16384)
            case = _prompt("", _log_int(rng, 1, 8), hq, hkv, d, n, dtype, rng.choice([4, 64]),
                           rng.choice([0.25, 0.5]), rng.choice([0, 0, 1, 2, 3]), rules)
            del case["name"]
        else:
            n = _log_int(rng, 500, 16384)
            case = _step("", kind, _log_int(rng, 1, 32), hq, hkv, d, n, n + rng.randint(0, 300), "bf16",
                         rng.choice([4, 64]), rng.choice([0.25, 0.5]), rules)
            del case["name"]
        if _cost(case) <= most:
            return case


# ---------------------------------------------------------------------------
# Rules and windows (plain arithmetic, as the method defines them).
# ---------------------------------------------------------------------------
def _rules(case):
    """(alpha, beta) per KV head with a mean window of case["mean"] of n."""
    rng = np.random.default_rng(case["rules"])
    n, hkv = float(case["n"]), case["hkv"]
    alpha = rng.choice([256.0, 512.0, 1024.0, 2048.0], size=hkv)
    beta = rng.choice([0.0, 0.25, 0.5, 0.75], size=hkv)
    lo, hi = 0.0, 1024.0
    for _ in range(100):
        f = 0.5 * (lo + hi)
        if np.minimum(n, f * (alpha + beta * n)).mean() < case["mean"] * n:
            lo = f
        else:
            hi = f
    return hi * alpha, hi * beta


def _window(alpha, beta, n, sink, flags):
    x = float(alpha) + float(beta) * float(n)
    if flags & moa.MOA_SPAN_INCLUDES_SINKS:
        return max(int(math.floor(min(max(x, 0.0), float(n)))) - sink, 1)
    return int(math.floor(min(max(x, 1.0), float(n))))


def _windows(case):
    return [_window(a, b, case["n"], case["sink"], case["flags"]) for a, b in zip(*_rules(case))]


def _first_visible(i, w, flags):
    """First key of the band of rows i (tensor or int), clipped at 0 by the caller."""
    if flags & moa.MOA_BLOCK_BAND:
        return (i // 64 - -(-w // 64) + 1) * 64
    return i - w + 1


def _pairs(n, w, sink, flags):
    """Visible (query, key) pairs of one head over a prompt of n tokens."""
    i = np.arange(n, dtype=np.int64)
    start = np.maximum(_first_visible(i, w, flags), 0)
    return int((i + 1 - start + np.minimum(start, sink)).sum())


def _positions(case):
    """Per-sequence positions of a ragged batch: spread from short to the longest, one slot idle."""
    b, top = case["b"], case["pos"]
    pos = [max(1, (top * (2 * k + 1)) // (2 * b)) for k in range(b)]
    pos[0] = top
    if b > 2:
        pos[b // 2] = -1
    return pos


def work(case):
    kind = case["kind"]
    if kind == "rules":
        nb = -(-case["n"] // 64)
        r = 54
        return {"bytes": case["heads"] * (nb * (nb + 1) // 2 * 4 + r * 8), "flops": case["heads"] * nb * (nb + 1)}
    b, hq, hkv, d, n = (case[k] for k in ("b", "hq", "hkv", "d", "n"))
    if kind == "influence":
        nb = -(-n // 64)
        causal = n * (n + 1) // 2
        # scores and gradients of every causal pair: two products, formed once
        return {"bytes": 2 * b * n * (2 * hq + 2 * hkv) * d + 4 * hq * nb * nb, "flops": 4 * d * causal * hq * b}
    es = 4 if case["dtype"] == "f32" else 2
    ws, s, group = _windows(case), case["sink"], hq // hkv
    if kind == "prompt":
        pairs = sum(_pairs(n, w, s, case["flags"]) for w in ws)
        kept = sum(min(n, s + w) for w in ws)
        return {"bytes": b * (es * d * (2 * n * hq + 2 * n * hkv + 2 * kept) + 4 * kept),
                "flops": 4 * d * pairs * group * b}
    positions = _positions(case) if kind == "ragged" else [case["pos"]] * b
    keys = sum(min(p + 1, s + w) for p in positions if p >= 0 for w in ws)
    return {"bytes": es * d * 2 * (keys + b * (hq + 2 * hkv)), "flops": 4 * d * keys * group}


# ---------------------------------------------------------------------------
# Inputs (plain torch, from the seed alone).
# ---------------------------------------------------------------------------
def _dtype(case):
    return torch.float32 if case.get("dtype") == "f32" else torch.bfloat16


def _randn(gen, shape, dtype):
    """N(0, 1) in fp32, rounded to dtype; drawn in slices of the first axis, so that no large fp32 copy is held."""
    out = torch.empty(shape, dtype=dtype, device=DEVICE)
    for i in range(shape[0]):
        out[i] = torch.randn(shape[1:], generator=gen, device=DEVICE)
    return out


def _inputs(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed))
    kind = case["kind"]
    if kind == "rules":
        nb = -(-case["n"] // 64)
        e = torch.randn((case["heads"], nb, nb), generator=gen, device=DEVICE) * 0.5 + 1.0
        return {"ebar": torch.tril(e) * 1e-5}
    b, hq, hkv, d, n = (case[k] for k in ("b", "hq", "hkv", "d", "n"))
    dt = _dtype(case)
    if kind in ("prompt", "influence"):
        q = _randn(gen, (b, n, hq, d), dt).add_(SINK_SHIFT)
        k = _randn(gen, (b, n, hkv, d), dt)
        k[:, :SINK_TOKENS] += SINK_SHIFT
        v = _randn(gen, (b, n, hkv, d), dt)
        x = {"q": q, "k": k, "v": v}
        if kind == "influence":
            x["dout"] = _randn(gen, (b, n, hq, d), dt)
        return x
    # caches as they stand before the step: sequence i has seen positions 0 .. pos_i - 1
    ws, s = _windows(case), case["sink"]
    rows = sum(s + w for w in ws)
    positions = _positions(case) if kind == "ragged" else [case["pos"]] * b
    kc = _randn(gen, (b, rows, d), dt)
    vc = _randn(gen, (b, rows, d), dt)
    pc = torch.empty((b, rows), dtype=torch.int32, device=DEVICE)
    done = {}
    for i, p in enumerate(positions):
        if p not in done:
            done[p] = torch.cat([_slot_positions(max(p, 0), w, s) for w in ws])
        pc[i] = done[p]
    r0 = 0
    for w in ws:
        kc[:, r0:r0 + SINK_TOKENS] += SINK_SHIFT
        r0 += s + w
    return {"k_cache": kc, "v_cache": vc, "pos_cache": pc,
            "q": _randn(gen, (b, hq, d), dt).add_(SINK_SHIFT),
            "k_new": _randn(gen, (b, 1, hkv, d), dt), "v_new": _randn(gen, (b, 1, hkv, d), dt),
            "positions": torch.tensor(positions, dtype=torch.int32, device=DEVICE)}


def _slot_positions(seen, w, s):
    """int32 [s + w]: the position that each slot of one head holds after `seen` tokens, -1 where empty."""
    pos = torch.full((s + w,), -1, dtype=torch.int32, device=DEVICE)
    k = min(seen, s)
    pos[:k] = torch.arange(k, dtype=torch.int32, device=DEVICE)
    p = torch.arange(max(s, seen - w), max(s, seen), device=DEVICE)
    pos[s + (p - s) % w] = p.to(torch.int32)
    return pos


def prepare(case, seed):
    x = _inputs(case, seed)
    kind = case["kind"]
    if kind == "rules":
        alpha, beta = search.candidate_rules()
        return dict(x, kind=kind, n=case["n"], sink=case["sink"], flags=case["flags"], alpha=alpha, beta=beta)
    if kind == "influence":
        return dict(x, kind=kind)
    alpha, beta = _rules(case)
    plan = moa.moa_plan(case["hq"], case["hkv"], case["d"], case["sink"], case["n"], case["dtype"], alpha, beta,
                        flags=case["flags"])
    state = dict(x, kind=kind, plan=plan)
    if kind == "prompt":
        state["k_cache"], state["v_cache"], state["pos_cache"] = moa.new_cache(plan, case["b"], DEVICE)
    else:
        state["pos"] = case["pos"]
        state["workspace"] = moa.new_workspace(plan, case["b"], DEVICE)
        state["o"] = torch.zeros_like(x["q"])
    return state


def run(state):
    kind = state["kind"]
    if kind == "rules":
        dl, density = moa.moa_rule_loss(state["ebar"], state["n"], state["sink"], state["alpha"], state["beta"],
                                        state["flags"])
        return {"dl": dl, "density": density}
    if kind == "influence":
        return {"ebar": moa.moa_influence(state["q"], state["k"], state["v"], state["dout"])}
    plan, kc, vc, pc = state["plan"], state["k_cache"], state["v_cache"], state["pos_cache"]
    if kind == "prompt":
        o = moa.moa_prefill(plan, state["q"], state["k"], state["v"])
        moa.moa_kv_append(plan, kc, vc, pc, state["k"], state["v"], 0)
    elif kind == "step":
        moa.moa_kv_append(plan, kc, vc, pc, state["k_new"], state["v_new"], state["pos"])
        o = moa.moa_decode(plan, state["q"], kc, vc, state["pos"], state["workspace"], o=state["o"])
    else:
        moa.moa_kv_append_ragged(plan, kc, vc, pc, state["k_new"], state["v_new"], state["positions"])
        o = moa.moa_decode_ragged(plan, state["q"], kc, vc, state["positions"], state["workspace"], o=state["o"])
    return {"o": o, "k_cache": kc, "v_cache": vc, "pos_cache": pc}


def tolerance(case):
    kind = case["kind"]
    if kind == "rules":
        return {"rel": 1e-12}          # fp64 sums
    if kind == "influence":
        return {"rel": 1e-5}           # fp32 sums over exact products of bf16 values
    if case["dtype"] == "f32":
        return {"rel": 4e-6}           # fp32 throughout
    return {"rel": 1e-2}               # bf16 outputs and weights, fp32 sums


# ---------------------------------------------------------------------------
# The same in 64 bits, without the library.
# ---------------------------------------------------------------------------
def _exact_attention(q, k, v, w, s, flags, group):
    """q [n, G, D], k, v [n, D] of one KV head -> [n, G, D] fp64, in blocks of rows."""
    n, d = k.shape
    k, v = k.double(), v.double()
    kt = k.t().contiguous()
    j = torch.arange(n, device=k.device)
    out = torch.empty((n, group, d), dtype=torch.float64, device=k.device)
    for r0 in range(0, n, 2048):
        i = torch.arange(r0, min(n, r0 + 2048), device=k.device)
        seen = (j[None, :] <= i[:, None]) & ((j[None, :] < s) | (j[None, :] >= _first_visible(i, w, flags)[:, None]))
        for g in range(group):
            sc = (q[r0:r0 + 2048, g].double() @ kt) / math.sqrt(d)
            p = torch.softmax(sc.masked_fill_(~seen, -math.inf), dim=1)
            out[r0:r0 + 2048, g] = p @ v
    return out


def exact(case, seed):
    kind = case["kind"]
    x = _inputs(case, seed)
    if kind == "rules":
        alpha, beta = search.candidate_rules()
        n, s, flags = case["n"], case["sink"], case["flags"]
        nb = -(-n // 64)
        i = torch.arange(n, device=DEVICE)
        blk = torch.nn.functional.one_hot(i // 64, nb).double()      # [n, nb]
        dl, dens = [], []
        for a, b in zip(alpha, beta):
            w = _window(a, b, n, s, flags)
            # hidden pairs per block: row i hides keys s .. first - 1 (none after the row itself)
            end = torch.minimum(_first_visible(i, w, flags).clamp(min=0), i + 1)
            start = torch.arange(nb, device=DEVICE) * 64
            count = (end[:, None].minimum(start + 64) - start.clamp(min=s)).clamp(min=0).double()   # [n, nb]
            pairs = blk.t().contiguous() @ count                      # [nb, nb]
            dl.append(x["ebar"].double().reshape(case["heads"], -1) @ pairs.reshape(-1))
            dens.append(min(s + w, n) / n)
        return {"dl": torch.stack(dl, 1), "density": torch.tensor(dens, dtype=torch.float64, device=DEVICE)}
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    group = hq // hkv
    if kind == "influence":
        b, n = case["b"], case["n"]
        nb = -(-n // 64)
        i = torch.arange(n, device=DEVICE)
        hidden = i[None, :] > i[:, None]
        sums = torch.zeros((hq, nb, nb), dtype=torch.float64, device=DEVICE)
        for m in range(b):
            for h in range(hq):
                g = h // group
                kt = x["k"][m, :, g].double().t().contiguous()
                vt = x["v"][m, :, g].double().t().contiguous()
                a = torch.softmax((x["q"][m, :, h].double() @ kt / math.sqrt(d)).masked_fill_(hidden, -math.inf), 1)
                grad = x["dout"][m, :, h].double() @ vt
                e = -a / (1 - a) * (grad - (grad * a).sum(1, keepdim=True))
                e[0] = 0                                              # a row's only weight leaves nothing
                e = torch.nn.functional.pad(e.masked_fill_(hidden, 0.0), (0, nb * 64 - n, 0, nb * 64 - n))
                sums[h] += e.reshape(nb, 64, nb, 64).sum((1, 3))
        size = torch.full((nb,), 64.0, dtype=torch.float64, device=DEVICE)
        size[-1] = n - 64 * (nb - 1)
        return {"ebar": sums / (b * size[:, None] * size[None, :])}
    ws, s = _windows(case), case["sink"]
    offs = np.concatenate([[0], np.cumsum([s + w for w in ws])]).tolist()
    if kind == "prompt":
        b, n = case["b"], case["n"]
        o = torch.empty((b, n, hq, d), dtype=torch.float64, device=DEVICE)
        kc = torch.zeros((b, offs[-1], d), dtype=torch.float64, device=DEVICE)
        vc = torch.zeros_like(kc)
        pc = torch.empty((b, offs[-1]), dtype=torch.int32, device=DEVICE)
        for g, w in enumerate(ws):
            rows = slice(offs[g], offs[g + 1])
            pos = _slot_positions(n, w, s)
            pc[:, rows] = pos
            full = pos >= 0
            for m in range(b):
                o[m, :, g * group:(g + 1) * group] = _exact_attention(
                    x["q"][m, :, g * group:(g + 1) * group], x["k"][m, :, g], x["v"][m, :, g], w, s, case["flags"],
                    group)
                kc[m, rows][full] = x["k"][m, pos[full].long(), g].double()
                vc[m, rows][full] = x["v"][m, pos[full].long(), g].double()
        return {"o": o, "k_cache": kc, "v_cache": vc, "pos_cache": pc}
    positions = x["positions"].tolist()
    o = torch.zeros(x["q"].shape, dtype=torch.float64, device=DEVICE)
    kc, vc, pc = x["k_cache"], x["v_cache"], x["pos_cache"]
    for m, p in enumerate(positions):
        if p < 0:
            continue
        for g, w in enumerate(ws):
            slot = offs[g] + (p if p < s else s + (p - s) % w)
            kc[m, slot], vc[m, slot], pc[m, slot] = x["k_new"][m, 0, g], x["v_new"][m, 0, g], p
            rows = slice(offs[g], offs[g] + min(p + 1, s + w))
            heads = slice(g * group, (g + 1) * group)
            a = torch.softmax(x["q"][m, heads].double() @ kc[m, rows].double().t().contiguous() / math.sqrt(d), 1)
            o[m, heads] = a @ vc[m, rows].double()
    return {"o": o, "k_cache": None, "v_cache": None, "pos_cache": pc}
