"""Cases on which the library's speed is measured: serving steps through its public calls.

A case is one serving step of a ragged batch: request r has ``cached`` tokens in the paged cache
and ``new`` tokens to compute.  ``kind`` says which calls a program makes for it:

  "extend"  efim_rope_append + efim_extend_attention (any lengths; cache hits and full misses)
  "decode"  efim_decode_step, one launch (at most 16 new tokens and 32 query rows per kv head)

``cache`` is the number format of the paged cache ("bf16" or "fp8": E4M3 codes), ``plan`` whether
the program keeps a plan object or hands over the batch description, ``layers`` how many attention
layers the pass runs (every layer with tensors and caches of its own).  Lengths come from the
case (``cached_lo`` .. ``new_hi``, drawn with ``lengths_seed``; the first ``misses`` requests have
nothing cached and miss_lo .. miss_hi new tokens), so that the work of a case does not depend on
the seed.  With ``reorder`` the seed permutes the requests: a pass then meets a batch that the
call before did not have, as the first layer of every step of a serving engine does; without it
the pass stands for one of the later layers of a step.

Inputs are standard normal times ``sigma``; the cached part of the cache is drawn directly (a
rotation of independent normal pairs is again normal).  Pages are shuffled over the cache with
an eighth of them unused.
"""
import math
import random

import torch

from paper_2505_21889_amd import binding as E


def _case(name, kind, batch, heads, head_dim, cached, new, **more):
    case = {
        "name": name, "kind": kind, "batch": batch, "q_heads": heads[0], "kv_heads": heads[1], "head_dim": head_dim,
        "cached_lo": cached[0], "cached_hi": cached[1], "new_lo": new[0], "new_hi": new[1],
        "misses": 0, "miss_lo": 0, "miss_hi": 0, "page": 16, "cache": "bf16", "base": 1.0e6, "interleaved": 0,
        "sigma": 1.0, "plan": False, "layers": 1, "reorder": False, "lengths_seed": 1,
    }
    case.update(more)
    return case


def listed():
    return [
        # one short completion on a small model: launches and host time
        _case("tiny_extend", "extend", 1, (4, 4), 64, (256, 256), (32, 32), base=1.0e4),
        # one user's next token through a model's layers: latency of a single launch, 32 times
        _case("user_decode", "decode", 1, (32, 8), 128, (2344, 2344), (1, 1), layers=32, base=5.0e5),
        # next token of 16 users of a multi-head model, the step kept as a plan object
        _case("decode_mha", "decode", 16, (32, 32), 128, (1024, 4096), (1, 1), plan=True, base=1.0e4),
        # next token of 32 users with long contexts and grouped heads, a new batch every step
        _case("decode_gqa", "decode", 32, (28, 4), 128, (2048, 8192), (1, 1), layers=16, reorder=True),
        # the same over an 8-bit cache
        _case("decode_gqa_fp8", "decode", 32, (28, 4), 128, (2048, 8192), (1, 1), cache="fp8"),
        # a handful of newly typed tokens per user, one launch
        _case("short_mha", "decode", 16, (32, 32), 128, (1024, 4096), (1, 16), base=1.0e4),
        # increments of an editor session behind cached prefix and suffix
        _case("extend_mha", "extend", 16, (32, 32), 128, (1024, 4096), (16, 128), base=1.0e4),
        _case("extend_gqa", "extend", 32, (28, 4), 128, (2048, 8192), (8, 64)),
        _case("extend_gqa_fp8", "extend", 32, (28, 4), 128, (2048, 8192), (8, 64), cache="fp8"),
        # a round of the 16-user infilling service, a new batch through several layers
        _case("service_round", "extend", 16, (32, 8), 128, (1216, 2960), (16, 256), layers=16, reorder=True, base=5.0e5),
        # infilling into long files
        _case("long_context", "extend", 4, (32, 8), 128, (16384, 16384), (512, 512), sigma=0.5),
        # a step that mixes cache hits with whole new prompts
        _case("mixed_step", "extend", 64, (32, 8), 128, (512, 8192), (1, 256), misses=32, miss_lo=1024, miss_hi=4096),
    ]


#: what the largest listed case costs, as an estimate that weighs bytes and operations
_MOST = 4.0e-3


def _estimate(case):
    w = work(case)
    return w["bytes"] / 4.0e12 + w["flops"] / 0.6e15


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    heads, head_dim = rng.choice([((32, 8), 128), ((28, 4), 128), ((32, 32), 128), ((4, 4), 64), ((32, 8), 64)])
    kind = rng.choice(["extend", "extend", "decode", "decode"])
    batch = _log(rng, 1, 64)
    lo = _log(rng, 256, 8192)
    cached = (lo, min(16384, int(lo * rng.uniform(1.0, 4.0))))
    more = {"page": rng.choice([16, 16, 16, 8, 32, 64, 256]), "cache": rng.choice(["bf16", "bf16", "bf16", "fp8"]),
            "base": rng.choice([1.0e4, 5.0e5, 1.0e6]), "interleaved": rng.choice([0, 0, 0, 1]),
            "sigma": rng.choice([1.0, 1.0, 0.5]), "lengths_seed": rng.randrange(1, 1 << 20)}
    if kind == "decode":
        most = min(16, 32 // (heads[0] // heads[1]))
        new = rng.choice([(1, 1), (1, 1), (1, most), (max(1, most // 2), most)])
        more["plan"] = more["cache"] == "bf16" and rng.random() < 0.3
    else:
        n = _log(rng, 4, 256)
        new = (n, min(512, int(n * rng.uniform(1.0, 8.0))))
        if rng.random() < 0.35:
            m = _log(rng, 512, 3072)
            more.update(misses=rng.randint(1, batch), miss_lo=m, miss_hi=min(4096, int(m * rng.uniform(1.0, 2.0))))
    if not more.get("plan") and rng.random() < 0.3:
        more.update(layers=rng.choice([4, 8, 16]), reorder=True)
    case = _case("", kind, batch, heads, head_dim, cached, new, **more)
    del case["name"]
    while _estimate(case) > _MOST:
        if case["layers"] > 1:
            case["layers"] //= 2
        else:
            case["batch"] = max(1, case["batch"] // 2)
            case["misses"] = min(case["misses"], case["batch"])
    return case


def _lengths(case):
    """[(cached, new)] of the requests, the same for every seed."""
    rng = random.Random(case["lengths_seed"])
    rows = []
    for r in range(case["batch"]):
        if r < case["misses"]:
            rows.append((0, rng.randint(case["miss_lo"], case["miss_hi"])))
        else:
            rows.append((rng.randint(case["cached_lo"], case["cached_hi"]), rng.randint(case["new_lo"], case["new_hi"])))
    rng.shuffle(rows)
    return rows


def work(case):
    rows = _lengths(case)
    d, hq, hkv = case["head_dim"], case["q_heads"], case["kv_heads"]
    kv = 1 if case["cache"] == "fp8" else 2
    new = sum(n for _, n in rows)
    pairs = sum(n * c + n * (n + 1) // 2 for c, n in rows)
    pages = sum(-(-(c + n) // case["page"]) for c, n in rows)
    read = sum(c for c, _ in rows) * 2 * hkv * d * kv + new * (hq + 2 * hkv) * d * 2 + 4 * pages
    written = new * hq * d * 2 + new * 2 * hkv * d * kv
    if case["kind"] == "extend":
        written += new * hq * d * 2  # the rotated queries
    return {"bytes": case["layers"] * (read + written), "flops": case["layers"] * 4 * d * hq * pairs}


def tolerance(case):
    # bf16 outputs from bf16 operands with fp32 sums: with the key ranges summed in another order
    # the listed cases differ from themselves by up to rel 3.2e-3 / max 2.3e-2 (the rounding of
    # the probabilities and of the output), and from 64-bit arithmetic by 2.3e-3 / 1.6e-2.  Caches
    # and rotated queries are compared as whole values and have to be the same.
    return {"rel": 1.0e-2, "max": 8.0e-2}


def prepare(case, seed):
    dev = "cuda"
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    rows = _lengths(case)
    if case["reorder"]:
        random.Random(seed).shuffle(rows)
    cached, new = [c for c, _ in rows], [n for _, n in rows]
    d, hq, hkv, page, layers = case["head_dim"], case["q_heads"], case["kv_heads"], case["page"], case["layers"]
    total = sum(new)

    need = [-(-(c + n) // page) for c, n in rows]
    used = sum(need)
    pages = used + max(2, used // 8)
    order = torch.randperm(pages, generator=torch.Generator().manual_seed(seed), dtype=torch.int64).to(torch.int32)
    table = torch.full((len(rows), max(need)), int(order[-1]), dtype=torch.int32)
    at = 0
    for r, k in enumerate(need):
        table[r, :k] = order[at:at + k]
        at += k
    table = table.to(dev)

    def normal(*shape):
        return torch.randn(shape, dtype=torch.bfloat16, device=dev, generator=gen).mul_(case["sigma"])

    scale = 4.0 * case["sigma"] / 448.0  # four standard deviations reach the largest code
    state = {"case": case, "table": table, "scale": scale}
    state["q"] = normal(layers, total, hq, d)
    state["k_new"], state["v_new"] = normal(layers, total, hkv, d), normal(layers, total, hkv, d)
    for name in ("k_cache", "v_cache"):
        x = normal(layers, pages, hkv, page, d)
        if case["cache"] == "fp8":
            x = torch.stack([(y.float() / scale).clamp_(-448, 448).to(torch.float8_e4m3fn).view(torch.uint8) for y in x])
        state[name] = x
    state["out"] = torch.zeros(layers, total, hq, d, dtype=torch.bfloat16, device=dev)
    state["per_layer"] = [{k: state[k][i] for k in ("q", "k_new", "v_new", "k_cache", "v_cache", "out")} for i in range(layers)]
    whole = torch.uint8 if case["cache"] == "fp8" else torch.int16
    state["outputs"] = {"out": state["out"], "k_cache": state["k_cache"].view(whole), "v_cache": state["v_cache"].view(whole)}
    if case["kind"] == "extend":
        state["outputs"]["q"] = state["q"].view(torch.int16)

    state["batch"] = batch = E.BatchDesc(cached, new, table, hq, hkv, d, page, pages)
    if case["plan"]:
        state["plan"] = E.Plan(batch, decode=case["kind"] == "decode")
        state["ws_bytes"] = E.efim_plan_workspace_bytes(state["plan"])
    elif case["kind"] == "decode":
        state["ws_bytes"] = E.efim_decode_workspace_bytes(batch)
    else:
        state["ws_bytes"] = E.efim_extend_workspace_bytes(batch)
    state["ws"] = torch.empty(max(state["ws_bytes"], 256), dtype=torch.uint8, device=dev)
    if case["plan"]:
        E.efim_plan_upload(state["plan"], state["ws"], state["ws_bytes"])
    return state


def run(state):
    case, batch, ws, nbytes, scale = state["case"], state["batch"], state["ws"], state["ws_bytes"], state["scale"]
    base, pairing, fp8 = case["base"], case["interleaved"], case["cache"] == "fp8"
    for t in state["per_layer"]:
        q, kn, vn, kc, vc, out = t["q"], t["k_new"], t["v_new"], t["k_cache"], t["v_cache"], t["out"]
        if case["kind"] == "decode":
            if case["plan"]:
                E.efim_decode_step_planned(state["plan"], state["table"], q, kn, vn, kc, vc, out, base, pairing, 0.0, ws)
            elif fp8:
                E.efim_decode_step_fp8(batch, q, kn, vn, kc, vc, out, base, pairing, 0.0, scale, scale, ws, nbytes)
            else:
                E.efim_decode_step(batch, q, kn, vn, kc, vc, out, base, pairing, 0.0, ws, nbytes)
        elif fp8:
            E.efim_rope_append_fp8(batch, q, kn, vn, kc, vc, base, pairing, scale, scale)
            E.efim_extend_attention_fp8(batch, q, kc, vc, out, 0.0, scale, scale, ws, nbytes)
        else:
            E.efim_rope_append(batch, q, kn, vn, kc, vc, base, pairing)
            E.efim_extend_attention(batch, q, kc, vc, out, 0.0, ws, nbytes)
    return state["outputs"]
