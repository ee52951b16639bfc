"""Timed cases of the A2SF hot path, through the public calls of paper_2407_20485_amd.binding.

A case is one call as a serving loop makes it: a prompt (`prefill`), a further chunk of a prompt
(`chunk`) or a generation step (`decode`) over `heads` K/V heads with `group` query heads each.
Fields of a case besides these:
    d, dtype         head dimension, "bf16" or "f32"
    n                rows of the prompt / of the chunk (prefill, chunk)
    select, recent   the budget; a decode or chunk cache starts full
    alpha            forgetting factor
    outputs          prefill: attention outputs wanted (False: scores and cache only)
    stable           decode: slots stay in ascending position

The inputs are drawn so that attention is concentrated on part of the tokens, as a trained model's
is (Section 2.2 of the paper): token 0 and as many others as the score-selected part of the budget
holds stand out in a prompt, and a full cache holds tokens whose weights spread over many orders of
magnitude.  Which token is kept or evicted then follows from the inputs and not from the rounding
of two nearly equal scores.
"""
import math

import torch

from paper_2407_20485_amd import binding as B

_DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
_STEPS = 4  # different tokens a decode loop feeds in turn


def _case(kind, heads, d, dtype, select, recent, alpha, n=0, group=1, outputs=True, stable=False, name=None):
    c = dict(kind=kind, heads=heads, group=group, d=d, dtype=dtype, n=n, select=select, recent=recent,
             alpha=alpha, outputs=outputs, stable=stable)
    return dict(c, name=name) if name else c


def listed():
    return [
        # one layer of a 7B model (32 heads), batch 1, cache ratio 0.2 of a 1024-token prompt: the
        # smallest call of a chat loop, where launch latency counts
        _case("decode", 32, 128, "bf16", 102, 102, 0.3, name="decode_layer"),
        # the same kind of step with a long context: 0.1 of 32768 tokens kept per head
        _case("decode", 32, 128, "bf16", 1638, 1638, 0.9, name="decode_long"),
        # all layers and sequences of a batch in one call: 32 layers x 16 sequences x 32 heads
        _case("decode", 16384, 128, "bf16", 100, 100, 0.5, name="decode_batched"),
        # a 13B layer (40 heads, batch 8), slots kept in ascending position
        _case("decode", 320, 128, "bf16", 204, 205, 0.1, stable=True, name="decode_stable"),
        # a grouped-query layer (8 K/V heads, 4 query heads each), batch 8, budget 1024
        _case("decode", 64, 128, "bf16", 512, 512, 0.5, group=4, name="decode_grouped"),
        # prompt of one layer of a 7B model, batch 1: a short call of four dependent kernels
        _case("prefill", 32, 128, "bf16", 102, 102, 0.3, n=1024, name="prefill_layer"),
        # prompts of many sequences and layers at once: 32 layers x 4 sequences x 32 heads
        _case("prefill", 4096, 128, "bf16", 100, 100, 0.5, n=2048, name="prefill_batched"),
        # one long document, 32 heads, slow forgetting (over a thousand rows carry weight)
        _case("prefill", 32, 128, "bf16", 1638, 1638, 0.9, n=32768, name="prefill_long"),
        # prompts as they come, of no round length, in a grouped-query layer: 8 K/V heads x 4, batch 4
        _case("prefill", 32, 128, "bf16", 150, 150, 0.5, n=3001, group=4, name="prefill_grouped_ragged"),
        # a small model's layer (12 heads of 64), batch 8, plain accumulation (alpha = 1), odd length
        _case("prefill", 96, 64, "bf16", 177, 178, 1.0, n=1777, name="prefill_d64_ragged"),
        # fp32 inputs: a layer of 32 heads
        _case("prefill", 32, 128, "f32", 100, 100, 0.3, n=1000, name="prefill_f32"),
        # a further chunk of 512 tokens of 16 long prompts (one layer of 32 heads), behind a full cache
        _case("chunk", 512, 128, "bf16", 256, 256, 0.5, n=512, name="chunk_layer"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above: 1 to 16384 heads, budgets of 16 to 4096 tokens, prompts of 40 to
    16384 tokens, chunks of 16 to 1024, both head sizes, fp32 and bf16, 1 to 8 query heads per K/V head."""
    kind = rng.choice(["decode", "decode", "prefill", "prefill", "prefill", "chunk"])
    d = rng.choice([64, 128, 128])
    dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
    e = 2 if dtype == "bf16" else 4
    group = rng.choice([1, 1, 1, rng.choice([2, 4, 8]), rng.randint(2, 8)])
    alpha = rng.choice([0.1, 0.3, 0.5, 0.9, 1.0])
    share = rng.choice([0.5, 0.5, rng.uniform(0.2, 0.8), 0.0])  # of the budget: the most recent tokens

    def split(budget):
        recent = int(share * budget)
        return budget - recent, recent

    if kind == "decode":
        budget = _log_int(rng, 16, min(4096, 16000 // group))
        heads = _log_int(rng, 1, max(1, min(16384, int(1.6e9 / (2 * budget * d * e)))))
        return _case(kind, heads, d, dtype, *split(budget), alpha, group=group, stable=rng.random() < 0.25)
    if kind == "prefill":
        n = _log_int(rng, 40, 16384 if dtype == "bf16" else 1500)
        budget = max(8, int(n * rng.uniform(0.05, 0.3)))
        most = (1e12 if dtype == "bf16" else 1e10) / (2.0 * d * n * n * group)
        heads = _log_int(rng, 1, max(1, min(4096, int(most))))
        return _case(kind, heads, d, dtype, *split(budget), alpha, n=n, group=group, outputs=rng.random() < 0.85)
    m = _log_int(rng, 16, 1024)
    budget = _log_int(rng, 32, 1024)
    most = (4e11 if dtype == "bf16" else 1e10) / (4.0 * d * m * (budget + m) * group)
    heads = _log_int(rng, 1, max(1, min(2048, int(most))))
    return _case(kind, heads, d, dtype, *split(budget), alpha, n=m, group=group)


def _unit(heads, d, gen):
    u = torch.randn(heads, d, generator=gen, device="cuda")
    return u / u.norm(dim=1, keepdim=True) * d ** 0.25  # two rows with this component: their logit is 1 higher


def _normal(shape, dtype, gen):
    return torch.randn(shape, dtype=dtype, generator=gen, device="cuda")


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    G, r, d, n, dt = case["heads"], case["group"], case["d"], case["n"], _DTYPES[case["dtype"]]
    budget = case["select"] + case["recent"]
    u = _unit(G, d, gen)
    code = B.dtype_code(dt)
    s = {"case": case}
    qshape = (G, n, d) if r == 1 else (G, r, n, d)
    lift = u[:, None, :] if r == 1 else u[:, None, None, :]
    if case["kind"] == "prefill":
        q, k, v = _normal(qshape, dt, gen), _normal((G, n, d), dt, gen), _normal((G, n, d), dt, gen)
        q += lift.to(dt)
        # the tokens that stand out: token 0 and others of the part that is not protected as recent
        last = min(n - case["recent"], max(case["select"], 3 * n // 4))
        pick = torch.rand(G, last, generator=gen, device="cuda")
        pick[:, 0] = 2.0
        which = pick.topk(max(1, case["select"]), dim=1).indices
        m = torch.zeros(G, n, device="cuda")
        m.scatter_(1, which, 8.0 + 3.0 * torch.rand(which.shape, generator=gen, device="cuda"))
        k += m[:, :, None].to(dt) * u[:, None, :].to(dt)
        cache = B.Cache(G, budget + 1, d, dt)
        ws = B.a2sf_workspace_bytes(G * r, n, cache.capacity, d, code, case["select"], case["recent"])
        s.update(q=q, k=k, v=v, o=torch.empty_like(q) if case["outputs"] else None)
    else:
        # a cache as earlier steps leave it: full, positions ascending, weights far apart
        extra = n if case["kind"] == "chunk" else 1
        cache = B.Cache(G, budget + extra, d, dt)
        m = 4.0 * torch.log(torch.rand(G, budget, generator=gen, device="cuda").clamp_min(1e-4))
        cache.k[:, :budget] = _normal((G, budget, d), dt, gen)
        cache.k[:, :budget] += m[:, :, None].to(dt) * u[:, None, :].to(dt)
        cache.v[:, :budget] = _normal((G, budget, d), dt, gen)
        w = torch.exp(m + torch.randn(G, budget, generator=gen, device="cuda"))
        cache.scores[:, :budget] = w / w.sum(dim=1, keepdim=True)
        gaps = 1 + (torch.rand(G, budget, generator=gen, device="cuda") * 5).int()
        gaps[:, budget - case["recent"]:] = 1
        cache.pos[:, :budget] = torch.cumsum(gaps, 1).int()
        top = 6 * budget  # the next position: the newest ones are consecutive up to it
        cache.pos[:, :budget] += top - cache.pos[:, budget - 1: budget].clone() - 1
        cache.len.fill_(budget)
        if case["kind"] == "chunk":
            q, k, v = _normal(qshape, dt, gen), _normal((G, n, d), dt, gen), _normal((G, n, d), dt, gen)
            q += lift.to(dt)
            m = 4.0 * torch.log(torch.rand(G, n, generator=gen, device="cuda").clamp_min(1e-4))
            k += m[:, :, None].to(dt) * u[:, None, :].to(dt)
            ws = B.a2sf_workspace_bytes(G * r, n, cache.capacity, d, code, case["select"], case["recent"])
            s.update(q=q, k=k, v=v, o=torch.empty_like(q), t=top)
        else:
            shape = (G, d) if r == 1 else (G, r, d)
            q = [_normal(shape, dt, gen) + (u if r == 1 else u[:, None, :]).to(dt) for _ in range(_STEPS)]
            k, v = ([_normal((G, d), dt, gen) for _ in range(_STEPS)] for _ in range(2))
            ws = B.a2sf_workspace_bytes(G * r, 0, cache.capacity, d, code, case["select"], case["recent"])
            if r > 1:
                ws += 4 * G * r * 64 * (d + 2)
            s.update(q=q, k=k, v=v, o=torch.empty(shape, dtype=dt, device="cuda"), t=top, step=0)
    s.update(cache=cache, workspace=torch.empty(ws, dtype=torch.uint8, device="cuda"))
    return s


def run(s):
    c, cache = s["case"], s["cache"]
    kept = (c["select"], c["recent"])
    if c["kind"] == "prefill":
        if c["group"] == 1:
            B.a2sf_prefill(s["q"], s["k"], s["v"], c["n"], c["alpha"], *kept, cache, o=s["o"], workspace=s["workspace"])
        else:
            B.a2sf_prefill_gqa(s["q"], s["k"], s["v"], c["n"], c["group"], c["alpha"], *kept, cache, o=s["o"],
                               workspace=s["workspace"])
    elif c["kind"] == "chunk":
        if c["group"] == 1:
            B.a2sf_prefill_chunk(s["q"], s["k"], s["v"], c["n"], s["t"], c["alpha"], *kept, cache, o=s["o"],
                                 workspace=s["workspace"])
        else:
            B.a2sf_prefill_chunk_gqa(s["q"], s["k"], s["v"], c["n"], s["t"], c["group"], c["alpha"], *kept, cache,
                                     o=s["o"], workspace=s["workspace"])
        s["t"] += c["n"]
    else:
        i = s["step"] % _STEPS
        mode = B.A2SF_EVICT_STABLE if c["stable"] else B.A2SF_EVICT_FAST
        if c["group"] == 1:
            B.a2sf_decode_step(s["q"][i], s["k"][i], s["v"][i], s["t"], cache, c["alpha"], *kept, s["o"], mode=mode,
                               workspace=s["workspace"])
        else:
            B.a2sf_decode_step_gqa(s["q"][i], s["k"][i], s["v"][i], s["t"], cache, c["group"], c["alpha"], *kept,
                                   s["o"], mode=mode, workspace=s["workspace"])
        s["t"] += 1
        s["step"] += 1
    # slots past a head's length are undefined: the cache is returned up to the budget, where it is full
    full = kept[0] + kept[1]
    return {"o": s["o"], "k": cache.k[:, :full], "v": cache.v[:, :full], "scores": cache.scores[:, :full],
            "pos": cache.pos[:, :full], "len": cache.len}


def work(case):
    G, r, d, n, budget = case["heads"], case["group"], case["d"], case["n"], case["select"] + case["recent"]
    e = 2 if case["dtype"] == "bf16" else 4
    row = d * e
    if case["kind"] == "prefill":
        kept = G * budget * (2 * row + 8)
        if case["outputs"]:  # Q, K, V in, O out, the kept rows written; logits and outputs of the lower triangle
            return {"bytes": G * n * row * (2 * r + 2) + kept, "flops": G * r * 2.0 * d * n * (n + 1)}
        # without outputs only the rows whose weight alpha^(n-1-i) is not zero in fp32 count
        rows = n if case["alpha"] >= 1.0 else min(n, int(160.0 / -math.log2(case["alpha"])) + 1)
        pairs = rows * (2 * n - rows + 1) / 2.0
        return {"bytes": G * row * (r * rows + n + budget) + kept, "flops": G * r * 2.0 * d * pairs}
    if case["kind"] == "chunk":
        # the chunk in, its outputs out, the cached keys, values and scores read, at most a cache of new rows written
        moved = min(n, budget)
        pairs = n * budget + n * (n + 1) / 2.0
        return {"bytes": G * (n * row * (2 * r + 2) + budget * (2 * row + 16) + moved * 2 * row),
                "flops": G * r * 4.0 * d * pairs}
    # cached rows, scores and positions read, scores written; the token's rows in, one row in its slot, outputs out
    length = budget + 1
    move = 2 * case["recent"] * 2 * row if case["stable"] else 0  # the newest rows move one slot down
    return {"bytes": G * (2 * length * row + 12 * length + (2 * r + 4) * row + move), "flops": G * r * 4.0 * d * length}


def tolerance(case):
    # bf16: outputs are rounded to 8 bits, and a prompt's probabilities are before they meet V; the same sums in
    # another order move a value by one such step.  fp32: sums of up to thousands of terms.  Whole values
    # (positions, lengths): a tie that is decided by the last bit may go either way.
    if case["dtype"] == "f32":
        return {"rel": 2e-5, "max": 1e-3, "differ": 1e-3}
    return {"rel": 1e-2, "max": 1e-1, "differ": 1e-3}


def _attend(q, k, v, off, alpha, want_o):
    """64-bit rows of m queries [h, r, m, d] against keys [h, off + m, d]: outputs and the summed scores."""
    h, r, m, d = q.shape
    nk = off + m
    kt, v = k.double().transpose(1, 2).contiguous(), v.double()
    o = torch.empty(h, r, m, d, dtype=torch.float64, device="cuda") if want_o else None
    scores = torch.zeros(h, nk, dtype=torch.float64, device="cuda")
    step = max(1, int(6e7 / nk / h))
    for i0 in range(0, m, step):
        rows = torch.arange(i0, min(m, i0 + step), device="cuda")
        seen = off + int(rows[-1]) + 1
        hidden = torch.arange(seen, device="cuda")[None, :] > off + rows[:, None]
        w = torch.where(rows == m - 1, 1.0, torch.pow(torch.tensor(alpha, dtype=torch.float64, device="cuda"),
                                                      (m - 1 - rows).double()))
        for j in range(r):
            p = torch.bmm(q[:, j, i0: i0 + len(rows)].double() / math.sqrt(d), kt[:, :, :seen].contiguous())
            p.masked_fill_(hidden, -math.inf)
            p = torch.softmax(p, dim=2)
            if want_o:
                o[:, j, i0: i0 + len(rows)] = torch.bmm(p, v[:, :seen].contiguous())
            scores[:, :seen] += torch.einsum("i,hij->hj", w, p)
    return o, scores


def _keep(scores, select, recent):
    """Slots that stay, ascending: the `recent` last and the `select` best of the others, ties to the lower slot."""
    L = scores.shape[1]
    rank = scores.clone()
    if recent:
        rank[:, L - recent:] = math.inf
    order = torch.sort(rank, dim=1, descending=True, stable=True).indices
    return torch.sort(order[:, : select + recent], dim=1).values


def exact(case, seed):
    s = prepare(case, seed)
    c, cache = case, s["cache"]
    G, r, d, n, kept = c["heads"], c["group"], c["d"], c["n"], (c["select"], c["recent"])
    budget = sum(kept)
    alpha = B.ctypes.c_float(c["alpha"]).value  # as the call gets it
    new = {"k": [], "v": [], "scores": [], "pos": [], "o": []}
    nk = n if c["kind"] == "prefill" else budget + max(1, n)
    heads = max(1, min(G, int(6e7 / nk / d)))
    for g0 in range(0, G, heads):
        g = slice(g0, min(G, g0 + heads))
        q = (s["q"][0] if c["kind"] == "decode" else s["q"])[g].reshape(-1, r, max(1, n), d)
        k, v = ((s[x][0][:, None] if c["kind"] == "decode" else s[x])[g] for x in "kv")
        pos = torch.arange(k.shape[1], device="cuda", dtype=torch.int32).expand(k.shape[:2])
        if c["kind"] != "prefill":
            k, v = torch.cat([cache.k[g, :budget], k], 1), torch.cat([cache.v[g, :budget], v], 1)
            pos = torch.cat([cache.pos[g, :budget], pos + s["t"]], 1)
        off = 0 if c["kind"] == "prefill" else budget
        o, scores = _attend(q, k, v, off, alpha, s["o"] is not None)
        if off:
            scores[:, :off] += alpha ** max(1, n) * cache.scores[g, :off].double()
        keep = _keep(scores, *kept)
        if c["kind"] == "decode" and not c["stable"]:
            # one token goes: the new one takes its slot
            out = torch.ones_like(scores, dtype=torch.bool).scatter_(1, keep, False).int().argmax(1)
            keep = torch.arange(budget, device="cuda").repeat(len(out), 1)
            keep[keep == out[:, None]] = budget
        rows = keep[:, :, None].expand(-1, -1, d)
        new["k"].append(k.gather(1, rows))
        new["v"].append(v.gather(1, rows))
        new["scores"].append(scores.gather(1, keep))
        new["pos"].append(pos.gather(1, keep))
        new["o"].append(o.reshape(-1, *s["o"].shape[1:]) if o is not None else None)
    got = {x: torch.cat(y) if y[0] is not None else None for x, y in new.items()}
    got["k"], got["v"] = got["k"].double(), got["v"].double()
    return {**got, "len": torch.full((G,), budget, dtype=torch.int32)}
