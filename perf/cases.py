"""What a program that decodes with this library has it do, as cases to be timed and checked.

Every case is a plain dict.  `kind` says what one pass is:

  step      one decode step of every layer of a stack (KVCache.step): the new token's rows join the cache
            and the attention over quantized cache, residual ring and outlier pools comes back; `rope`:
            the query and the new Key are handed over before their rotary embedding.  The pass ends by
            taking the token back (its ring row is written again by the next pass).
  decode    the attention alone, the token being in the cache already (KVCache.decode).
  verify    the attention of `tokens` drafted tokens at once (KVCache.decode_multi).
  ragged    one decode step's attention over sequences of different lengths in a paged cache, dealt by a
            launch plan (RaggedKVCache.make_plan, then .decode of every layer).
  prefill   the prompt of a whole batch quantized into an emptied cache (KVCache.prefill).
  join      the prompt of one sequence quantized into its slot of a running batch, every layer
            (RaggedKVCache.prefill_sequence).
  generate  a short prompt, then `steps` consecutive decode steps, group steps among them.

Inputs follow the recipe of the repository's synthetic workloads, drawn on the device: Keys ~ N(0,1) with
four fixed channels per kv head x20 and one token in fifty an outlier token (its whole Key row x10 or
x0.05), Values ~ N(0,1), queries ~ N(0, q_scale^2).
"""
from __future__ import annotations

import math

import torch

from paper_2505_10938_amd import cache as KC

HD = 128


def _case(name, kind, **kw):
    c = dict(kind=kind, layers=1, batch=1, q_heads=32, kv_heads=32, context=4096, bits=2, group_k=32, group_v=32,
             residual=128, budget=8, aux=32, q_scale=1.0)
    if name:
        c["name"] = name
    c.update(kw)
    return c


def listed():
    return [
        # one sequence, short context, one layer: what is left is the launch and its latencies
        _case("step_small_1k", "step", q_heads=8, kv_heads=8, context=1023, group_v=128, budget=4),
        # one sequence through the 32 layers of a multi-head model, rotation included: interactive use
        _case("step_b1_4k_rope", "step", layers=32, context=4099, rope=True),
        # a batch of 8 on a multi-head model (four of its layers, so that the caches in between are not reused)
        _case("step_b8_4k_mha", "step", layers=4, batch=8, context=4096),
        # a batch of 16 on a grouped-query model at 8k
        _case("step_b16_8k_gqa", "step", layers=4, batch=16, kv_heads=8, context=8200),
        # few long sequences, many outlier tokens
        _case("decode_b4_32k_gqa", "decode", layers=4, batch=4, kv_heads=8, context=32768, budget=32, q_scale=0.1),
        # a serving batch of 128: one layer of the stack, 2-bit and 4-bit codes
        _case("step_b128_4k_gqa", "step", batch=128, kv_heads=8, context=4100),
        _case("step_b128_4k_gqa_4bit", "step", batch=128, kv_heads=8, context=4100, bits=4),
        # four drafted tokens verified at once; groups of 128, residual 32, three outlier tokens
        _case("verify4_b8_4k_g128", "verify", layers=4, batch=8, context=4001, group_k=128, group_v=128, residual=32,
              budget=3, tokens=4),
        # continuous batching: 32 sequences of 128 .. 8192 tokens behind a page table
        _case("ragged_b32_8k_paged", "ragged", layers=4, batch=32, kv_heads=8, context=8192),
        # the prompts of a batch of 8
        _case("prefill_b8_4k", "prefill", batch=8, context=4096),
        # one long prompt joins a running batch of a grouped-query model
        _case("join_8k_gqa", "join", layers=4, batch=2, kv_heads=8, context=8191),
        # a batch of 16 from a short odd prompt on: 40 steps of two layers, one or two group steps among them
        _case("generate_b16", "generate", layers=2, batch=16, kv_heads=8, context=301, steps=40, rope=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges: other batches, head counts, context lengths (odd ones mostly),
    bit widths, group sizes, windows and budgets."""
    most = max(work(c)["bytes"] for c in listed())
    caps = {"prefill": 700e6, "join": 150e6, "generate": 2e9}
    while True:
        kind = rng.choice(["step", "step", "step", "decode", "verify", "ragged", "prefill", "join", "generate"])
        g = rng.choice([1, 1, 2, 4, 4, 8])
        group = rng.choice([32, 32, 64, 128])
        c = _case(None, kind, bits=rng.choice([2, 2, 4]), group_k=group, group_v=rng.choice([32, 32, 64, 128]),
                  residual=rng.choice([0, 32, 100, 128, 256]), budget=rng.choice([0, 3, 8, 8, 32]),
                  aux=rng.choice([16, 32, 64]), q_scale=rng.choice([0.1, 1.0]))
        c["kv_heads"] = rng.choice([4, 8, 8, 32]) if g < 8 else rng.choice([4, 8])
        c["q_heads"] = g * c["kv_heads"]
        c["batch"] = _log_int(rng, 1, 128)
        c["context"] = _log_int(rng, 300, 32768)
        c["layers"] = rng.choice([1, 2, 4])
        if kind == "step":
            c["rope"] = rng.random() < 0.3
        elif kind == "verify":
            if g == 8:
                continue
            c["tokens"] = rng.choice([t for t in (2, 4, 8) if t * g <= 8])
        elif kind == "ragged":
            c["batch"], c["context"] = max(2, min(c["batch"], 64)), min(c["context"], 8192)
            c["residual"] = max(c["residual"], 32)
            if c["batch"] * c["kv_heads"] > 256:
                continue
        elif kind == "join":
            c["batch"], c["context"] = 2, min(c["context"], 8192)
        elif kind == "generate":
            c["batch"], c["context"], c["layers"] = min(c["batch"], 32), 200 + c["context"] % 300, min(c["layers"], 2)
            c["steps"], c["rope"] = 40, rng.random() < 0.5
        elif kind == "prefill":
            c["layers"] = 1
        if c["batch"] * c["kv_heads"] > 1024 or work(c)["bytes"] > min(most, caps.get(kind, most)):
            continue
        return c


# ---- sizes --------------------------------------------------------------------------------------------------

def _n_quant(c, n):
    """Quantized tokens of a sequence of n: the oldest group goes whenever the ring holds R + G."""
    return c["group_k"] * ((n - c["residual"]) // c["group_k"]) if n >= c["residual"] + c["group_k"] else 0


def _context(c):
    """Tokens in the cache before the pass.  A single step must leave the ring short of full (the pass is
    repeated on the same state); a verified run of tokens must lie in the ring."""
    n = c["context"]
    if c["kind"] == "step" and n - _n_quant(c, n) + 1 == c["residual"] + c["group_k"]:
        n -= 1
    if c["kind"] == "verify":
        n += max(0, c["tokens"] - (n - _n_quant(c, n)))
    return n


def _lengths(c):
    """The sequences' lengths of a ragged batch: spread evenly over the logarithm, in a scattered order."""
    b, top = c["batch"], c["context"]
    low = min(128, top)
    n = [int(round(low * (top / low) ** (i / max(1, b - 1)))) for i in range(b)]
    return [n[(i * 7 + 3) % b] if math.gcd(7, b) == 1 else n[i] for i in range(b)]


def _capacity(c, n):
    G = c["group_k"]
    return G * max(1, -(-_n_quant(c, n) // G))


def _attention_bytes(c, n, tokens=1):
    """One unit, one launch: codes, steps and zeros, mask words, full-precision rows, queries, outputs."""
    nq = _n_quant(c, n)
    g = c["q_heads"] // c["kv_heads"]
    per = 2 * HD * c["bits"] / 8 + 4 * HD / c["group_k"] + 4 * HD / c["group_v"] + 1 / 8
    return nq * per + (n - nq) * 4 * HD + min(c["budget"], nq) * 4 * HD + tokens * 2 * g * HD * 2


def _prompt_bytes(c, n):
    """One unit's prompt: its rows read once, codes and meta and the rows that stay written once."""
    nq = _n_quant(c, n)
    per = 2 * HD * c["bits"] / 8 + 4 * HD / c["group_k"] + 4 * HD / c["group_v"] + 1 / 8
    return n * 4 * HD + nq * per + (n - nq) * 4 * HD


def work(case):
    c = case
    n, g, kind = _context(c), c["q_heads"] // c["kv_heads"], c["kind"]
    units = c["layers"] * c["batch"] * c["kv_heads"]
    if kind in ("step", "decode", "verify"):
        t, n = c.get("tokens", 1), n + (kind == "step")
        return {"bytes": int(units * _attention_bytes(c, n, t)), "flops": int(units * 4 * g * t * HD * n)}
    if kind == "ragged":
        per_seq = [c["layers"] * c["kv_heads"] * _attention_bytes(c, m) for m in _lengths(c)]
        return {"bytes": int(sum(per_seq)), "flops": int(c["layers"] * c["q_heads"] * 4 * HD * sum(_lengths(c)))}
    if kind in ("prefill", "join"):
        units = units if kind == "prefill" else c["layers"] * c["kv_heads"]
        return {"bytes": int(units * _prompt_bytes(c, n)), "flops": int(units * n * HD * 8)}
    total = units * _prompt_bytes(c, n)
    flops = units * n * HD * 8
    for i in range(1, c["steps"] + 1):
        total += units * _attention_bytes(c, n + i)
        flops += units * 4 * g * HD * (n + i)
        if _n_quant(c, n + i) > _n_quant(c, n + i - 1):      # a group: its rows in, its codes out
            total += units * c["group_k"] * 6 * HD
    return {"bytes": int(total), "flops": int(flops)}


# ---- inputs -------------------------------------------------------------------------------------------------

def _generator(seed, tag):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1_000_003 * seed + 7919 * tag + 17)
    return gen


def _rows(c, seed, layer, batch, n, tag=0):
    """fp16 [batch, kv_heads, n, 128] Keys and Values of one layer."""
    gen = _generator(seed, 64 * tag + layer)
    h = c["kv_heads"]
    k = torch.randn(batch, h, n, HD, generator=gen, device="cuda")
    boost = torch.ones(h, HD, device="cuda")
    boost.scatter_(1, torch.rand(h, HD, generator=_generator(seed, 5000 + layer), device="cuda").argsort(1)[:, :4], 20.0)
    pick = torch.rand(batch, h, n, 1, generator=gen, device="cuda")
    k = k * boost[:, None] * torch.where(pick < 0.01, 10.0, torch.where(pick < 0.02, 0.05, 1.0))
    v = torch.randn(batch, h, n, HD, generator=gen, device="cuda")
    return k.half(), v.half()


def _query(c, seed, shape, tag):
    return (torch.randn(shape, generator=_generator(seed, 9000 + tag), device="cuda") * c["q_scale"]).half()


def _angles(n):
    """Cosines and sines of position n (base 10000), fp32 [128]."""
    a = n * 10000.0 ** (-torch.arange(HD // 2, dtype=torch.float64) / (HD // 2))
    return torch.cat([a.cos(), a.sin()]).float().cuda()


def _config(c, max_seq):
    return KC.make_config(c["layers"], c["batch"], c["q_heads"], c["kv_heads"], max_seq, c["bits"], c["group_k"],
                          c["group_v"], c["residual"], c["budget"], c["aux"])


def prepare(case, seed):
    c = case
    n, kind, b, h = _context(c), c["kind"], c["batch"], c["kv_heads"]
    layers = range(c["layers"])
    s = {"case": c}
    if kind == "ragged":
        lengths = _lengths(c)
        G = c["group_k"]
        cfg = _config(c, _capacity(c, max(lengths)))
        groups = [_n_quant(c, m) // G for m in lengths]
        kv = KC.RaggedKVCache(cfg, n_pages=max(1, sum(groups)))
        order = torch.randperm(max(1, sum(groups)), generator=torch.Generator().manual_seed(seed)).int()
        table = torch.zeros(b, cfg.max_seq // G, dtype=torch.int32)
        at = 0
        for i, m in enumerate(groups):
            table[i, :m] = order[at:at + m]
            at += m
        kv.page_table.copy_(table)
        for i, m in enumerate(lengths):
            rows = [_rows(c, seed, l, 1, m, tag=i) for l in layers]
            kv.prefill_sequence(i, [k[0] for k, _ in rows], [v[0] for _, v in rows])
        s.update(cache=kv, q=[_query(c, seed, (b, c["q_heads"], HD), l) for l in layers])
        s["out"] = [torch.empty_like(q) for q in s["q"]]
        return s
    if kind in ("prefill", "join"):
        cfg = _config(c, _capacity(c, n))
        rows = [_rows(c, seed, l, b if kind == "prefill" else 1, n) for l in layers]
        if kind == "prefill":
            s.update(cache=KC.KVCache(cfg), rows=rows)
        else:
            s.update(cache=KC.RaggedKVCache(cfg), k=[k[0] for k, _ in rows], v=[v[0] for _, v in rows])
        return s
    steps = c.get("steps", 0)
    kv = KC.KVCache(_config(c, _capacity(c, n + steps)))
    s["cache"] = kv
    if kind == "generate":
        s["rows"] = [_rows(c, seed, l, b, n) for l in layers]
        s["new"] = [_new_token(c, seed, l, steps) for l in layers]
        s["rope"] = [_angles(n + i) for i in range(steps)] if c.get("rope") else [None] * steps
        s["out"] = [torch.empty(steps, b, c["q_heads"], HD, dtype=torch.float16, device="cuda") for _ in layers]
        return s
    for l in layers:
        kv.prefill(l, *_rows(c, seed, l, b, n))
    t = c.get("tokens", 0)
    if kind == "step":
        s["new"] = [[x[0] for x in _new_token(c, seed, l, 1)] for l in layers]
        s["rope"] = _angles(n) if c.get("rope") else None
        s["q"] = [x[2] for x in s["new"]]
    else:
        s["q"] = [_query(c, seed, (b, t, c["q_heads"], HD) if t else (b, c["q_heads"], HD), l) for l in layers]
    s["out"] = [torch.empty_like(q) for q in s["q"]]
    return s


def _new_token(c, seed, layer, steps):
    """(Keys, Values, queries) of the tokens decoded in the pass, each a list over the steps."""
    k, v = _rows(c, seed, layer, c["batch"], steps, tag=100)
    q = _query(c, seed, (steps, c["batch"], c["q_heads"], HD), 200 + layer)
    return ([k[:, :, i].contiguous() for i in range(steps)], [v[:, :, i].contiguous() for i in range(steps)],
            [q[i] for i in range(steps)])


# ---- one pass -----------------------------------------------------------------------------------------------

def _cache_contents(kv):
    names = ("k_codes", "k_meta", "v_codes", "v_meta", "mask", "k_res", "v_res", "pool_k", "pool_v", "pool_idx",
             "pool_score", "pool_count", "aux_count", "frozen")
    return {n: getattr(kv, n) for n in names}


def _empty(kv):
    """The cache as for new sequences."""
    for t in (kv.pool_count, kv.aux_count, kv.frozen):
        t.zero_()
    for l in range(kv.cfg.layers):
        kv.n_quant[l] = kv.n_res[l] = kv.res_start[l] = 0


def run(state):
    s = state
    c, kv = s["case"], s["cache"]
    kind, layers = c["kind"], range(c["layers"])
    if kind == "step":
        for l in layers:
            k, v, q = s["new"][l]
            kv.step(l, k, v, q, s["out"][l], rope=s["rope"])
            kv.n_res[l] -= 1                                   # the token is taken back
        return {"out": s["out"], "k_res": kv.k_res, "v_res": kv.v_res}
    if kind == "decode":
        for l in layers:
            kv.decode(l, s["q"][l], s["out"][l])
        return {"out": s["out"]}
    if kind == "verify":
        for l in layers:
            kv.decode_multi(l, s["q"][l], s["out"][l])
        return {"out": s["out"]}
    if kind == "ragged":
        kv.make_plan()
        for l in layers:
            kv.decode(l, s["q"][l], s["out"][l], planned=True)
        return {"out": s["out"]}
    if kind == "prefill":
        _empty(kv)
        kv.prefill(0, *s["rows"][0])
        return {**_cache_contents(kv), "selected": kv.prefill_selected}
    if kind == "join":
        kv.prefill_sequence(1, s["k"], s["v"])
        return {**_cache_contents(kv), "seq_state": kv.seq_state}
    _empty(kv)
    for l in layers:
        kv.prefill(l, *s["rows"][l])
    for i in range(c["steps"]):
        for l in layers:
            k, v, q = (x[i] for x in s["new"][l])
            kv.step(l, k, v, q, s["out"][l][i], rope=s["rope"][i])
    return {"out": s["out"], **_cache_contents(kv)}


# ---- what the results should be -----------------------------------------------------------------------------

def tolerance(case):
    """Prompts: every byte.  Attention: outputs are fp16; against 64 bits they are off by 1.5e-4 .. 2.1e-4 (2-norm,
    measured on every kind), which is that rounding, and by one ulp, 9.8e-4, at most where two results straddle
    a rounding boundary.  Four times that.  Cache contents that a case
    also returns (rings, codes, pools) are whole values and equal."""
    if case["kind"] in ("prefill", "join"):
        return "exact"
    return {"rel": 1e-3, "max": 4e-3}


def _selected(c, k):
    """Which tokens of [units, n, 128] Keys (n a multiple of the group) win a place in the outlier pool when
    their group is quantized: the pool keeps the N smallest L1 norms so far, ties to the lower index, and the
    first group whose evictions do not fit in the auxiliary pool ends it."""
    U, n, _ = k.shape
    G, N, A = c["group_k"], c["budget"], c["aux"]
    flags = torch.zeros(U, n, dtype=torch.bool, device=k.device)
    if N == 0 or n == 0:
        return flags
    score = torch.cat([x.double().abs().sum(2) for x in k.split(8)])
    pool = torch.empty(U, 0, dtype=torch.float64, device=k.device)     # ascending by (score, index)
    live = torch.ones(U, dtype=torch.bool, device=k.device)
    aux = torch.zeros(U, dtype=torch.long, device=k.device)
    for i in range(n // G):
        group = score[:, i * G:(i + 1) * G]
        P = pool.shape[1]
        both, order = torch.cat([pool, group], 1).sort(dim=1, stable=True)   # older first among equals
        keep = min(N, P + G)
        new = order[:, :keep] >= P
        evicted = P - (keep - new.sum(1))
        live = live & (aux + evicted <= A)
        aux = aux + evicted * live
        mine = torch.zeros(U, P + G, dtype=torch.bool, device=k.device).scatter_(1, order[:, :keep], True)
        flags[:, i * G:(i + 1) * G] = mine[:, P:] & live[:, None]
        # (a unit that has stopped keeps a pool that no longer matters)
        pool = both[:, :keep]
    return flags


def _round_trip(x, dim, bits):
    """Eq. 2 along `dim`: fp16 step and zero, nearest code, back as zero + code * step in 64 bits."""
    x = x.float()
    lo, hi = x.amin(dim, keepdim=True) + 0.0, x.amax(dim, keepdim=True)
    levels = 2 ** bits - 1
    inv = torch.tensor(1.0 / levels, dtype=torch.float32, device=x.device)
    step = ((hi - lo) * inv).half().float()
    t = x - lo
    code = torch.zeros_like(t)
    for j in range(levels):
        code += (t >= (j + 0.5) * step) & (step > 0)
    return lo.double() + code.double() * step.double()


def _effective(c, k, v):
    """[units, n, 128] rows (n a multiple of the group) as the attention sees them, 64 bits: an outlier token
    as it is, any other as its codes say, the codes taken with outlier rows replaced by the group's mean."""
    U, n, _ = k.shape
    if n == 0:
        return k.double(), v.double()
    G = c["group_k"]
    flags = _selected(c, k)
    m = flags.view(U, n // G, G, 1)
    out = []
    for x, value in ((k, False), (v, True)):
        xg = x.view(U, n // G, G, HD)
        parts = []
        for a, mask in zip(xg.split(4), m.split(4)):
            mean = a.double().mean(2, keepdim=True).float().half()
            y = torch.where(mask, mean, a)
            if value:
                w = c["group_v"]
                back = _round_trip(y.view(*y.shape[:3], HD // w, w), 4, c["bits"]).view(y.shape)
            else:
                back = _round_trip(y, 2, c["bits"])
            parts.append(torch.where(mask, a.double(), back).view(a.shape[0], n, HD))
        out.append(torch.cat(parts))
    return out


def _rotate(x, angles):
    """The rotation of the first half's channels against the second's, rounded once per product and sum."""
    cos, sin = angles[:HD // 2], angles[HD // 2:]
    lo, hi = x[..., :HD // 2].float(), x[..., HD // 2:].float()
    return torch.cat([lo * cos - hi * sin, hi * cos + lo * sin], -1).half()


def _attend(q, k, v):
    """q [units, rows, 128], k and v [units, n, 128]: softmax attention in 64 bits."""
    out = []
    for a, b, w in zip(q.split(8), k.split(8), v.split(8)):
        scores = torch.matmul(b.double(), a.double().transpose(1, 2).contiguous()) / math.sqrt(HD)   # [u, n, rows]
        p = torch.softmax(scores, dim=1).transpose(1, 2).contiguous()
        out.append(torch.matmul(p, w.double()))
    return torch.cat(out)


def _unit_outputs(c, q, k, v, nq, tokens=1):
    """Attention over [units, n, 128] rows of which the first nq are quantized; q [units, tokens * g, 128]."""
    parts = []
    step = max(1, int(2e8 // (k.shape[1] * HD)) // 8 * 8)
    for a, kk, vv in zip(q.split(step), k.split(step), v.split(step)):
        ek, ev = _effective(c, kk[:, :nq].contiguous(), vv[:, :nq].contiguous())
        ek, ev = torch.cat([ek, kk[:, nq:].double()], 1), torch.cat([ev, vv[:, nq:].double()], 1)
        g, n = a.shape[1] // tokens, ek.shape[1]
        parts.append(torch.cat([_attend(a[:, i * g:(i + 1) * g], ek[:, :n - (tokens - 1 - i)],
                                        ev[:, :n - (tokens - 1 - i)]) for i in range(tokens)], 1))
    return torch.cat(parts)


def exact(case, seed):
    c = case
    kind, b, h, g = c["kind"], c["batch"], c["kv_heads"], c["q_heads"] // c["kv_heads"]
    n, U = _context(c), c["batch"] * c["kv_heads"]
    if kind in ("prefill", "join") or work(c)["flops"] > 1.2e10:
        return None
    none = dict.fromkeys(("k_res", "v_res"))
    outs = []
    for l in range(c["layers"]):
        if kind == "ragged":
            q = _query(c, seed, (b, c["q_heads"], HD), l)
            rows = []
            for i, m in enumerate(_lengths(c)):
                k, v = _rows(c, seed, l, 1, m, tag=i)
                rows.append(_unit_outputs(c, q[i].view(h, g, HD), k[0], v[0], _n_quant(c, m)).view(1, h * g, HD))
            outs.append(torch.cat(rows))
            continue
        k, v = (x.view(U, n, HD) for x in _rows(c, seed, l, b, n))
        if kind == "step":
            kn, vn, qn = (x[0] for x in _new_token(c, seed, l, 1))
            if c.get("rope"):
                kn, qn = _rotate(kn, _angles(n)), _rotate(qn, _angles(n))
            k, v = torch.cat([k, kn.view(U, 1, HD)], 1), torch.cat([v, vn.view(U, 1, HD)], 1)
            outs.append(_unit_outputs(c, qn.view(U, g, HD), k, v, _n_quant(c, n)).view(b, h * g, HD))
        elif kind == "generate":
            per_step = []
            kn, vn, qn = _new_token(c, seed, l, c["steps"])
            for i in range(c["steps"]):
                ki, qi = kn[i], qn[i]
                if c.get("rope"):
                    ki, qi = _rotate(ki, _angles(n + i)), _rotate(qi, _angles(n + i))
                k, v = torch.cat([k, ki.view(U, 1, HD)], 1), torch.cat([v, vn[i].view(U, 1, HD)], 1)
                per_step.append(_unit_outputs(c, qi.view(U, g, HD), k, v, _n_quant(c, n + i + 1)).view(b, h * g, HD))
            outs.append(torch.stack(per_step))
        else:
            t = c.get("tokens", 1)
            q = _query(c, seed, (b, t, c["q_heads"], HD) if "tokens" in c else (b, c["q_heads"], HD), l)
            rows = q.view(b, t, h, g, HD).transpose(1, 2).reshape(U, t * g, HD)
            o = _unit_outputs(c, rows, k, v, _n_quant(c, n), t)
            outs.append(o.view(b, h, t, g, HD).transpose(1, 2).reshape(q.shape))
    if kind == "step":
        return {"out": outs, **none}
    if kind == "generate":
        names = ("k_codes", "k_meta", "v_codes", "v_meta", "mask", "k_res", "v_res", "pool_k", "pool_v", "pool_idx",
                 "pool_score", "pool_count", "aux_count", "frozen")
        return {"out": outs, **dict.fromkeys(names)}
    return {"out": outs}
