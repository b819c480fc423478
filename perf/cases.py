"""What this library is timed on: its calls as a serving program makes them, over the sizes such programs have.

A case is a dict of plain values.  Four kinds:
  decode    one decode step (sqa_decode_step): all layers in one call, or one call per layer as inside a model
  scores    the prompt's accumulated attention (sqa_prefill_scores, with or without given softmax normalisers)
  probe     the cosine probe of the hidden states, alone, per sequence, or inside the residual add
  compress  the prompt's K / V gathered into the layer caches (sqa_prefill_compress_layers), for a whole batch
            or for one sequence that joins a running one

Shapes are those of workloads.py and bench.py (4 to 80 layers, 1 to 8 query heads per KV head, head size 64 or
128, prompts up to 8192, batches up to 224, budgets of 15 to 30 per cent of the prompt with a share p of 0.3 to
0.4 for the unimportant layers) and, in draw(), sizes in between and odd ones.
"""
from __future__ import annotations

import math

import torch

from paper_2404_04793_amd import binding as sqa

N_SINK = 4
STEPS = 8              # different decode inputs that a state holds and takes in turn
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
BLOCK = 16


# ---- the cases ------------------------------------------------------------------------------------------------
def _decode(name, L, n_high, b_low, b_high, tokens, B, Hq, Hkv, D, dtype, policy, order="evict_then_attend",
            layout="dense", ragged=False, calls="together"):
    return dict(name=name, kind="decode", layers=L, n_high=n_high, b_low=b_low, b_high=b_high, tokens=tokens, batch=B,
                heads=Hq, kv_heads=Hkv, dim=D, dtype=dtype, policy=policy, order=order, layout=layout, ragged=ragged,
                calls=calls)


def _scores(name, B, Hq, Hkv, P, D, dtype, ragged=False, lse=False):
    return dict(name=name, kind="scores", batch=B, heads=Hq, kv_heads=Hkv, prompt=P, dim=D, dtype=dtype, ragged=ragged,
                lse=lse)


def _probe(name, form, L, tokens, hidden, dtype, n_seq=1):
    return dict(name=name, kind="probe", form=form, layers=L, tokens=tokens, hidden=hidden, dtype=dtype, n_seq=n_seq)


def _compress(name, L, n_high, b_low, b_high, P, B, Hkv, D, dtype, policy, layout="dense", ragged=False, join=False):
    return dict(name=name, kind="compress", layers=L, n_high=n_high, b_low=b_low, b_high=b_high, prompt=P, batch=B,
                kv_heads=Hkv, dim=D, dtype=dtype, policy=policy, layout=layout, ragged=ragged, join=join)


def listed():
    return [
        # the smallest call there is: four fp32 layers, one sequence (launch and call latency)
        _decode("decode_tiny_f32", 4, 2, 17, 85, 272, 1, 4, 4, 64, "f32", "h2o"),
        # a decode step inside a model: one call per layer, batch 8 of the Llama-2-7B shape
        _decode("decode_7b_layer_by_layer", 32, 4, 143, 2271, 2304, 8, 32, 32, 128, "bf16", "h2o", calls="layers"),
        # the same layers when their inputs are known up front: the benchmark's headline step
        _decode("decode_7b_h2o", 32, 4, 143, 2271, 2304, 8, 32, 32, 128, "bf16", "h2o"),
        # grouped queries, sinks + window (the Mistral-7B configuration)
        _decode("decode_mistral_streaming", 32, 17, 368, 1987, 4608, 32, 32, 8, 128, "bf16", "streaming"),
        # 8 query heads per KV head, 80 layers, sliding window (the Llama-2-70B configuration)
        _decode("decode_70b_sliding", 80, 20, 491, 3439, 8448, 16, 64, 8, 128, "bf16", "sliding"),
        # many short units: batch 224 (the throughput configuration); the largest decode step
        _decode("decode_stress_h2o", 32, 4, 35, 571, 1536, 224, 32, 32, 128, "bf16", "h2o"),
        # a serving loop: sequences of different length and budget, rows in blocks, grouped queries under H2O,
        # eviction after the attention
        _decode("decode_serving_blocked", 32, 6, 301, 2003, 3333, 13, 32, 4, 128, "bf16", "h2o",
                order="attend_then_evict", layout="blocked", ragged=True),
        # H2O prompt scores of one layer, batch 8 of the 7B shape
        _scores("scores_7b", 8, 32, 32, 2048, 128, "bf16"),
        # the same producer in fp32 at head size 64, prompts of different length (the small configuration's
        # number format and head size)
        _scores("scores_f32_ragged", 4, 16, 8, 777, 64, "f32", ragged=True),
        # the probe inside the residual add of one layer: what a prefill pays per layer
        _probe("probe_residual_layer", "residual", 1, 16384, 4096, "bf16"),
        # prompt compression of all layers of a batch (7B shape)
        _compress("compress_7b_h2o", 32, 4, 143, 2271, 2048, 8, 32, 128, "bf16", "h2o"),
        # one sequence joins a running batch: its prompt into blocks that another one gave back
        _compress("compress_join_blocked", 32, 6, 301, 2003, 1777, 13, 8, 128, "bf16", "h2o", layout="blocked", join=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode"] * 5 + ["scores"] * 2 + ["probe"] + ["compress"] * 2)
    dtype = rng.choice(["bf16"] * 4 + ["f32"])
    D = rng.choice([64, 128, 128])
    policy = rng.choice(["h2o", "h2o", "streaming", "sliding"])
    if kind == "decode":
        g, Hkv = rng.choice([1, 1, 2, 4, 8]), rng.choice([2, 4, 8, 16, 32])
        while g * Hkv > 64:
            Hkv //= 2
        L = _log_int(rng, 1, 80)
        n_high = max(1, int(L * rng.uniform(0.1, 0.5)))
        b_low = _log_int(rng, 16, 1300)
        b_high = min(8192, int(b_low * rng.uniform(1.5, 16)))
        layout = rng.choice(["dense", "dense", "blocked", "packed"])
        c = _decode("", L, n_high, b_low, b_high, int(b_high * rng.uniform(0.9, 1.6)) + 1, _log_int(rng, 1, 224), g * Hkv,
                    Hkv, D, dtype, policy, order=rng.choice(["evict_then_attend"] * 3 + ["attend_then_evict"]),
                    layout=layout, ragged=layout == "packed" or rng.random() < 0.2,
                    calls="layers" if L <= 40 and rng.random() < 0.3 else "together")
        while work(c)["bytes"] > 8e9:
            c["batch"] = max(1, c["batch"] * 2 // 3)
    elif kind == "scores":
        g, Hkv = rng.choice([1, 2, 4, 8]), rng.choice([2, 4, 8, 16, 32])
        while g * Hkv > 64:
            Hkv //= 2
        c = _scores("", _log_int(rng, 1, 16), g * Hkv, Hkv, _log_int(rng, 40, 4096), D, dtype, ragged=rng.random() < 0.4,
                    lse=rng.random() < 0.3)
        most = 1.3e11 if dtype == "bf16" and D == 128 else 1.5e10
        while work(c)["flops"] > most:
            if c["batch"] > 1:
                c["batch"] = max(1, c["batch"] * 2 // 3)
            else:
                c["prompt"] = c["prompt"] * 2 // 3
    elif kind == "probe":
        form = rng.choice(["alone", "residual", "residual", "per_sequence"])
        n_seq = rng.randint(2, 16) if form == "per_sequence" else 1
        c = _probe("", form, _log_int(rng, 1, 32), n_seq * _log_int(rng, 17, 4096), rng.choice([256, 1024, 2048, 4096, 5120, 8192]),
                   dtype, n_seq)
        while work(c)["bytes"] > 8e9:
            c["layers"] = max(1, c["layers"] * 2 // 3)
            c["tokens"] = max(n_seq, c["tokens"] * 4 // 5)
    else:
        L = _log_int(rng, 1, 80)
        P = _log_int(rng, 64, 4096)
        n_high = max(1, int(L * rng.uniform(0.1, 0.5)))
        b_low = max(8, int(P * rng.uniform(0.05, 0.15)))
        b_high = max(b_low + 1, int(P * rng.uniform(0.2, 1.2)))
        join = rng.random() < 0.4
        layout = rng.choice(["dense", "blocked"]) if join else rng.choice(["dense", "dense", "blocked", "packed"])
        c = _compress("", L, n_high, b_low, b_high, P, _log_int(rng, 2 if join else 1, 32), rng.choice([4, 8, 16, 32]), D, dtype,
                      policy, layout=layout, ragged=layout == "packed" or (not join and rng.random() < 0.3), join=join)
        # (the prompts lie in memory whole, whatever is kept of them)
        while 2 * c["layers"] * c["batch"] * c["kv_heads"] * P * D * (2 if dtype == "bf16" else 4) > 10e9:
            c["batch"] = max(2 if join else 1, c["batch"] * 2 // 3)
            c["layers"] = max(1, c["layers"] * 3 // 4)
            c["n_high"] = max(1, min(c["n_high"], c["layers"]))
    del c["name"]
    return c


# ---- sizes that follow from a case ----------------------------------------------------------------------------
def _budgets(c):
    """Per layer; the layers with the large budget lie at both ends."""
    L, n = c["layers"], c["n_high"]
    first = (n + 1) // 2
    return [c["b_high"] if l < first or l >= L - (n - first) else c["b_low"] for l in range(L)]


def _fractions(c):
    """How long each sequence is, as a share of the longest."""
    B = c["batch"]
    return [1.0 - 0.5 * (b / max(B - 1, 1)) if c["ragged"] else 1.0 for b in range(B)]


def _seq_budget(budget, f):
    return max(8, int(budget * f)) if f < 1.0 else budget


def _work_tokens(c):
    """Tokens attended in one step, summed over layers and sequences."""
    total = 0
    for budget in _budgets(c):
        for f in _fractions(c):
            b, n = _seq_budget(budget, f), max(8, int(c["tokens"] * f))
            extra = 1 if c["order"] == "attend_then_evict" else 0
            total += min(n + 1, b + extra)
    return total


def work(case):
    c = case
    if c["kind"] == "decode":
        e = 2 if c["dtype"] == "bf16" else 4
        tok = _work_tokens(c)
        units = c["layers"] * c["batch"] * c["kv_heads"]
        row = c["dim"] * e
        nbytes = tok * c["kv_heads"] * (2 * row + (8 if c["policy"] == "h2o" else 0)) + 2 * units * row \
            + 2 * c["layers"] * c["batch"] * c["heads"] * row
        return {"bytes": nbytes, "flops": 4.0 * tok * c["heads"] * c["dim"]}
    if c["kind"] == "scores":
        e = 2 if c["dtype"] == "bf16" else 4
        lens = [max(1, int(c["prompt"] * f)) for f in _fractions(c)]
        nbytes = sum(n * (c["heads"] + c["kv_heads"]) * c["dim"] * e for n in lens) + 4 * c["batch"] * c["kv_heads"] * c["prompt"] \
            + (4 * sum(lens) * c["heads"] if c["lse"] else 0)
        return {"bytes": nbytes, "flops": sum(float(n) * (n + 1) * c["dim"] * c["heads"] for n in lens)}
    if c["kind"] == "probe":
        e = 2 if c["dtype"] == "bf16" else 4
        elems = c["layers"] * c["tokens"] * c["hidden"]
        return {"bytes": elems * e * (3 if c["form"] == "residual" else 2), "flops": 6.0 * elems}
    e = 2 if c["dtype"] == "bf16" else 4
    seqs = [1.0] if c["join"] else _fractions(c)
    nbytes = 0
    for budget in _budgets(c):
        for f in seqs:
            n = max(1, int(c["prompt"] * f))
            keep = min(n, _seq_budget(budget, f))
            per_unit = 4 * keep * c["dim"] * e + 4 * keep + 16
            if c["policy"] == "h2o":
                per_unit += 4 * n + 4 * keep
            nbytes += c["kv_heads"] * per_unit
    return {"bytes": nbytes, "flops": 0.0}


# ---- inputs ---------------------------------------------------------------------------------------------------
def _gen(seed, stream):
    return torch.Generator(device="cuda").manual_seed(seed * 1009 + stream)


def _normal(shape, dtype, gen):
    return torch.empty(shape, dtype=dtype, device="cuda").normal_(generator=gen)


def _directions(c, seed):
    """One unit vector per (layer, KV head): queries lean towards it, heavy hitters' keys too."""
    u = _normal((c.get("layers", 1), c["kv_heads"], c["dim"]), torch.float32, _gen(seed, 1))
    return u / u.norm(dim=-1, keepdim=True)


def _keys(shape, dtype, gen, u, share=0.02, lean=3.0):
    """K [B, H, n, D]: normal, and in `share` of a sequence's positions leaning towards u [H, D]."""
    K = _normal(shape, dtype, gen)
    heavy = torch.rand(shape[0], 1, shape[2], 1, device="cuda", generator=gen) < share
    K += (heavy * (lean * u[None, :, None, :])).to(dtype)
    return K


def _queries(c, seed, lead, u):
    """[*lead, Hkv, g, D] normal + 3 u, as [*lead, Hq, D]."""
    g = c["heads"] // c["kv_heads"]
    q = _normal((*lead, c["kv_heads"], g, c["dim"]), DTYPES[c["dtype"]], _gen(seed, 2))
    q += (3.0 * u).to(q.dtype)
    return q.reshape(*lead, c["heads"], c["dim"])


def _layer_cache(c, seed, l):
    """The dense contents of layer l's cache just before a step: K, V [B, Hkv, cap, D], score, pos [B, Hkv, cap],
    state [B, Hkv, 4], and per sequence the budget and the tokens seen.  Slots [0, hh) hold the kept older
    tokens, the rest is a ring of the recent ones (ascending while the unit is not full)."""
    budget, B, H = _budgets(c)[l], c["batch"], c["kv_heads"]
    gen = _gen(seed, 100 + l)
    cap = budget
    K = _keys((B, H, cap, c["dim"]), DTYPES[c["dtype"]], gen, _directions(c, seed)[l])
    V = _normal((B, H, cap, c["dim"]), DTYPES[c["dtype"]], gen)
    r = torch.rand(B, H, cap, device="cuda", generator=gen)
    heads = torch.rand(B, H, device="cuda", generator=gen)
    score = torch.zeros(B, H, cap, device="cuda")
    pos = torch.full((B, H, cap), -1, dtype=torch.int32, device="cuda")
    state = torch.zeros(B, H, 4, dtype=torch.int32, device="cuda")
    state[..., 2] = -2
    s = torch.arange(cap, device="cuda")
    seq = []
    for b, f in enumerate(_fractions(c)):
        bud, n = _seq_budget(budget, f), max(8, int(c["tokens"] * f))
        seq.append((bud, n))
        hh = bud // 2 if c["policy"] == "h2o" else (N_SINK if c["policy"] == "streaming" else 0)
        rec = bud - hh
        if n < bud:                                            # everything seen is still there
            pos[b, :, :n] = s[:n].to(torch.int32)
            state[b, :, 0] = n
            score[b, :, :n] = 0.2 + r[b, :, :n]
            continue
        state[b, :, 0] = bud
        head = (heads[b] * rec).to(torch.int64).clamp_(max=rec - 1)
        state[b, :, 1] = head.to(torch.int32)
        if hh:
            older = s[:hh] if c["policy"] == "streaming" else s[:hh] * (n - rec) // hh
            pos[b, :, :hh] = older.to(torch.int32)
        pos[b, :, hh:bud] = (n - rec + (s[None, :rec] - head[:, None]) % rec).to(torch.int32)
        score[b, :, :hh] = 1.0 + 4.0 * r[b, :, :hh]             # heavy hitters have the larger sums
        score[b, :, hh:bud] = 1.5 * r[b, :, hh:bud]
    return K, V, score, pos, state, seq


def _row_index(c, caches, l, unit_caps):
    """Row of each unit's slots in the layer's K / V: index [U, cap], and which of them exist."""
    U, cap = c["batch"] * c["kv_heads"], caches.capacities[l]
    s = torch.arange(cap, device="cuda")
    if c["layout"] == "blocked":
        t = caches.block_table[l].to(torch.int64)
        return t[:, s // BLOCK] * BLOCK + s % BLOCK, torch.ones(U, cap, dtype=torch.bool, device="cuda")
    own = torch.tensor(unit_caps[l], device="cuda")
    start = torch.cumsum(own, 0) - own
    return start[:, None] + s[None, :], s[None, :] < own[:, None]


def _one_arena(caches):
    """Gives all layers' caches one buffer per kind of data (aligned to 256 bytes), as a program with an arena
    has them, and enters the new addresses into the layer table."""
    out = {}
    for name, field in (("K", "K"), ("V", "V"), ("score", "score_acc"), ("pos", "pos"), ("state", "unit_state")):
        parts = getattr(caches, name)
        if parts[0] is None:
            continue
        es = parts[0].element_size()
        sizes = [(t.numel() * es + 255) // 256 * 256 // es for t in parts]
        flat = torch.zeros(sum(sizes), dtype=parts[0].dtype, device="cuda")
        at = 0
        for i, t in enumerate(parts):
            v = flat[at:at + t.numel()].view(t.shape)
            v.copy_(t)
            parts[i] = v
            setattr(caches.table[i], field, v.data_ptr())
            at += sizes[i]
        out[name] = flat
    caches.lens, caches.head, caches.hint = ([s[..., k] for s in caches.state] for k in range(3))
    caches.table_dev = torch.frombuffer(bytearray(bytes(memoryview(caches.table))), dtype=torch.uint8).to("cuda")
    return out


def _unit_caps(c):
    """Slots of every unit, [layer][unit]: all its layer's budget, or (packed) its own."""
    return [[_seq_budget(b, f) if c["layout"] == "packed" else b for f in _fractions(c) for _ in range(c["kv_heads"])]
            for b in _budgets(c)]


def _new_caches(c):
    budgets, caps = _budgets(c), _unit_caps(c)
    packed = c["layout"] == "packed"
    return sqa.LayerCaches(budgets, [max(x) for x in caps], c["batch"], c["kv_heads"], c["dim"], DTYPES[c["dtype"]], "cuda",
                           c["policy"] == "h2o", unit_capacities=caps if packed else None, blocked=c["layout"] == "blocked")


def _budget_seq(c):
    return torch.tensor([[_seq_budget(b, f) for f in _fractions(c)] for b in _budgets(c)], dtype=torch.int32, device="cuda")


def _decode_inputs(c, seed):
    L, B, H, D, dt = c["layers"], c["batch"], c["kv_heads"], c["dim"], DTYPES[c["dtype"]]
    u = _directions(c, seed)
    q = _queries(c, seed, (STEPS, L, B), u[:, None, :, None, :])
    k = _normal((STEPS, L, B, H, D), dt, _gen(seed, 3))
    v = _normal((STEPS, L, B, H, D), dt, _gen(seed, 4))
    return q, k, v


def _prepare_decode(c, seed):
    caches, caps = _new_caches(c), _unit_caps(c)
    buffers = _one_arena(caches)
    for l in range(c["layers"]):
        K, V, score, pos, state, _ = _layer_cache(c, seed, l)
        if c["layout"] == "dense":
            caches.K[l].copy_(K)
            caches.V[l].copy_(V)
        else:
            at, there = _row_index(c, caches, l, caps)
            D = c["dim"]
            caches.K[l].view(-1, D)[at[there]] = K.view(*at.shape, D)[there]
            caches.V[l].view(-1, D)[at[there]] = V.view(*at.shape, D)[there]
        if c["layout"] == "packed":
            there = there.view(score.shape)
            score, pos = score[there], pos[there]
        if c["policy"] == "h2o":
            caches.score[l].copy_(score)
        caches.pos[l].copy_(pos)
        caches.state[l].copy_(state)
    q, k, v = _decode_inputs(c, seed)
    st = {"case": c, "caches": caches, "buffers": buffers, "q": q, "k": k, "v": v, "out": torch.zeros_like(q[0]),
          "at": 0, "pos": c["tokens"], "opts": [None] * c["layers"]}
    layers = c["calls"] == "layers"
    if c["ragged"]:
        st["budget_seq"] = _budget_seq(c)
        st["pos_seq"] = torch.tensor([max(8, int(c["tokens"] * f)) for f in _fractions(c)], dtype=torch.int32, device="cuda")
        st["opts"] = [sqa.batch_opts(budget_seq=st["budget_seq"][l], new_pos_seq=st["pos_seq"], order=c["order"])
                      for l in range(c["layers"] if layers else 1)]
    elif c["order"] != "evict_then_attend":
        st["opts"] = [sqa.batch_opts(order=c["order"])] * c["layers"]
    if layers:
        st["ws"] = [sqa.decode_workspace(caches, c["heads"], c["policy"], l, 1) for l in range(c["layers"])]
    else:
        st["ws"] = sqa.decode_workspace(caches, c["heads"], c["policy"])
    return st


def _run_decode(st):
    c, t = st["case"], st["at"] % STEPS
    q, k, v, out, caches = st["q"][t], st["k"][t], st["v"][t], st["out"], st["caches"]
    if c["calls"] == "layers":
        for l in range(c["layers"]):
            sqa.decode_step(q[l], k[l], v[l], st["pos"], c["policy"], N_SINK, caches, out[l], st["ws"][l], layer0=l, n_layers=1,
                            opts=st["opts"][l])
    else:
        sqa.decode_step(q, k, v, st["pos"], c["policy"], N_SINK, caches, out, st["ws"], opts=st["opts"][0])
    st["at"] += 1
    st["pos"] += 1
    if c["ragged"]:
        st["pos_seq"].add_(1)
    return {"out": out, **st["buffers"]}


def _exact_decode(c, seed):
    if work(c)["bytes"] > 1.4e10:
        return None
    q, k, v = _decode_inputs(c, seed)
    q, k, v = q[0], k[0], v[0]
    B, H, D, g = c["batch"], c["kv_heads"], c["dim"], c["heads"] // c["kv_heads"]
    ae, h2o = c["order"] == "attend_then_evict", c["policy"] == "h2o"
    outs, scores, caps = [], [], _unit_caps(c)
    for l, budget in enumerate(_budgets(c)):
        K, V, score, pos, state, seq = _layer_cache(c, seed, l)
        sc_out = torch.zeros(B, H, budget, dtype=torch.float64, device="cuda")
        out = torch.empty(B, c["heads"], D, dtype=torch.float64, device="cuda")
        for b, (bud, n) in enumerate(seq):
            full = n >= bud
            hh = bud // 2 if h2o else (N_SINK if c["policy"] == "streaming" else 0)
            held = bud if full else n
            hidx = torch.arange(H, device="cuda")
            wr = (hh + state[b, :, 1]).long() if full else torch.full((H,), n, device="cuda")      # slot of the new token
            Kb, Vb, sb = K[b, :, :held].double(), V[b, :, :held].double(), score[b, :, :held].double()

            def leaves(sc):
                """Heavy slot that gives way to the token leaving the ring, -1: the latter goes itself."""
                heavy, leaver = sc[:, :hh], sc[hidx, wr]
                low = heavy.min(dim=1).values
                at = torch.where(heavy == low[:, None], pos[b, :, :hh].long(), -2).max(dim=1).indices
                return torch.where(leaver > low, at, -1)

            def put(x, victim, new):
                """x with the ring leaver moved to `victim` and `new` in its place."""
                moved = victim >= 0
                x = x.clone()
                x[hidx[moved], victim[moved]] = x[hidx[moved], wr[moved]]
                x[hidx, wr] = new
                return x

            none = torch.full((H,), -1, device="cuda")
            kb, vb = k[l, b].double(), v[l, b].double()
            if full and not ae:
                victim = leaves(score[b, :, :held]) if h2o else none
                Kb, Vb, sb = put(Kb, victim, kb), put(Vb, victim, vb), put(sb, victim, 0.0)
            else:
                Kb, Vb = torch.cat([Kb, kb[:, None]], 1), torch.cat([Vb, vb[:, None]], 1)
                sb = torch.cat([sb, torch.zeros(H, 1, dtype=torch.float64, device="cuda")], 1)
            p = torch.softmax(torch.matmul(q[l, b].view(H, g, D).double(), Kb.transpose(1, 2).contiguous()) / math.sqrt(D), -1)
            out[b] = torch.matmul(p, Vb).reshape(c["heads"], D)
            sb = sb + p.sum(1)
            if full and ae:
                victim = leaves(sb[:, :held].float()) if h2o else none
                sb = put(sb[:, :held], victim, sb[:, held])
            sc_out[b, :, :sb.shape[1]] = sb
        outs.append(out)
        if c["layout"] == "packed":
            there = torch.arange(max(caps[l]), device="cuda")[None] < torch.tensor(caps[l], device="cuda")[:, None]
            sc_out = sc_out.view(B * H, -1)[:, :max(caps[l])][there]
        sc_out = sc_out.reshape(-1)
        scores.append(torch.cat([sc_out, sc_out.new_zeros(-sc_out.numel() % 64)]))
    got = {"out": torch.stack(outs), "K": None, "V": None, "pos": None, "state": None}
    if h2o:
        got["score"] = torch.cat(scores)
    return got


def _score_inputs(c, seed):
    B, P, dt = c["batch"], c["prompt"], DTYPES[c["dtype"]]
    u = _directions(c, seed)[0]
    K = _keys((B, c["kv_heads"], P, c["dim"]), dt, _gen(seed, 5), u)
    g = c["heads"] // c["kv_heads"]
    Q = _normal((B, c["kv_heads"], g, P, c["dim"]), dt, _gen(seed, 6))
    Q += (3.0 * u[None, :, None, None, :]).to(dt)
    return Q.reshape(B, c["heads"], P, c["dim"]), K, [max(1, int(P * f)) for f in _fractions(c)]


def _logits(c, Q, K, b, h, dtype):
    """Causal logits [P, P] of query head h of sequence b."""
    P = c["prompt"]
    x = torch.matmul(Q[b, h].to(dtype), K[b, h // (c["heads"] // c["kv_heads"])].to(dtype).T.contiguous()) / math.sqrt(c["dim"])
    return x.masked_fill_(torch.ones(P, P, dtype=torch.bool, device="cuda").triu_(1), -math.inf)


def _prepare_scores(c, seed):
    Q, K, lens = _score_inputs(c, seed)
    st = {"case": c, "Q": Q, "K": K, "opts": None, "lse": None}
    if c["ragged"]:
        st["len"] = torch.tensor(lens, dtype=torch.int32, device="cuda")
        st["opts"] = sqa.batch_opts(prompt_len=st["len"])
    if c["lse"]:                                               # what a fused attention forward hands over
        st["lse"] = torch.stack([torch.stack([torch.logsumexp(_logits(c, Q, K, b, h, torch.float32), 1)
                                              for h in range(c["heads"])]) for b in range(c["batch"])])
    return st


def _exact_scores(c, seed):
    if work(c)["flops"] > 2e11:
        return None
    Q, K, lens = _score_inputs(c, seed)
    got = torch.zeros(c["batch"], c["kv_heads"], c["prompt"], dtype=torch.float64, device="cuda")
    for b in range(c["batch"]):
        for h in range(c["heads"]):
            p = torch.softmax(_logits(c, Q, K, b, h, torch.float64), 1)
            got[b, h // (c["heads"] // c["kv_heads"])] += p[:lens[b]].sum(0)
    return {"scores": got}


def _probe_inputs(c, seed):
    """Hidden states and what the attention adds to them, larger in the first and the last layer."""
    L, dt = c["layers"], DTYPES[c["dtype"]]
    shape = (L, c["tokens"], c["hidden"])
    a, r = _normal(shape, dt, _gen(seed, 7)), _normal(shape, dt, _gen(seed, 8))
    for l in range(L):
        r[l] *= 2.0 if l in (0, L - 1) else 0.45
    return a, r


def _seq_starts(c):
    n, T = c["n_seq"], c["tokens"]
    return [T * i * (i + n) // (2 * n * n) for i in range(n)] + [T]


def _prepare_probe(c, seed):
    a, r = _probe_inputs(c, seed)
    st = {"case": c, "h_in": a, "cos": torch.zeros(c["layers"], device="cuda")}
    if c["form"] == "residual":
        st["attn"], st["h_out"] = r, torch.zeros_like(a)
    else:
        st["h_out"] = a + r
    need = sqa._lib.sqa_layer_importance_workspace_bytes(c["layers"], c["tokens"], c["hidden"])
    st["ws"] = torch.empty(max(need, 8), dtype=torch.uint8, device="cuda")
    st["start"] = torch.tensor(_seq_starts(c), dtype=torch.int32, device="cuda")
    return st


def _run_probe(st):
    c = st["case"]
    if c["form"] == "residual":
        return {"cos": sqa.residual_add_importance(st["h_in"], st["attn"], st["h_out"], st["cos"], st["ws"]), "h_out": st["h_out"]}
    if c["form"] == "per_sequence":
        return {"cos": sqa.layer_importance_seq(st["h_in"], st["h_out"], st["start"])}
    return {"cos": sqa.layer_importance(st["h_in"], st["h_out"], st["cos"], st["ws"])}


def _exact_probe(c, seed):
    a, r = _probe_inputs(c, seed)
    cos, stored = [], []
    for l in range(c["layers"]):
        x = a[l].double()
        if c["form"] == "residual":
            if c["tokens"] * c["hidden"] * c["layers"] <= 1 << 28:
                stored.append(x + r[l].double())
        y = (a[l] + r[l]).double()                             # as stored: the probe is taken of the stored values
        each = (x * y).sum(1) / (x.norm(dim=1).clamp(min=1e-8) * y.norm(dim=1).clamp(min=1e-8))
        if c["form"] == "per_sequence":
            s = _seq_starts(c)
            cos.append(torch.stack([each[i:j].mean() if j > i else each.new_zeros(()) for i, j in zip(s, s[1:])]))
        else:
            cos.append(each.mean())
    got = {"cos": torch.stack(cos)}
    if c["form"] == "residual":
        got["h_out"] = torch.stack(stored) if stored else None
    return got


def _prepare_compress(c, seed):
    B, H, P, D, dt = c["batch"], c["kv_heads"], c["prompt"], c["dim"], DTYPES[c["dtype"]]
    rows = 1 if c["join"] else B
    st = {"case": c, "K": [], "V": [], "scores": [], "opts": None, "table": None}
    for l in range(c["layers"]):
        gen = _gen(seed, 100 + l)
        st["K"].append(_normal((rows, H, P, D), dt, gen))
        st["V"].append(_normal((rows, H, P, D), dt, gen))
        # column sums of a causal softmax: larger for early tokens, a few much larger than the rest
        s = torch.empty(rows, H, P, device="cuda").exponential_(generator=gen)
        st["scores"].append(s * torch.log(P / (torch.arange(P, device="cuda") + 1.0) + 1.0) if c["policy"] == "h2o" else None)
    caches = _new_caches(c)
    st["caches"], st["buffers"] = caches, _one_arena(caches)
    if c["join"]:
        st["table"] = caches.sequence_table(seed % B)
    elif c["ragged"]:
        st["len"] = torch.tensor([max(1, int(P * f)) for f in _fractions(c)], dtype=torch.int32, device="cuda")
        st["budget_seq"], st["status"] = _budget_seq(c), torch.zeros(1, dtype=torch.int32, device="cuda")
        st["opts"] = sqa.batch_opts(prompt_len=st["len"], budget_seq=st["budget_seq"], status=st["status"])
    return st


def prepare(case, seed):
    return {"decode": _prepare_decode, "scores": _prepare_scores, "probe": _prepare_probe,
            "compress": _prepare_compress}[case["kind"]](case, seed)


def run(state):
    kind = state["case"]["kind"]
    if kind == "decode":
        return _run_decode(state)
    if kind == "scores":
        return {"scores": sqa.prefill_scores(state["Q"], state["K"], opts=state["opts"], row_lse=state["lse"])}
    if kind == "probe":
        return _run_probe(state)
    sqa.prefill_compress_layers(state["K"], state["V"], state["scores"], state["case"]["policy"], N_SINK, state["caches"],
                                opts=state["opts"], table=state["table"])
    return state["buffers"]


def exact(case, seed):
    if case["kind"] == "compress":                             # rows and scores are copied, nothing is computed
        return None
    return {"decode": _exact_decode, "scores": _exact_scores, "probe": _exact_probe}[case["kind"]](case, seed)


def tolerance(case):
    if case["kind"] == "compress":
        return "exact"
    if case["kind"] == "scores":                               # fp32 sums of up to thousands of rows (3e-7 measured),
        return {"rel": 4e-6, "max": 4e-5}                      # given normalisers are rounded to fp32 as well
    if case["dtype"] == "f32" or (case["kind"] == "probe" and case["form"] != "residual"):
        return {"rel": 2e-6, "max": 2e-5, "differ": 1e-4}      # (1e-7 measured)
    return {"rel": 8e-3, "max": 4e-2, "differ": 1e-4}          # bf16 outputs: 2e-3 measured, 2^-9 per value at most
