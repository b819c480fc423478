"""Decode calls of more work items than the chip has CUs: their workgroups have 4 waves (calls of up to 256, which most
small tests are, have 8 and another end of a step).  What a step of a real model over all its layers launches, at sizes that
a test can follow: a sample of the units, from the GPU's own state, against the oracle."""
import numpy as np
import pytest
import torch

from oracle import sqa_oracle as O
from tests.harness import TOL, check_step_scores, export_state, np64, oracle_view, rel_err, uses_matrix_cores
from tests.test_gpu_stepping import _run_case

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
EA, AE = "evict_then_attend", "attend_then_evict"


@pytest.fixture(scope="module")
def sqa():
    from paper_2404_04793_amd import binding
    return binding


def _plan(sqa, budgets, B, g, Hkv, D, dtype, policy, blocked=False, caps=None):
    p = sqa.decode_plan(budgets, caps or budgets, B, g * Hkv, Hkv, D, dtype, policy, blocked)
    assert p["waves"] == 4 and p["workgroups"] > 256
    return p


def _dtype(dtype):
    return torch.float32 if dtype == "f32" else torch.bfloat16


CASES = [
    # dtype, D, g, policy, order, blocked, B (of 8 KV heads each), budgets, pieces per unit
    ("f32", 64, 1, "h2o", EA, False, 33, [300], 1),          # 264 whole units: long tails by all waves only above 512 slots
    ("f32", 128, 1, "h2o", AE, True, 33, [140], 1),
    ("f32", 128, 2, "h2o", EA, True, 17, [37, 300], 1),
    ("f32", 128, 4, "h2o", EA, False, 33, [300], 1),
    ("f32", 128, 8, "h2o", AE, False, 33, [300], 1),
    ("f32", 64, 4, "h2o", AE, True, 33, [300], 1),
    ("bf16", 64, 1, "h2o", EA, True, 33, [300], 1),
    ("bf16", 64, 2, "h2o", AE, False, 33, [600], 1),
    ("bf16", 64, 4, "h2o", EA, False, 17, [300, 37], 1),
    ("bf16", 128, 2, "h2o", EA, True, 33, [600], 1),
    ("f32", 128, 4, "sliding", EA, True, 33, [300], 1),
    ("f32", 128, 8, "streaming", EA, True, 33, [300], 1),
    ("f32", 64, 2, "streaming", AE, False, 33, [300], 1),
    ("bf16", 64, 4, "sliding", EA, False, 33, [300], 1),
    ("bf16", 128, 1, "streaming", EA, True, 33, [300], 1),
    ("bf16", 128, 4, "streaming", EA, False, 33, [300], 1),
    ("bf16", 64, 1, "h2o", EA, False, 33, [330], 1),         # units that fill up (330 of 300 + 12 tokens)
    # 160 units in three pieces each
    ("f32", 64, 1, "h2o", EA, False, 20, [1400], 3),
    ("f32", 128, 4, "h2o", AE, False, 20, [1400], 3),
    ("bf16", 64, 4, "h2o", AE, True, 20, [1400], 3),
    ("bf16", 128, 2, "h2o", EA, True, 20, [1400], 3),
    ("bf16", 128, 1, "sliding", EA, False, 20, [1400], 3),
]


@pytest.mark.parametrize("dtype,D,g,policy,order,blocked,B,budgets,pieces", CASES,
                         ids=["%s_D%d_g%d_%s_%s_%s_%s" % (c[0], c[1], c[2], c[3], c[4][:6], "blocked" if c[5] else "dense",
                                                          "x".join(map(str, c[7]))) for c in CASES])
def test_stepping(sqa, dtype, D, g, policy, order, blocked, B, budgets, pieces):
    S = 12 if budgets == [330] else 5
    P = 300 if budgets == [330] else max(budgets) + 20
    p = _plan(sqa, budgets, B, g, 8, D, dtype, policy, blocked, [min(b, P + S) for b in budgets])
    assert p["layers"][0]["workgroups_per_unit"] == pieces
    _run_case(sqa, ("four_waves", dtype, 8 * g, 8, D, B, P, S, policy, budgets, order), stride=B * 8 * len(budgets) // 5,
              blocked=blocked, need_both_outcomes=False)


def _step_and_check(sqa, caches, ws, out, q, k, v, pos, budget, policy, units, order=EA, opts=None, new_pos=None):
    """One step of a single layer; the named units (b, h, budget) against the oracle from their state before it."""
    B, Hq, D = q.shape[-3:]
    g = Hq // caches.Hkv
    dtype = "f32" if q.dtype == torch.float32 else "bf16"
    before = {(b, h): export_state(caches, 0, b, h) for b, h, _ in units}
    sqa.decode_step(q, k, v, pos, policy, 4, caches, out, ws, opts=opts if opts is not None else sqa.batch_opts(order=order))
    qn, kn, vn, o = np64(q), np64(k), np64(v), np64(out)
    for b, h, bud in units:
        at = pos if new_pos is None else new_pos[b]
        want, c2 = O.decode_step(oracle_view(before[b, h]), qn[0, b, h * g:(h + 1) * g], kn[0, b, h], vn[0, b, h], at, bud, policy,
                                 4, order=order)
        got = export_state(caches, 0, b, h)
        assert got["pos"].tolist() == c2["pos"].tolist(), (at, b, h)
        assert np.array_equal(got["K"], c2["K"]) and np.array_equal(got["V"], c2["V"])
        assert rel_err(o[0, b, h * g:(h + 1) * g], want) < TOL[dtype]
        if policy == "h2o":
            check_step_scores(got, before[b, h], c2, uses_matrix_cores(dtype, D, g), (at, b, h))


@pytest.mark.parametrize("order", [EA, AE])
@pytest.mark.parametrize("dtype,D,g,B,b", [("f32", 64, 1, 33, 300), ("bf16", 128, 2, 33, 600), ("f32", 128, 4, 33, 140),
                                           ("bf16", 64, 8, 33, 300), ("f32", 64, 2, 20, 1400)])
def test_equal_scores(sqa, dtype, D, g, B, b, order):
    """Equal keys and scores: every heavy hitter ties for the lowest score, a thread meets it several times, and the highest
    position has to go (the recent window's scores are higher, so its leaver moves in).  Whole units, and units in pieces."""
    Hkv, P = 8, b + 40
    _plan(sqa, [b], B, g, Hkv, D, dtype, "h2o")
    dt = _dtype(dtype)
    gen = torch.Generator(device=DEV).manual_seed(b)
    mk = lambda *shape: torch.randn(*shape, generator=gen, device=DEV).to(dt)
    sc = torch.ones(B, Hkv, P, device=DEV)
    sc[..., P - (b - b // 2):] = 2.0
    caches = sqa.LayerCaches([b], [b], B, Hkv, D, dt, DEV, True)
    sqa.prefill_compress(torch.zeros(B, Hkv, P, D, dtype=dt, device=DEV), mk(B, Hkv, P, D), sc, "h2o", 4, caches, 0)
    ws = sqa.decode_workspace(caches, Hkv * g, "h2o")
    for t in range(3):
        q = mk(1, B, Hkv * g, D)
        _step_and_check(sqa, caches, ws, torch.empty_like(q), q, torch.zeros(1, B, Hkv, D, dtype=dt, device=DEV), mk(1, B, Hkv, D), P + t, b,
                        "h2o", [(0, 0, b), (B // 2, 3, b), (B - 1, 7, b)], order)
    assert sqa.read_device_status(ws) == 0


@pytest.mark.parametrize("policy,dtype,D,g,layout,order", [("h2o", "f32", 64, 1, "packed", EA), ("h2o", "bf16", 64, 4, "blocked", EA),
                                                           ("h2o", "f32", 128, 4, "packed", AE), ("streaming", "bf16", 128, 2, "packed", EA),
                                                           ("sliding", "f32", 128, 2, "dense", EA), ("h2o", "bf16", 128, 4, "packed", EA)])
def test_sequences_of_different_length(sqa, policy, dtype, D, g, layout, order):
    """Prompts, budgets and positions per sequence; every third sequence sits a step out and stays as it is."""
    B, Hkv, P, S = 66, 4, 260, 4
    plen = [P - 3 * b for b in range(B)]
    bseq = [min(200 - 2 * b, plen[b]) for b in range(B)]
    dt = _dtype(dtype)
    gen = torch.Generator(device=DEV).manual_seed(D + g)
    mk = lambda *shape: torch.randn(*shape, generator=gen, device=DEV).to(dt)
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device=DEV)
    caps = [[x for x in bseq for _ in range(Hkv)]]
    caches = sqa.LayerCaches([200], [200], B, Hkv, D, dt, DEV, policy == "h2o", unit_capacities=caps if layout == "packed" else None,
                             blocked=layout == "blocked")
    _plan(sqa, [200], B, g, Hkv, D, dtype, policy, layout == "blocked")
    sc = torch.rand(B, Hkv, P, generator=gen, device=DEV) + 0.1
    pl, bs = i32(plen), i32([bseq])
    status = torch.zeros(1, dtype=torch.int32, device=DEV)
    sqa.prefill_compress_layers([mk(B, Hkv, P, D)], [mk(B, Hkv, P, D)], [sc] if policy == "h2o" else None, policy, 4, caches,
                                opts=sqa.batch_opts(prompt_len=pl, budget_seq=bs, status=status))
    assert int(status.item()) == 0
    ws = sqa.decode_workspace(caches, Hkv * g, policy)
    at = list(plen)
    for t in range(S):
        on = [b % 3 != t % 3 for b in range(B)]
        new_pos = [at[b] if on[b] else -1 for b in range(B)]
        new_pos_d = i32(new_pos)
        q, k, v = mk(1, B, Hkv * g, D), mk(1, B, Hkv, D), mk(1, B, Hkv, D)
        out = torch.full_like(q, 7.0)
        idle = [b for b in (0, 1, 2, B - 1) if not on[b]]
        kept = {b: export_state(caches, 0, b, Hkv - 1) for b in idle}
        _step_and_check(sqa, caches, ws, out, q, k, v, 0, None, policy, [(b, h, bseq[b]) for b, h in ((0, 0), (1, 3), (31, 1), (B - 1, 3)) if on[b]],
                        order, sqa.batch_opts(budget_seq=bs, new_pos_seq=new_pos_d, order=order), new_pos)
        for b, c in kept.items():
            got = export_state(caches, 0, b, Hkv - 1)
            assert bool((out[0, b] == 7.0).all()) and all(np.array_equal(got[x], c[x]) for x in ("pos", "K", "V", "score"))
        at = [x + int(a) for x, a in zip(at, on)]
    assert sqa.read_device_status(ws) == 0


@pytest.mark.parametrize("policy,dtype,D,g", [("h2o", "f32", 64, 1), ("h2o", "bf16", 128, 2), ("streaming", "bf16", 64, 4), ("sliding", "f32", 128, 2)])
def test_from_an_empty_cache(sqa, policy, dtype, D, g):
    B, Hkv, b = 33, 8, 6
    dt = _dtype(dtype)
    _plan(sqa, [b], B, g, Hkv, D, dtype, policy)
    caches = sqa.LayerCaches([b], [b], B, Hkv, D, dt, DEV, policy == "h2o")
    ws = sqa.decode_workspace(caches, Hkv * g, policy)
    gen = torch.Generator(device=DEV).manual_seed(g)
    mk = lambda *shape: torch.randn(*shape, generator=gen, device=DEV).to(dt)
    for t in range(9):
        q = mk(1, B, Hkv * g, D)
        _step_and_check(sqa, caches, ws, torch.empty_like(q), q, mk(1, B, Hkv, D), mk(1, B, Hkv, D), t, b, policy, [(0, 0, b), (B - 1, 7, b)])
    assert sqa.read_device_status(ws) == 0


def test_faulty_units_are_reported_and_left_alone(sqa):
    """264 units: a length beyond the budget, a block number outside the pools, and (packed) a unit without any slot."""
    B, Hkv, D, b, P = 33, 8, 64, 40, 50
    _plan(sqa, [b], B, 1, Hkv, D, "f32", "h2o", True)
    K, V, sc = (torch.randn(B, Hkv, P, D, device=DEV), torch.randn(B, Hkv, P, D, device=DEV), torch.rand(B, Hkv, P, device=DEV))
    q, k, v = (torch.randn(1, B, Hkv, D, device=DEV) for _ in range(3))
    for fault, code in (("length", 8), ("block", 2), ("no slots", 6)):
        caps = [[b] * (B * Hkv)]
        caps[0][8] = 0 if fault == "no slots" else b
        packed = fault == "no slots"
        caches = sqa.LayerCaches([b], [b], B, Hkv, D, torch.float32, DEV, True, blocked=not packed, unit_capacities=caps if packed else None)
        if not packed:
            sqa.prefill_compress(K, V, sc, "h2o", 4, caches, 0)
        good = export_state(caches, 0, 1, 0) if fault == "length" else None
        if fault == "length":
            caches.lens[0][1, 0] = b + 1
        elif fault == "block":
            caches.block_table[0][8, 1] = caches.K[0].shape[0]          # one past the last block
        ws = sqa.decode_workspace(caches, Hkv, "h2o")
        out = torch.full_like(q, 3.0)
        _step_and_check(sqa, caches, ws, out, q, k, v, P, b, "h2o", [(0, 7, b), (1, 1, b), (B - 1, 0, b)])     # the neighbours step
        assert sqa.read_device_status(ws) == code and bool((out[0, 1, 0] == 0).all()), fault
        assert int(caches.lens[0][1, 0]) == {"length": b + 1, "block": b, "no slots": 0}[fault]
        if fault == "length":
            caches.lens[0][1, 0] = b
            got = export_state(caches, 0, 1, 0)
            assert all(np.array_equal(got[x], good[x]) for x in ("pos", "K", "V", "score"))


@pytest.mark.parametrize("dtype,D,g,B,b", [("bf16", 128, 1, 20, 1400), ("f32", 128, 4, 33, 140)])
def test_replays_of_a_recorded_step(sqa, dtype, D, g, B, b):
    """Steps recorded into a graph (positions from a device array) and replayed, with eager work and a wait between the
    replays: the same bytes as eager steps, for units in pieces (arrival counters return to zero) and whole ones."""
    Hkv, P, S = 8, b + 10, 4
    _plan(sqa, [b], B, g, Hkv, D, dtype, "h2o")
    dt = _dtype(dtype)
    gen = torch.Generator(device=DEV).manual_seed(b)
    mk = lambda *shape: torch.randn(*shape, generator=gen, device=DEV).to(dt)
    K, V, sc = mk(B, Hkv, P, D), mk(B, Hkv, P, D), torch.rand(B, Hkv, P, generator=gen, device=DEV)
    q, k, v = mk(S, 1, B, Hkv * g, D), mk(S, 1, B, Hkv, D), mk(S, 1, B, Hkv, D)
    runs = []
    for replay in (False, True):
        caches = sqa.LayerCaches([b], [b], B, Hkv, D, dt, DEV, True)
        sqa.prefill_compress(K, V, sc, "h2o", 4, caches, 0)
        ws = sqa.decode_workspace(caches, Hkv * g, "h2o")
        pos = torch.full((B,), P, dtype=torch.int32, device=DEV)
        opts = sqa.batch_opts(new_pos_seq=pos)
        qi, ki, vi = (torch.empty_like(x[0]) for x in (q, k, v))
        out = torch.zeros_like(qi)
        step = lambda: sqa.decode_step(qi, ki, vi, 0, "h2o", 4, caches, out, ws, opts=opts)
        if replay:
            pos.fill_(-1)                                    # (a first step that every sequence sits out)
            step()
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                step()
        snaps = []
        for t in range(S):
            for x, y in ((qi, q), (ki, k), (vi, v)):
                x.copy_(y[t])
            pos.fill_(P + t)
            graph.replay() if replay else step()
            _ = (out.float().sum() + 1).item()
            snaps.append([x.clone() for x in (out, caches.pos[0], caches.score[0], caches.state[0], caches.K[0])])
        assert sqa.read_device_status(ws) == 0
        runs.append(snaps)
    for a, c in zip(*runs):
        assert all(torch.equal(x, y) for x, y in zip(a, c))


@pytest.mark.parametrize("dtype,D,g", [("f32", 64, 1), ("bf16", 128, 1), ("f32", 128, 4), ("bf16", 128, 8)])
def test_one_call_over_layers_and_one_per_layer_agree_to_rounding(sqa, dtype, D, g):
    """132 units per layer: 8 waves each in a call over one layer, 4 in a call over both.  Whole units either way, so only the
    order in which the waves' parts are added differs; the tokens kept are the same (scores that are far apart), and a call
    made twice gives the same bytes."""
    B, Hkv, L, P, S, budgets = 33, 4, 2, 250, 5, [200, 143]
    dt = _dtype(dtype)
    _plan(sqa, budgets, B, g, Hkv, D, dtype, "h2o")
    assert all(sqa.decode_plan([b], [b], B, g * Hkv, Hkv, D, dtype, "h2o")["waves"] == 8 for b in budgets)
    gen = torch.Generator(device=DEV).manual_seed(D + g)
    mk = lambda *shape: torch.randn(*shape, generator=gen, device=DEV).to(dt)
    K, V = [mk(B, Hkv, P, D) for _ in range(L)], [mk(B, Hkv, P, D) for _ in range(L)]
    sc = [torch.argsort(torch.rand(B, Hkv, P, generator=gen, device=DEV), dim=-1).float() for _ in range(L)]
    q, k, v = mk(S, L, B, Hkv * g, D), mk(S, L, B, Hkv, D), mk(S, L, B, Hkv, D)
    runs = []
    for together in (True, True, False):
        caches = sqa.LayerCaches(budgets, budgets, B, Hkv, D, dt, DEV, True)
        sqa.prefill_compress_layers(K, V, sc, "h2o", 4, caches)
        ws = sqa.decode_workspace(caches, Hkv * g, "h2o")
        wl = [sqa.decode_workspace(caches, Hkv * g, "h2o", l, 1) for l in range(L)]
        out = torch.empty_like(q)
        for t in range(S):
            if together:
                sqa.decode_step(q[t], k[t], v[t], P + t, "h2o", 4, caches, out[t], ws)
            else:
                for l in range(L):
                    sqa.decode_step(q[t, l], k[t, l], v[t, l], P + t, "h2o", 4, caches, out[t, l], wl[l], layer0=l, n_layers=1)
        runs.append((out, caches))
    (a, ca), (b, cb), (c, cc) = runs
    assert torch.equal(a, b) and all(torch.equal(x, y) for x, y in zip(ca.score + ca.pos + ca.state, cb.score + cb.pos + cb.state))
    assert rel_err(np64(a), np64(c)) < TOL[dtype]
    for l in range(L):
        assert torch.equal(ca.pos[l], cc.pos[l])
        # each step adds probabilities that are off by a few 1e-6 of themselves in either run (on the matrix cores by the
        # rounding of a bf16 number, 2^-8, relative to one reference or another), and rounds the sum
        rel = 2 * ((2.0 ** -8 if uses_matrix_cores(dtype, D, g) else 1e-5) + S * 2.0 ** -23)
        x, y = np64(ca.score[l]), np64(cc.score[l])
        assert np.all(np.abs(x - y) <= rel * np.abs(x) + 1e-37)
