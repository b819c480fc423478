"""The launch plan of the decode step (sqa_decode_plan: host arithmetic, no GPU): the configurations that
bench.py times and the profiles describe, and invariants over random shapes."""
import ctypes as C

import numpy as np
import pytest

from paper_2404_04793_amd import binding as sqa
from paper_2404_04793_amd import workloads as W

# budgets of the five workloads (their group sizes and the budget rule are pinned in the oracle tests)
BUDGETS = {
    "llama2_7b": [2271, 2271] + [143] * 28 + [2271, 2271],
    "stress_7b": [571, 571] + [35] * 28 + [571, 571],
    "mistral_7b": [1987] * 2 + [1987] * 14 + [368] * 15 + [1987],          # 17 important layers, 15 unimportant
    "llama2_70b": [3439] * 10 + [491] * 27 + [3439] + [491] * 15 + [3439] + [491] * 18 + [3439] * 8,
}


def _plan(name, policy=None, blocked=False, layers=None):
    wl = W.WORKLOADS[name]
    b = BUDGETS[name] if layers is None else [BUDGETS[name][i] for i in layers]
    assert layers is not None or len(b) == wl.L
    caps = [min(x, wl.P + wl.S) for x in b]
    return sqa.decode_plan(b, caps, wl.B, wl.Hq, wl.Hkv, wl.D, "bf16", policy or wl.policy, blocked), b, wl


def test_llama2_7b_launch_is_the_one_the_profile_describes():
    p, b, wl = _plan("llama2_7b")
    units = wl.B * wl.Hkv
    assert p["workgroups"] == 4 * units + 28 * units // 4 == 2816           # whole long units, four short units per workgroup
    assert p["matrix_cores"] == 0 and p["wide_tail"] == 0 and p["table_entries"] == 0
    for lay, x in zip(p["layers"], b):
        assert lay["wave_per_unit"] == (1 if x == 143 else 0)
        assert lay["workgroups_per_unit"] == (0 if x == 143 else 1)         # no unit is split
    assert p["lds_bytes"] == 2304 * 4                                        # the step's logits of one 2271-token unit
    one, _, _ = _plan("llama2_7b", layers=[0])
    assert one["workgroups"] == units and one["wide_tail"] == 1 and one["layers"][0]["workgroups_per_unit"] == 1
    short, _, _ = _plan("llama2_7b", layers=[5])
    assert short["workgroups"] == units and short["layers"][0]["wave_per_unit"] == 0   # 256 units: too few for one wave each


def test_stress_mistral_70b_launches():
    p, b, wl = _plan("stress_7b")
    units = wl.B * wl.Hkv
    assert p["workgroups"] == 4 * units + 28 * units // 4 == 78848
    p, b, wl = _plan("mistral_7b")
    assert p["matrix_cores"] == 1 and p["workgroups"] == 32 * wl.B * wl.Hkv == 8192
    assert all(l["workgroups_per_unit"] == 1 and l["probs_in_lds"] == 0 for l in p["layers"])
    p, b, wl = _plan("llama2_70b")
    assert p["matrix_cores"] == 1 and p["workgroups"] == 80 * wl.B * wl.Hkv == 10240
    # H2O with grouped queries: probabilities stay in LDS where 2 bytes x heads x tokens fit beside the stage buffers
    p, b, _ = _plan("mistral_7b", policy="h2o")
    assert all(l["probs_in_lds"] == 1 for l in p["layers"])
    p, b, _ = _plan("llama2_70b", policy="h2o")
    # (a 3439-token unit keeps what fits -- its leading tiles -- and passes the rest through the workspace)
    assert [l["probs_in_lds"] for l in p["layers"]] == [1 if x == 491 else 2 for x in b]
    assert p["lds_bytes"] <= 160 * 1024 // 3                                  # three workgroups per CU


def test_blocked_allocation_adds_the_staged_table():
    dense, b, _ = _plan("llama2_7b")
    blk, _, _ = _plan("llama2_7b", blocked=True)
    assert blk["table_entries"] == (2271 + 15) // 16
    assert blk["lds_bytes"] == dense["lds_bytes"] + 4 * blk["table_entries"]
    assert blk["workgroups"] == dense["workgroups"]
    small = sqa.decode_plan([35] * 32, [35] * 32, 224, 32, 32, 128, "bf16", "h2o", True)
    assert small["table_entries"] == 4 * (256 // 16) or small["table_entries"] >= 4 * 3   # a row per wave


@pytest.mark.parametrize("seed", range(60))
def test_plan_invariants_on_random_shapes(seed):
    r = np.random.default_rng(seed)
    L = int(r.integers(1, 81))
    Hkv = int(r.choice([1, 2, 4, 8, 32]))
    g = int(r.choice([1, 2, 4, 8]))
    B = int(r.choice([1, 2, 8, 16, 64, 224]))
    D = int(r.choice([64, 128]))
    dtype = str(r.choice(["bf16", "f32"]))
    policy = str(r.choice(["h2o", "sliding", "streaming"]))
    budgets = [int(x) for x in r.choice([8, 35, 143, 368, 571, 2271, 3439, 9000, 40000], size=L)]
    caps = [min(b, int(r.choice([b, b, 300, 5000]))) for b in budgets]
    blocked = bool(r.integers(0, 2)) and max(min(b, c) for b, c in zip(budgets, caps)) <= 16 * 1024
    try:
        p = sqa.decode_plan(budgets, caps, B, g * Hkv, Hkv, D, dtype, policy, blocked)
    except sqa.SqaError as e:
        assert e.code == 6                                                    # only: does not fit (LDS, counters)
        return
    units = B * Hkv
    total = 0
    for lay, b, c in zip(p["layers"], budgets, caps):
        n = min(b, c) + 1                                                     # attend-then-evict attends one more
        assert lay["slots_per_workgroup"] % 64 == 0
        if lay["wave_per_unit"]:
            assert lay["workgroups_per_unit"] == 0 and n <= lay["slots_per_workgroup"] and units * L >= 4096
            total += (units + 3) // 4
        else:
            k = lay["workgroups_per_unit"]
            assert k >= 1 and k * lay["slots_per_workgroup"] >= n > (k - 1) * lay["slots_per_workgroup"]
            total += units * k
        assert not lay["probs_in_lds"] or (p["matrix_cores"] and policy == "h2o")
    assert p["workgroups"] == total
    assert p["lds_bytes"] <= 160 * 1024
    assert p["matrix_cores"] == int(dtype == "bf16" and D == 128 and g >= 4)
    assert p["wide_tail"] == int(total <= 512)
    assert (p["table_entries"] > 0) == blocked
    t = (sqa.LayerCacheStruct * L)()
    for i in range(L):
        t[i].capacity, t[i].budget = caps[i], budgets[i]
    assert p["workspace_bytes"] <= sqa._lib.sqa_decode_workspace_bytes(t, L, B, g * Hkv, Hkv, D, sqa.POLICY[policy])


@pytest.mark.parametrize("dtype,D,g,waves", [("f32", 64, 1, 8), ("f32", 128, 4, 8), ("f32", 128, 8, 4), ("bf16", 64, 2, 8), ("bf16", 64, 8, 4),
                                             ("bf16", 128, 1, 8), ("bf16", 128, 4, 8), ("bf16", 128, 8, 8)])
@pytest.mark.parametrize("policy,blocked", [("h2o", False), ("sliding", True)])
def test_waves_per_workgroup(dtype, D, g, waves, policy, blocked):
    """8 waves where a call has at most 256 workgroups, except under 8 heads off the matrix cores; the number follows from
    the whole call, not from a layer."""
    for B, H, layers, n, expect in ((32, 8, 1, 256, waves), (33, 8, 1, 264, 4), (1, 257, 1, 257, 4), (32, 8, 2, 512, 4), (16, 4, 4, 256, waves),
                                    (1, 1, 1, 1, waves), (64, 64, 2, 2048, 4)):
        p = sqa.decode_plan([143] * layers, [143] * layers, B, g * H, H, D, dtype, policy, blocked)
        assert p["workgroups"] == n and p["waves"] == expect, (B, H, layers)
        assert p["layers"][0]["wave_per_unit"] == int(n == 2048)          # (2 x 4096 units in workgroups of 4)
    # few long units, cut into pieces
    p = sqa.decode_plan([4000], [4000], 2, 8 * g, 8, D, dtype, policy, blocked)
    assert p["layers"][0]["workgroups_per_unit"] > 1 and p["waves"] == (waves if p["workgroups"] <= 256 else 4)
    assert sqa._lib.sqa_decode_plan_waves(None, 1, 1, 1, 1, 64, 0, 0) == 0


@pytest.mark.parametrize("D,budgets,pieces", [(64, [4745, 4785, 4830], [5, 4, 5]), (128, [4300, 4557, 5200], [5, 3, 5])])
def test_cut_does_not_depend_on_where_the_scratch_lies(D, budgets, pieces):
    """96 units, 8 query heads over 1: the finer cut where its scratch fits the static array of sqa_decode_step_static,
    the coarser one where only that fits, the finer one again where neither does (the static call is then refused)."""
    array = 16 * 1024 * 1024 - 1024 * 1024 - 16 * 1024
    for b, n in zip(budgets, pieces):
        p = sqa.decode_plan([b], [b], 12, 64, 8, D, "bf16", "h2o")
        assert p["layers"][0]["workgroups_per_unit"] == n, b
        assert (p["workspace_bytes"] <= array + 4096) == (b != budgets[-1]), (b, p["workspace_bytes"])


@pytest.mark.parametrize("budgets,B,Hq,Hkv,D,dtype,policy,workgroups,pieces", [
    # up to 320 slots a unit stays whole (319 + the new one), from there on it is cut in three (matrix cores: in two)
    ([319], 1, 8, 8, 128, "bf16", "h2o", 8, [1]), ([320], 1, 8, 8, 128, "bf16", "h2o", 24, [3]),
    ([320], 1, 32, 8, 128, "bf16", "h2o", 16, [2]), ([2000, 300], 1, 8, 8, 64, "f32", "sliding", None, [None, 1]),
    # more than two workgroups per CU: not in a heavy kernel with short work items ...
    ([1450] + [529] * 6, 5, 64, 8, 64, "bf16", "h2o", 320, [2] + [1] * 6),
    ([4165] + [988] * 4, 6, 64, 8, 128, "bf16", "sliding", 336, [3] + [1] * 4),
    ([1067] * 3 + [706] * 13, 2, 8, 8, 64, "bf16", "sliding", 304, [2] * 3 + [1] * 13),
    # ... but with long ones, and in the kernels that keep four on a CU
    ([8192] * 5 + [557] * 11, 13, 8, 2, 128, "bf16", "h2o", 676, [3] * 5 + [1] * 11),
    ([8192, 1948, 1948], 9, 16, 8, 128, "bf16", "h2o", 720, [6, 2, 2]),
    ([1543] * 3 + [481] * 3, 13, 8, 2, 128, "f32", "h2o", 702, [7] * 3 + [2] * 3),
    # never more than three
    ([3439] * 2 + [2000] * 14, 4, 32, 8, 128, "f32", "h2o", 576, [2] * 2 + [1] * 14)])
def test_finer_cuts_and_where_they_end(budgets, B, Hq, Hkv, D, dtype, policy, workgroups, pieces):
    p = sqa.decode_plan(budgets, budgets, B, Hq, Hkv, D, dtype, policy)
    assert workgroups is None or p["workgroups"] == workgroups
    got = [l["workgroups_per_unit"] for l in p["layers"]]
    assert all(y is None or x == y for x, y in zip(got, pieces)), got


def test_units_of_more_than_65535_items_are_refused():
    for b, code in ((65535 * 1280 - 1, 0), (65535 * 1280, 6)):                 # (8192 / 8 slots an item and a quarter more)
        t = (sqa.LayerCacheStruct * 1)()
        t[0].capacity = t[0].budget = b
        info = sqa.DecodePlanInfo()
        assert sqa._lib.sqa_decode_plan(t, 1, 1, 8, 1, 64, 1, 2, C.byref(info), None) == code
        assert (sqa._lib.sqa_decode_workspace_bytes(t, 1, 1, 8, 1, 64, 2) > 0) == (code == 0)


def test_plan_argument_errors():
    lib = sqa._lib
    t = (sqa.LayerCacheStruct * 1)()
    t[0].capacity, t[0].budget = 8, 8
    info = sqa.DecodePlanInfo()
    call = lambda **kw: lib.sqa_decode_plan(kw.get("t", t), kw.get("n", 1), kw.get("B", 1), kw.get("Hq", 4), kw.get("Hkv", 4),
                                            kw.get("D", 128), kw.get("dt", 1), kw.get("pol", 2), kw.get("info", C.byref(info)), None)
    assert call() == 0 and info.workgroups == 4
    assert call(t=None) == 1 and call(info=None) == 1
    assert call(dt=4) == 3 and call(pol=9) == 4
    assert call(Hq=6) == 2 and call(D=100) == 2 and call(n=0) == 2 and call(B=0) == 2
    t[0].budget = 0
    assert call() == 5
    t[0].budget, t[0].capacity = 8, 0
    assert call() == 6
