"""GPU parity: the HIP library against the CPU oracle, element by element, on
the same seeded inputs.  Everything here goes through the C ABI (binding.py is
argument marshalling only).  Tolerances: 1e-5 relative for fp32 inputs, 2e-2
for bf16 (per output vector, max|x-ref|/max|ref|); kept indices, lengths and
budgets bit-exact."""
import os

import numpy as np
import pytest
import torch

from oracle import sqa_oracle as O
from oracle import pipeline as OP
from paper_2404_04793_amd import workloads as W
from tests.harness import (TOL, check_scores_after_run, check_step_scores, clustering_margin, export_state, import_state,
                           near_tie_swap, np64, oracle_view, rel_err, round_scores_f32, unit_kv, uses_matrix_cores)

pytestmark = pytest.mark.gpu

DEV = "cuda:0"


@pytest.fixture(scope="module")
def sqa():
    from paper_2404_04793_amd import binding
    return binding


def _cos_rel(c, ref):
    return float(np.max(np.abs(c - ref) / np.maximum(np.abs(ref), 1e-3)))


# ---------------------------------------------------------------- importance

@pytest.mark.parametrize("dtype,L,T,d", [("f32", 4, 256, 256), ("bf16", 3, 1037, 4096), ("bf16", 2, 37, 328),
                                          ("f32", 1, 5, 8), ("bf16", 1, 4099, 512)])
def test_layer_importance(sqa, dtype, L, T, d):
    wl = W.scaled(W.WORKLOADS["tiny"], L=L, hidden=d, dtype=dtype, B=1, P=T)
    hs = [W.hidden_states(wl, l, DEV) for l in range(L)]
    h_in = torch.stack([x[0] for x in hs]).contiguous()
    h_out = torch.stack([x[1] for x in hs]).contiguous()
    cos = sqa.layer_importance(h_in, h_out).cpu().numpy().astype(np.float64)
    ref = O.layer_importance(np64(h_in), np64(h_out))
    assert _cos_rel(cos, ref) < TOL[dtype] if dtype == "f32" else _cos_rel(cos, ref) < 1e-5
    # run-to-run identical bytes
    again = sqa.layer_importance(h_in, h_out).cpu().numpy()
    assert np.array_equal(again.view(np.uint32), cos.astype(np.float32).view(np.uint32))


def test_layer_importance_closed_forms(sqa):
    a = torch.randn(2, 64, 128, device=DEV)
    z = a.clone(); z[0, 3] = 0
    assert np.allclose(sqa.layer_importance(a, a).cpu().numpy(), 1.0, atol=1e-6)
    assert np.allclose(sqa.layer_importance(a, -a).cpu().numpy(), -1.0, atol=1e-6)
    c = sqa.layer_importance(z, a).cpu().numpy()
    assert abs(c[0] - 63 / 64) < 1e-6 and abs(c[1] - 1) < 1e-6          # zero row contributes 0


@pytest.mark.parametrize("dtype,L,T,d,inplace", [("f32", 2, 131, 256, None), ("bf16", 3, 1037, 4096, None),
                                                  ("bf16", 2, 37, 328, "h_in"), ("f32", 1, 67, 520, "attn_out")])
def test_residual_add_importance(sqa, dtype, L, T, d, inplace):
    """The probe fused into the residual add: stored h_out bit for bit, cosine as the stand-alone probe."""
    wl = W.scaled(W.WORKLOADS["tiny"], L=L, hidden=d, dtype=dtype, B=1, P=T)
    hs = [W.hidden_states(wl, l, DEV) for l in range(L)]
    h_in = torch.stack([x[0] for x in hs]).contiguous()
    attn = (torch.stack([x[1] for x in hs]).float() * 0.37).to(h_in.dtype).contiguous()   # any second tensor
    a_host, r_host = h_in.float().cpu().numpy(), attn.float().cpu().numpy()
    want = O.residual_hidden(a_host, r_host, dtype)
    ref = O.layer_importance(a_host.astype(np.float64), want.astype(np.float64))
    h_out = {None: torch.empty_like(h_in), "h_in": h_in, "attn_out": attn}[inplace]
    cos = sqa.residual_add_importance(h_in, attn, h_out).cpu().numpy().astype(np.float64)
    got = h_out.float().cpu().numpy()
    assert np.array_equal(got.view(np.uint32), want.view(np.uint32))
    assert _cos_rel(cos, ref) < 1e-5
    if inplace is None:                      # same stored tensor through the stand-alone probe: same bytes out
        alone = sqa.layer_importance(h_in, h_out).cpu().numpy()
        assert np.array_equal(alone.view(np.uint32), cos.astype(np.float32).view(np.uint32))


@pytest.mark.parametrize("dtype,d", [("f32", 8), ("bf16", 8), ("f32", 128), ("bf16", 256), ("bf16", 264), ("f32", 256), ("bf16", 512),
                                     ("bf16", 520), ("f32", 264)])
@pytest.mark.parametrize("T", [1, 3, 31, 32, 33, 96, 97, 128, 129, 1030])
def test_importance_of_short_rows(sqa, dtype, d, T):
    """Rows of up to 1 KiB share a wave (32 or 64 lanes each), one workgroup's result needs no second kernel: around those
    numbers of rows, pieces per row and workgroups, alone, inside the residual add (in place too) and per sequence.  (The rows
    at which cosines are worked out inside the loop: test_gpu_probe_rows.py.)  fp32 products over at most 520 elements."""
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator().manual_seed(T * 1000 + d)
    a, r = (torch.randn(2, T, d, generator=gen).to(tdt).to(DEV) for _ in range(2))
    h = torch.empty_like(a)
    cos = sqa.residual_add_importance(a, r, h)
    assert torch.equal(h, a + r)
    ref = O.layer_importance(np64(a), np64(h))
    assert _cos_rel(cos.cpu().numpy().astype(np.float64), ref) < 1e-5
    assert torch.equal(cos, sqa.layer_importance(a, h))
    for inplace in ("h_in", "attn_out"):
        x, y = a.clone(), r.clone()
        z = x if inplace == "h_in" else y
        assert torch.equal(cos, sqa.residual_add_importance(x, y, z)) and torch.equal(z, h)
    cut = [0, T // 3, T // 3, T]
    per = sqa.layer_importance_seq(a, h, torch.tensor(cut, dtype=torch.int32, device=DEV)).cpu().numpy().astype(np.float64)
    for i in range(3):
        if cut[i] == cut[i + 1]:
            assert np.all(per[:, i] == 0.0)
        else:
            assert _cos_rel(per[:, i], O.layer_importance(np64(a[:, cut[i]:cut[i + 1]]), np64(h[:, cut[i]:cut[i + 1]]))) < 1e-5


@pytest.mark.parametrize("L,T,d", [(2, 1021, 520), (1, 1025, 520), (1, 4099, 520),    # 256, 257 and 1024 partial sums
                                   (2, 1021, 64), (1, 1025, 128), (1, 4099, 64),      # short rows: 32, 33 and 129 of them
                                   (1, 8192, 128), (1, 8193, 128),                    # ... 256 and 257
                                   (1, 32768, 4096), (2, 16383, 4096)])                # h_out of 256 MiB, and just below
def test_residual_add_importance_store_forms(sqa, L, T, d):
    """Stored sums bit for bit, and the same cosines as the probe of the stored values, around the number of partial
    sums one wave adds up and around the size from which h_out is stored non-temporally."""
    gen = torch.Generator(device=DEV).manual_seed(T)
    a = torch.randn(L, T, d, device=DEV, generator=gen).bfloat16()
    r = torch.randn(L, T, d, device=DEV, generator=gen).bfloat16()
    h = torch.empty_like(a)
    cos = sqa.residual_add_importance(a, r, h)
    assert torch.equal(h, a + r)
    assert torch.equal(cos, sqa.layer_importance(a, h))
    x, y = a[:, :2000].double(), h[:, :2000].double()
    part = sqa.layer_importance(a[:, :2000].contiguous(), h[:, :2000].contiguous()).double()
    want = ((x * y).sum(-1) / (x.norm(dim=-1) * y.norm(dim=-1))).mean(-1)
    assert float((part - want).abs().max()) < 1e-6       # fp32 products over at most 4096 elements, fp64 mean


def test_tiny_budgets_from_gpu_cosines(sqa):
    wl = W.WORKLOADS["tiny"]
    hs = [W.hidden_states(wl, l, DEV) for l in range(wl.L)]
    h_in = torch.stack([x[0] for x in hs]); h_out = torch.stack([x[1] for x in hs])
    cos = sqa.layer_importance(h_in, h_out).cpu().numpy()
    ref = O.layer_importance(np64(h_in), np64(h_out)).astype(np.float32)
    got = sqa.allocate_budgets(cos, wl.total_budget, wl.p)
    want = O.allocate_budgets(ref, wl.total_budget, wl.p)
    assert got[0] == want[0] == [85, 17, 17, 85] and got[1] == want[1]


# ---------------------------------------------------------------- prefill scores

@pytest.mark.parametrize("dtype,B,Hq,Hkv,P,D", [("f32", 1, 2, 2, 100, 64), ("bf16", 2, 4, 2, 193, 128),
                                                 ("f32", 1, 4, 1, 64, 128), ("bf16", 1, 1, 1, 1, 64),
                                                 ("f32", 1, 1, 1, 257, 64),
                                                 # bf16 at D = 128 runs on the matrix cores: ragged and tiny prompts
                                                 ("bf16", 1, 1, 1, 1, 128), ("bf16", 1, 2, 2, 64, 128),
                                                 ("bf16", 1, 4, 1, 65, 128), ("bf16", 2, 8, 2, 300, 128),
                                                 ("bf16", 1, 1, 1, 1000, 128)])
def test_prefill_scores(sqa, dtype, B, Hq, Hkv, P, D):
    wl = W.scaled(W.WORKLOADS["tiny"], L=1, Hq=Hq, Hkv=Hkv, D=D, B=B, P=P, dtype=dtype)
    K, _ = W.prompt_kv(wl, 0, DEV)
    Q = W.prompt_q(wl, 0, DEV)
    got = sqa.prefill_scores(Q, K).cpu().numpy().astype(np.float64)
    Qn, Kn = np64(Q), np64(K)
    g = Hq // Hkv
    for b in range(B):
        for h in range(Hkv):
            ref = O.prefill_scores(Qn[b, h * g:(h + 1) * g], Kn[b, h])
            assert rel_err(got[b, h], ref) < TOL[dtype]
            assert abs(got[b, h].sum() - g * P) < 1e-3 * g * P


def _random_score_cases(n, seed=606):
    r = np.random.default_rng(seed)
    out = []
    for k in range(n):
        dtype = ["bf16", "f32"][int(r.integers(2))]
        D, g = [64, 128][int(r.integers(2))], [1, 2, 4, 8][int(r.integers(4))]
        Hkv, B = int(r.integers(1, 4)), int(r.integers(1, 4))
        P = int(r.choice([1, 2, 15, 16, 17, 31, 33, 63, 64, 65, 127, 128, 129, 200, 255, 257, 384, 500, 777]))
        ragged = bool(r.integers(2))
        plen = [int(r.integers(0, P + 1)) if ragged else P for _ in range(B)]
        out.append(("sc%02d_%s_D%d_g%d_P%d%s" % (k, dtype, D, g, P, "_ragged" if ragged else ""), dtype, D, g, Hkv, B, P, plen,
                    ragged, int(r.integers(3)) == 0))
    return out


# (SQA_RANDOM_CASES=1500 python -m pytest tests/test_gpu_parity.py -m gpu -k random_shapes  runs a longer campaign)
RANDOM_SCORES = _random_score_cases(max(1, int(os.environ.get("SQA_RANDOM_CASES", "28")) // 2))


@pytest.mark.parametrize("case", RANDOM_SCORES, ids=[c[0] for c in RANDOM_SCORES])
def test_prefill_scores_random_shapes(sqa, case):
    """The score producer on seeded random shapes (prompt lengths around its tile sizes, per-sequence lengths down
    to zero, a wider logit range in a third of the cases): two passes, and one pass from the oracle's normalisers."""
    _, dtype, D, g, Hkv, B, P, plen, ragged, wide = case
    wl = W.scaled(W.WORKLOADS["tiny"], L=1, Hq=Hkv * g, Hkv=Hkv, D=D, B=B, P=P, dtype=dtype)
    K, _ = W.prompt_kv(wl, 0, DEV)
    Q = W.prompt_q(wl, 0, DEV)
    if wide:
        K, Q = (K.float() * 3).to(K.dtype), (Q.float() * 2).to(Q.dtype)
    opts = sqa.batch_opts(prompt_len=torch.tensor(plen, dtype=torch.int32, device=DEV)) if ragged else None
    got = sqa.prefill_scores(Q, K, opts=opts).cpu().numpy().astype(np.float64)
    Qn, Kn = np64(Q), np64(K)
    for b in range(B):
        for h in range(Hkv):
            m = plen[b]
            if m:
                ref = O.prefill_scores(Qn[b, h * g:(h + 1) * g, :m], Kn[b, h, :m])
                assert rel_err(got[b, h, :m], ref) < TOL[dtype]
                assert abs(got[b, h, :m].sum() - g * m) < 2e-3 * g * m
            assert np.all(got[b, h, m:] == 0.0)
    if not ragged:
        lse = np.stack([np.stack([O.prefill_row_lse(Qn[b, hq:hq + 1], Kn[b, hq // g])[0] for hq in range(Hkv * g)]) for b in range(B)])
        got2 = sqa.prefill_scores(Q, K, row_lse=torch.tensor(lse, dtype=torch.float32, device=DEV)).cpu().numpy().astype(np.float64)
        for b in range(B):
            for h in range(Hkv):
                assert rel_err(got2[b, h], O.prefill_scores(Qn[b, h * g:(h + 1) * g], Kn[b, h])) < TOL[dtype]


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)])
@pytest.mark.parametrize("P", [129, 191, 193, 320])
def test_prefill_scores_by_query_head_and_by_kv_head(sqa, dtype, D, P):
    """A partial row of column sums per query head and workgroup, added up afterwards; with a workspace of two floats
    per query row fewer of them, or two passes.  Both against the oracle, around the edges of the 64-row stripes and
    tiles, with one key whose logits are -inf (it counts nothing)."""
    g, Hkv, B = 4, 2, 2
    wl = W.scaled(W.WORKLOADS["tiny"], L=1, Hq=Hkv * g, Hkv=Hkv, D=D, B=B, P=P, dtype=dtype)
    K, _ = W.prompt_kv(wl, 0, DEV)
    Q = W.prompt_q(wl, 0, DEV)
    K[:, :, 5, 0], Q[..., 0] = -float("inf"), Q[..., 0].abs() + 0.5
    whole = sqa.prefill_scores(Q, K)
    small = torch.empty_like(whole)
    ws = torch.empty(B * Hkv * g * P * 8, dtype=torch.uint8, device=DEV)
    rc = sqa._lib.sqa_prefill_scores(Q.data_ptr(), K.data_ptr(), 0 if dtype == "f32" else 1, B, Hkv * g, Hkv, P, D,
                                     small.data_ptr(), ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    Qn, Kn = np64(Q), np64(K)
    Kn[:, :, 5, 0] = -1e6                             # (the oracle's logits stay finite; exp gives 0 all the same)
    for got in (whole.cpu().numpy().astype(np.float64), small.cpu().numpy().astype(np.float64)):
        for b in range(B):
            for h in range(Hkv):
                ref = O.prefill_scores(Qn[b, h * g:(h + 1) * g], Kn[b, h])
                assert ref[5] == 0.0 and rel_err(got[b, h], ref) < TOL[dtype]


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)])
def test_prefill_scores_with_runs_of_keys_that_count_nothing(sqa, dtype, D):
    """Logits of -inf for whole groups of 4 and 16 keys, the first that a lane sees of a row among them."""
    g, Hkv, P = 2, 2, 193
    wl = W.scaled(W.WORKLOADS["tiny"], L=1, Hq=Hkv * g, Hkv=Hkv, D=D, B=1, P=P, dtype=dtype)
    K, _ = W.prompt_kv(wl, 0, DEV)
    Q = W.prompt_q(wl, 0, DEV)
    none = torch.zeros(P, dtype=torch.bool, device=DEV)
    none[4:12] = none[16:32] = none[68:72] = True
    K[:, :, none, 0], Q[..., 0] = -float("inf"), Q[..., 0].abs() + 0.5
    got = np64(sqa.prefill_scores(Q, K))[0]
    Kn, off = np64(K)[0], none.cpu().numpy()
    Kn[:, off, 0] = -1e6                              # (the oracle's logits stay finite; exp gives 0 all the same)
    for h in range(Hkv):
        ref = O.prefill_scores(np64(Q)[0, h * g:(h + 1) * g], Kn[h])
        assert np.all(got[h][off] == 0.0) and rel_err(got[h], ref) < TOL[dtype]


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)])
@pytest.mark.parametrize("B,Hkv,g,P,plen", [
    (1, 1, 1, 33, None), (1, 1, 2, 63, [31]), (2, 1, 1, 65, [65, 0]),     # edges of a stripe (32 or 64 rows) and of a block of 16 keys
    (1, 2, 2, 1100, None), (1, 1, 1, 2115, None),                         # few heads: 8 waves; beyond what they keep of a stripe's keys
    (40, 4, 1, 577, [577 - 3 * b for b in range(40)]),                    # many heads: 4 waves, some keys taken twice
    (24, 4, 2, 1040, None)])                                              # ... several stripes per workgroup
def test_prefill_scores_in_one_pass(sqa, dtype, D, B, Hkv, g, P, plen):
    """Stripes of query rows whose exponentials stay in registers: one and several stripes per workgroup, both wave counts,
    prompts longer than what is kept, sequences of other lengths, and a workspace with room for fewer workgroups.  fp32
    arithmetic on exact inputs: a logit's error is below D 2^-24 |q| |k| / sqrt(D) ~ 1e-5, its exponential's the same."""
    gen = torch.Generator(device="cpu").manual_seed(P + B)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K = (torch.randn(B, h, P, D, generator=gen).to(dt).to(DEV) for h in (Hkv * g, Hkv))
    lens = torch.tensor([P] * B if plen is None else plen, dtype=torch.int32, device=DEV)
    opts = None if plen is None else sqa.batch_opts(prompt_len=lens)
    got = np64(sqa.prefill_scores(Q, K, opts=opts))
    small = torch.full((B, Hkv, P), float("nan"), device=DEV)
    ws = torch.empty(B * Hkv * g * P * 2, device=DEV)
    rc = sqa._lib.sqa_prefill_scores_ex(Q.data_ptr(), K.data_ptr(), 0 if dtype == "f32" else 1, B, Hkv * g, Hkv, P, D, small.data_ptr(),
                                        ws.data_ptr(), ws.numel() * 4, torch.cuda.current_stream().cuda_stream, sqa._opts(opts))
    assert rc == 0 and rel_err(np64(small), got) < 1e-6      # (the same terms added in another order)
    for b in sorted({0, B // 2, B - 1}):
        m = P if plen is None else plen[b]
        for h in sorted({0, Hkv - 1}):
            assert np.all(got[b, h, m:] == 0.0)
            if m:
                ref = O.prefill_scores(np64(Q[b, h * g:(h + 1) * g, :m]), np64(K[b, h, :m]))
                assert rel_err(got[b, h, :m], ref) < 1e-5


def _scores_with_workspace(sqa, Q, K, floats, opts=None):
    """prefill_scores with a workspace of that many floats per query row (full of NaN before) -> scores, workspace."""
    B, Hq, P, D = Q.shape
    out = torch.full((B, K.shape[1], P), float("nan"), device=DEV)
    ws = torch.full((floats, B, Hq, P), float("nan"), device=DEV)
    rc = sqa._lib.sqa_prefill_scores_ex(Q.data_ptr(), K.data_ptr(), 0 if Q.dtype == torch.float32 else 1, B, Hq, K.shape[1], P, D,
                                        out.data_ptr(), ws.data_ptr(), ws.numel() * 4, torch.cuda.current_stream().cuda_stream, sqa._opts(opts))
    assert rc == 0
    return np64(out), ws


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)])
@pytest.mark.parametrize("B,Hkv,g,P,plen,floats", [
    (1, 1, 3, 4100, None, 3), (1, 1, 3, 4100, None, 2),     # beyond one pass; second pass per query head, and per KV head
    (1, 2, 1, 4161, None, 3),
    (2, 2, 2, 1930, [1930, 333], 2),                        # few heads, room for two workgroups each: two passes are faster
    (20, 32, 1, 45, [45 - b % 7 for b in range(20)], 3)])   # many short prompts, the larger types in one pass
def test_prefill_scores_in_two_passes(sqa, dtype, D, B, Hkv, g, P, plen, floats):
    """Row statistics, then column sums of exp2(s - m_i) / l_i: around the 64-row tiles, sequences of other lengths, a key whose
    logits are -inf.  That a call went this way shows in its workspace, which then holds the rows' normalisers."""
    gen = torch.Generator(device="cpu").manual_seed(P + B)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K = (torch.randn(B, h, P, D, generator=gen).to(dt).to(DEV) for h in (Hkv * g, Hkv))
    K[:, :, 5, 0], Q[..., 0] = -float("inf"), Q[..., 0].abs() + 0.5
    lens = torch.tensor([P] * B if plen is None else plen, dtype=torch.int32, device=DEV)
    got, ws = _scores_with_workspace(sqa, Q, K, floats, None if plen is None else sqa.batch_opts(prompt_len=lens))
    for b, h in sorted({(0, 0), (B // 2, Hkv // 2), (B - 1, Hkv - 1)}):
        m = P if plen is None else plen[b]
        q, k = np64(Q[b, h * g:(h + 1) * g, :m]), np64(K[b, h, :m])
        k[5, 0] = -1e6                                      # (the oracle's logits stay finite; exp gives 0 all the same)
        if (B, P) != (20, 45) or (dtype, D) in (("bf16", 64), ("f32", 64)):
            stat = np64(ws[0, b, h * g:(h + 1) * g, :m])
            if (dtype, D) != ("bf16", 128):
                stat -= np.log2(np64(ws[1, b, h * g:(h + 1) * g, :m]))
            assert np.abs(stat - O.prefill_row_lse(q, k) / np.log(2.0)).max() < 1e-4
        ref = O.prefill_scores(q, k)
        assert np.all(got[b, h, m:] == 0.0) and got[b, h, 5] == 0.0 and rel_err(got[b, h, :m], ref) < 1e-5


def _scores_us(sqa, Q, K, floats, scores, lse=None):
    """Least time of a prompt-score call with a workspace of that many floats per query row, of 5 series."""
    B, Hq, P, D = Q.shape
    ws = torch.empty(int(B * Hq * P * floats), device=DEV)
    args = (B, Hq, K.shape[1], P, D, scores.data_ptr(), ws.data_ptr(), ws.numel() * 4, torch.cuda.current_stream().cuda_stream, None)
    dt = 0 if Q.dtype == torch.float32 else 1
    def series(n):
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0.record()
        for _ in range(n):
            rc = (sqa._lib.sqa_prefill_scores_ex(Q.data_ptr(), K.data_ptr(), dt, *args) if lse is None else
                  sqa._lib.sqa_prefill_scores_lse(Q.data_ptr(), K.data_ptr(), lse.data_ptr(), dt, *args))
            assert rc == 0
        t1.record()
        torch.cuda.synchronize()
        return t0.elapsed_time(t1) / n * 1e3
    series(3)
    return min(series(10) for _ in range(5))


@pytest.mark.parametrize("B,H,P", [(11, 4, 3817), (23, 2, 3742)])
def test_prefill_scores_more_workspace_is_not_slower(sqa, B, H, P):
    """44 and 46 heads: all workgroups of a KV head run on one of the 8 XCDs, and some have 6 heads, others 5.  A cut that
    counts the rounds over the whole chip puts one more workgroup on the full ones than they have places for (275 against
    214 us), which a smaller workspace, with room for fewer workgroups, is spared."""
    Q, K = (torch.randn(B, H, P, 128, device=DEV).to(torch.bfloat16) for _ in range(2))
    scores = torch.empty(B, H, P, device=DEV)
    room = sqa._lib.sqa_prefill_scores_workspace_bytes(B, H, H, P, 128) // (4 * B * H * P)
    full = _scores_us(sqa, Q, K, room, scores)
    for floats in (5, 8):
        assert full < 1.12 * _scores_us(sqa, Q, K, min(floats, room), scores)


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("H,P", [(16, 2048), (8, 4096)])
def test_prefill_scores_with_a_small_workspace_takes_two_passes(sqa, dtype, D, H, P):
    """Few heads and a workspace of 2 or 3 floats per query row: one pass would have 2 or 3 workgroups per head.  The
    second pass alone (given normalisers) is about half of two passes; one pass in so few workgroups takes 3 to 9 times as long."""
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K = (torch.randn(1, H, P, D, device=DEV).to(dt) for _ in range(2))
    scores = torch.empty(1, H, P, device=DEV)
    half = _scores_us(sqa, Q, K, 3, scores, torch.full((1, H, P), 8.0, device=DEV))
    for floats in (2, 3):
        assert _scores_us(sqa, Q, K, floats, scores) < 2.6 * half


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("bf16", 128)])
@pytest.mark.parametrize("g,P", [(1, 200), (4, 200), (4, 100)])      # column sums per KV head, per query head, per KV head
def test_given_normalisers_in_memory_the_call_writes(sqa, dtype, D, g, P):
    """row_lse handed over in the buffer of the scores, at its start or beyond it, or in the workspace: the same scores."""
    B, Hkv = 2, 2
    rows, outs = B * Hkv * g * P, B * Hkv * P
    gen = torch.Generator(device="cpu").manual_seed(P + g)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K = (torch.randn(B, h, P, D, generator=gen).to(dt).to(DEV) for h in (Hkv * g, Hkv))
    lse = torch.tensor(np.stack([np.stack([O.prefill_row_lse(np64(Q)[b, h:h + 1], np64(K)[b, h // g])[0] for h in range(Hkv * g)])
                                 for b in range(B)]), dtype=torch.float32, device=DEV)
    want = sqa.prefill_scores(Q, K, row_lse=lse).flatten()

    def run(row_lse, out, ws):
        row_lse.copy_(lse.flatten())
        rc = sqa._lib.sqa_prefill_scores_lse(Q.data_ptr(), K.data_ptr(), row_lse.data_ptr(), 0 if dtype == "f32" else 1, B, Hkv * g,
                                             Hkv, P, D, out.data_ptr(), ws.data_ptr(), ws.numel() * 4,
                                             torch.cuda.current_stream().cuda_stream, None)
        assert rc == 0
        return out

    new = lambda n: torch.zeros(n, device=DEV)
    for at in (0, outs // 2, rows - 1):                 # the scores lie within the normalisers, or run out of them
        both = new(rows + outs)
        assert torch.equal(run(both[:rows], both[at:at + outs], new(2 * rows)), want), at
    both = new(rows + outs)
    assert torch.equal(run(both[4:4 + rows], both[:outs], new(2 * rows)), want)
    for at in (0, rows):
        ws = new(3 * rows)
        assert torch.equal(run(ws[at:at + rows], new(outs), ws), want), at
    ws = new(2 * rows)                                  # no room left for sums per query head: the same ones per KV head
    assert rel_err(np64(run(ws[rows // 2:rows // 2 + rows], new(outs), ws)), np64(want)) < 1e-6      # fp32 sums of g * P terms, reordered


def _wide_range_qk(case, P, Hq, Hkv, D):
    """Queries and keys that share one direction u; the keys' component along u sets the logit level."""
    r = torch.Generator().manual_seed({"steps_up": 11, "late_peak": 12, "steps_down": 13}[case])
    u = torch.randn(D, generator=r)
    u = u / u.norm() * D ** 0.5
    pos = torch.arange(P)
    if case == "steps_up":                       # + 24 units (log2) every 40 keys
        a = (pos // 40) * 0.5
    elif case == "steps_down":
        a = ((P - 1 - pos) // 40) * 0.5
    else:                                        # one key 290 units above the rest
        a = torch.zeros(P)
        a[200] = 6.0
    Q = torch.randn(1, Hq, P, D, generator=r) + 3.0 * u
    K = torch.randn(1, Hkv, P, D, generator=r) + a[None, None, :, None] * u
    return Q.to(torch.bfloat16), K.to(torch.bfloat16)


@pytest.mark.parametrize("case", ["steps_up", "late_peak", "steps_down"])
def test_prefill_scores_wide_logit_range(sqa, case):
    """Logits that move by hundreds of units along a row: a level that steps up every 40 keys keeps
    exceeding a row's running reference, one dominant key exceeds it once by far, a falling level never
    does.  (The matrix-core kernels take their exponentials against a reference that only moves when a
    partial sum shows it is far too low.)"""
    Hq, Hkv, P, D = 4, 2, 600, 128
    Q, K = _wide_range_qk(case, P, Hq, Hkv, D)
    Q, K = Q.to(DEV), K.to(DEV)
    got = sqa.prefill_scores(Q, K).cpu().numpy().astype(np.float64)
    assert np.all(np.isfinite(got))
    Qn, Kn = np64(Q), np64(K)
    g = Hq // Hkv
    for h in range(Hkv):
        ref = O.prefill_scores(Qn[0, h * g:(h + 1) * g], Kn[0, h])
        assert rel_err(got[0, h], ref) < TOL["bf16"]
        assert abs(got[0, h].sum() - g * P) < 1e-3 * g * P


@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128)])
@pytest.mark.parametrize("case", ["steps_up", "late_peak", "steps_down"])
def test_prefill_scores_wide_logit_range_in_two_passes(sqa, case, dtype, D):
    """The same beyond 4096 tokens.  Logits reach 5000 in the exp2 domain, where fp32 holds them to 5e-4: so far may an
    exponential be off."""
    P = 4110
    Q, K = (x.to(torch.float32 if dtype == "f32" else torch.bfloat16).to(DEV) for x in _wide_range_qk(case, P, 2, 1, D))
    got, ws = _scores_with_workspace(sqa, Q, K, 3)
    Qn, Kn = np64(Q)[0], np64(K)[0, 0]
    assert np.all(np.isfinite(got)) and rel_err(got[0, 0], O.prefill_scores(Qn, Kn)) < 2e-3
    stat = np64(ws[0, 0]) - (0.0 if (dtype, D) == ("bf16", 128) else np.log2(np64(ws[1, 0])))
    assert np.abs(stat - O.prefill_row_lse(Qn, Kn) / np.log(2.0)).max() < 2e-3


# ---------------------------------------------------------------- prefill compress

def _mk_caches(sqa, budgets, caps, B, Hkv, D, dtype, h2o=True, blocked=False):
    """blocked: K and V as pools of 16-row blocks dealt to the units in a seeded random order (block table)."""
    return sqa.LayerCaches(budgets, caps, B, Hkv, D, torch.float32 if dtype == "f32" else torch.bfloat16, DEV, h2o,
                           blocked=blocked, block_seed=sum(budgets))


@pytest.mark.parametrize("blocked", [False, True], ids=["dense", "blocked"])
@pytest.mark.parametrize("policy", ["sliding", "streaming", "h2o"])
@pytest.mark.parametrize("dtype,B,Hkv,P,D,b", [("f32", 1, 2, 256, 64, 51), ("bf16", 2, 3, 700, 128, 143),
                                                ("bf16", 1, 1, 64, 128, 64), ("f32", 1, 1, 40, 128, 100),
                                                ("bf16", 1, 2, 1031, 64, 6), ("bf16", 1, 1, 513, 128, 512)])
def test_prefill_compress(sqa, policy, dtype, B, Hkv, P, D, b, blocked):
    wl = W.scaled(W.WORKLOADS["tiny"], L=1, Hq=Hkv, Hkv=Hkv, D=D, B=B, P=P, dtype=dtype)
    K, V = W.prompt_kv(wl, 0, DEV)
    r = np.random.default_rng(P + b)
    sc = r.random((B, Hkv, P)).astype(np.float32)
    sc[:, :, r.integers(0, P, size=P // 3)] = 0.25          # many exact ties
    sc[:, :, r.integers(0, P, size=5)] = 0.0
    scores = torch.from_numpy(sc).to(DEV)
    caches = _mk_caches(sqa, [b], [max(min(P, b), 1) + 1], B, Hkv, D, dtype, blocked=blocked)
    sqa.prefill_compress(K, V, scores if policy == "h2o" else None, policy, 4, caches, 0)
    kept = sqa.kept_idx_sorted(caches, 0).cpu().numpy()
    Kn, Vn = np64(K), np64(V)
    for bi in range(B):
        for h in range(Hkv):
            want = O.prefill_compress(Kn[bi, h], Vn[bi, h], sc[bi, h].astype(np.float64), b, policy, 4)
            n = len(want["pos"])
            assert int(caches.lens[0][bi, h]) == n and int(caches.head[0][bi, h]) == 0
            assert kept[bi, h, :n].tolist() == want["pos"].tolist() and np.all(kept[bi, h, n:] == -1)
            got = export_state(caches, 0, bi, h)
            assert caches.pos[0][bi, h, :n].cpu().tolist() == want["pos"].tolist()   # ascending slots
            assert np.array_equal(got["K"], want["K"]) and np.array_equal(got["V"], want["V"])
            if policy == "h2o":
                assert np.array_equal(got["score"], want["score"])


@pytest.mark.parametrize("blocked", [False, True], ids=["dense", "blocked"])
@pytest.mark.parametrize("dtype,D,P,budgets", [("bf16", 128, 1400, [100, 1287, 1399]), ("f32", 64, 2305, [641, 2304, 3000]),
                                               ("f32", 128, 1100, [33, 64, 65]), ("bf16", 64, 17000, [1031, 6]),
                                               # 384 units in one launch, between one and two per CU: shared out for the
                                               # two long layers, and (lengths alike) not at all
                                               ("bf16", 128, 400, [8] * 30 + [390] * 2), ("bf16", 64, 400, [150] * 32)])
def test_prefill_compress_units_shared_out(sqa, dtype, D, P, budgets, blocked):
    """Few units, so that several workgroups copy a unit's rows (shares with and without remainders, more workgroups
    than a share needs), and more than 1024 candidates with many equal scores (each thread lists a run of
    positions), below and above the number whose scores are staged; sequences of different length and budget."""
    B, Hkv = (2, 2) if len(budgets) < 10 else (6, 2)
    n = len(budgets)
    gen = torch.Generator(device="cpu").manual_seed(P)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    plen = [P, P - P // 3, 1, P, P, P][:B]
    bseq = [[b, max(2, b // 2), 2, b, b, b][:B] for b in budgets]
    Ks = [torch.randn(B, Hkv, P, D, generator=gen).to(dt).to(DEV) for _ in range(n)]
    Vs = [torch.randn(B, Hkv, P, D, generator=gen).to(dt).to(DEV) for _ in range(n)]
    Ss = [(torch.randint(0, 40, (B, Hkv, P), generator=gen).float() / 16).to(DEV) for _ in range(n)]
    i32 = lambda x: torch.tensor(x, dtype=torch.int32, device=DEV)
    status, pl, bs = i32([0]), i32(plen), i32(bseq)
    for opts in (None, sqa.batch_opts(prompt_len=pl, budget_seq=bs, status=status)):
        caches = _mk_caches(sqa, budgets, [min(P, b) for b in budgets], B, Hkv, D, dtype, blocked=blocked)
        sqa.prefill_compress_layers(Ks, Vs, Ss, "h2o", 4, caches, opts=opts)
        for l in (range(n) if n < 10 else (0, n - 2, n - 1)):
            for b in range(B):
                p, bud = (P, budgets[l]) if opts is None else (plen[b], bseq[l][b])
                for h in range(Hkv):
                    want = O.prefill_compress(np64(Ks[l])[b, h, :p], np64(Vs[l])[b, h, :p], np64(Ss[l])[b, h, :p], bud, "h2o", 4)
                    got = export_state(caches, l, b, h)
                    assert got["pos"].tolist() == want["pos"].tolist(), (l, b, h)
                    assert all(np.array_equal(got[f], want[f]) for f in ("K", "V", "score")), (l, b, h)
                    assert caches.state[l][b, h].tolist() == [len(want["pos"]), 0, -2, 0]
    assert int(status) == 0


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("B,b", [(64, 127), (64, 128), (63, 127)])     # 2048 units on both sides of 128 rows, and 2016
def test_prefill_compress_of_many_short_units(sqa, dtype, D, B, b):
    Hkv, P = 32, 300
    gen = torch.Generator(device=DEV).manual_seed(b)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    K, V = (torch.randn(B, Hkv, P, D, generator=gen, device=DEV).to(dt) for _ in range(2))
    sc = torch.randint(0, 40, (B, Hkv, P), generator=gen, device=DEV).float() / 16
    caches = _mk_caches(sqa, [b], [b], B, Hkv, D, dtype)
    sqa.prefill_compress(K, V, sc, "h2o", 4, caches, 0)
    assert bool((caches.state[0].view(-1, 4) == torch.tensor([b, 0, -2, 0], dtype=torch.int32, device=DEV)).all())
    for x, h in ((0, 0), (1, 31), (B // 2, 7), (B - 1, 31)):
        want = O.prefill_compress(np64(K)[x, h], np64(V)[x, h], np64(sc)[x, h], b, "h2o", 4)
        got = export_state(caches, 0, x, h)
        assert got["pos"].tolist() == want["pos"].tolist(), (x, h)
        assert all(np.array_equal(got[f], want[f]) for f in ("K", "V", "score")), (x, h)


@pytest.mark.parametrize("dtype,D", [("bf16", 128), ("f32", 64)])
@pytest.mark.parametrize("policy,units,P,b,blocked", [("h2o", 6, 500, 211, True),           # stores: a pool of 320 MiB, little of it written
                                                      ("sliding", 1100, 70, 33, True),       # ... in many short units
                                                      ("h2o", 80, 4096, 4100, False)])       # stores and loads: 320 MiB left, twice that moved
def test_prefill_compress_into_caches_beyond_the_infinity_cache(sqa, dtype, D, policy, units, P, b, blocked):
    """Calls over caches of 320 MiB and more (in blocks: pools; dense: the rows that the call leaves) store rows
    non-temporally, and launches that move 256 MiB read them so too: the same rows, scores and positions as in a pool just below
    that size, or with a call per layer."""
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device=DEV).manual_seed(units)
    L = 2
    Ks, Vs = ([torch.randn(units, 1, P, D, device=DEV, generator=gen).to(tdt) for _ in range(L)] for _ in range(2))
    Ss = [torch.rand(units, 1, P, device=DEV, generator=gen) for _ in range(L)]
    limit = (320 << 20) // (L * 2 * D * Ks[0].element_size())          # slots of a layer
    got = []
    for big in (False, True):
        if blocked:
            own = units * ((b + 15) // 16)
            caches = sqa.LayerCaches([b] * L, [b] * L, units, 1, D, tdt, DEV, True, blocked=True,
                                     spare_blocks=(limit // 16 if big else min(limit // 16 - 1, own + 3)) - own)
        else:
            assert units * min(P, b) >= limit
            caches = sqa.LayerCaches([b] * L, [P] * L, units, 1, D, tdt, DEV, True)
        if blocked or big:
            sqa.prefill_compress_layers(Ks, Vs, Ss, policy, 4, caches)
        else:
            for l in range(L):
                sqa.prefill_compress_layers(Ks[l:l + 1], Vs[l:l + 1], Ss[l:l + 1], policy, 4, caches, layer0=l)
        n = min(P, b)
        rows = [unit_kv(caches, l, u, 0, n) for l in range(L) for u in (0, units // 2, units - 1)]
        got.append((rows, [[x[l].view(units, -1)[:, :n].cpu() for x in (caches.pos, caches.score)] for l in range(L)],
                    [s.cpu() for s in caches.state]))
    for (k0, v0), (k1, v1) in zip(got[0][0], got[1][0]):
        assert np.array_equal(k0, k1) and np.array_equal(v0, v1)
    for x, y in zip(got[0][1], got[1][1]):
        assert torch.equal(x[0], y[0]) and torch.equal(x[1], y[1])
    for x, y in zip(got[0][2], got[1][2]):
        assert torch.equal(x, y)
    keep = O.select_keep(np.arange(P), Ss[1][units - 1, 0].cpu().numpy(), b, policy)
    assert np.array_equal(np.sort(got[1][1][1][0][units - 1].numpy()), np.sort(keep))
    assert np.array_equal(got[1][0][-1][0], np64(Ks[1][units - 1, 0])[got[1][1][1][0][units - 1].numpy()])


def test_prefill_compress_layers_matches_single_layer_calls(sqa):
    """One launch over 35 layers with different budgets (two batches of kernel arguments) == 35 calls."""
    B, Hkv, P, D, L = 2, 2, 300, 128, 35
    r = np.random.default_rng(5)
    budgets = [int(x) for x in r.integers(2, 340, size=L)]
    Ks = [torch.randn(B, Hkv, P, D, device=DEV).to(torch.bfloat16) for _ in range(L)]
    Vs = [torch.randn(B, Hkv, P, D, device=DEV).to(torch.bfloat16) for _ in range(L)]
    Ss = [torch.rand(B, Hkv, P, device=DEV) for _ in range(L)]
    caps = [min(b, P) for b in budgets]
    a = _mk_caches(sqa, budgets, caps, B, Hkv, D, "bf16")
    b = _mk_caches(sqa, budgets, caps, B, Hkv, D, "bf16")
    sqa.prefill_compress_layers(Ks, Vs, Ss, "h2o", 4, a)
    for l in range(L):
        sqa.prefill_compress(Ks[l], Vs[l], Ss[l], "h2o", 4, b, l)
    for l in range(L):
        assert torch.equal(a.pos[l], b.pos[l]) and torch.equal(a.lens[l], b.lens[l])
        assert torch.equal(a.K[l].view(torch.int16), b.K[l].view(torch.int16))
        assert torch.equal(a.V[l].view(torch.int16), b.V[l].view(torch.int16))
        assert torch.equal(a.score[l], b.score[l]) and bool((a.hint[l] == -2).all())


def _score_bits(kind, n, r):
    """Non-negative fp32 scores given by their bit patterns, which the selection works on."""
    one = 0x3f800000
    if kind == "equal":
        bits = np.full(n, one)
    elif kind == "two":
        bits = one + r.integers(0, 2, n)
    elif kind.startswith("range"):                     # that many different patterns, next to each other
        bits = one + r.integers(0, int(kind[5:]), n)
    elif kind == "wide":                               # from 0 and the smallest denormal to +inf
        bits = r.choice(np.array([0, 1, 2, 0x007fffff, 0x00800000, one, 0x7f7fffff, 0x7f800000]), n)
    elif kind == "steps":                              # a few values many octaves apart, one of them crowded
        bits = np.where(r.random(n) < 0.7, one, r.choice(np.array([one - (20 << 23), one + 1, one + (9 << 23)]), n))
    else:
        return r.exponential(size=n).astype(np.float32)
    return bits.astype(np.uint32).view(np.float32)


@pytest.mark.parametrize("P,b", [(300, 3), (300, 180), (1500, 700)])
@pytest.mark.parametrize("kind", ["equal", "two", "range255", "range256", "range257", "range300", "range5000", "range70000", "wide", "steps",
                                  "exponential"])
def test_prefill_compress_selection_of_close_and_far_scores(sqa, kind, P, b):
    """Bins over the range the keys have: ranges around the number of bins and its square, bins that are taken whole,
    equal scores (the earlier position is kept).  Bit for bit."""
    B, Hkv, D = 1, 3, 64
    r = np.random.default_rng(P + b + len(kind))
    K = torch.randn(B, Hkv, P, D, device=DEV).to(torch.bfloat16)
    sc = np.stack([_score_bits(kind, P, r) for _ in range(Hkv)])[None]
    caches = _mk_caches(sqa, [b], [b], B, Hkv, D, "bf16")
    sqa.prefill_compress(K, K, torch.from_numpy(sc).to(DEV), "h2o", 4, caches, 0)
    for h in range(Hkv):
        keep = O.select_keep(np.arange(P), sc[0, h].astype(np.float64), b, "h2o")
        assert caches.pos[0][0, h, :b].cpu().tolist() == keep.tolist()
        assert torch.equal(caches.score[0][0, h, :b].cpu(), torch.from_numpy(sc[0, h][keep]))


def test_prefill_compress_large_prompt_h2o_global_keys(sqa):
    """More candidates than the LDS staging limit: the select reads scores from memory."""
    B, Hkv, P, D, b = 1, 1, 20000, 64, 300
    K = torch.randn(B, Hkv, P, D, device=DEV).to(torch.bfloat16); V = K.clone()
    sc = np.random.default_rng(1).integers(0, 50, size=(B, Hkv, P)).astype(np.float32) / 8
    caches = _mk_caches(sqa, [b], [b], B, Hkv, D, "bf16")
    sqa.prefill_compress(K, V, torch.from_numpy(sc).to(DEV), "h2o", 4, caches, 0)
    keep = O.select_keep(np.arange(P), sc[0, 0].astype(np.float64), b, "h2o")
    assert caches.pos[0][0, 0, :b].cpu().tolist() == keep.tolist()


@pytest.mark.parametrize("dtype,D,g,P", [("bf16", 128, 1, 300), ("bf16", 128, 4, 257), ("f32", 64, 2, 130), ("bf16", 64, 1, 90),
                                         ("f32", 128, 1, 64)])
def test_prefill_scores_from_given_row_normalisers(sqa, dtype, D, g, P):
    """sqa_prefill_scores_lse: one pass over the logits with the caller's ln-normalisers (as a fused attention
    kernel returns them) against the oracle fed the same numbers, and against the two-pass call."""
    B, Hkv = 2, 2
    wl = W.scaled(W.WORKLOADS["tiny"], L=1, Hq=Hkv * g, Hkv=Hkv, D=D, B=B, P=P, dtype=dtype)
    K, _ = W.prompt_kv(wl, 0, DEV)
    Q = W.prompt_q(wl, 0, DEV)
    Qn, Kn = np64(Q), np64(K)
    lse = np.stack([np.concatenate([O.prefill_row_lse(Qn[b, h * g:(h + 1) * g], Kn[b, h]) for h in range(Hkv)]) for b in range(B)])
    lse32 = torch.from_numpy(lse.astype(np.float32)).to(DEV).contiguous()                 # [B, Hq, P]
    got = sqa.prefill_scores(Q, K, row_lse=lse32).cpu().numpy().astype(np.float64)
    two_pass = sqa.prefill_scores(Q, K).cpu().numpy().astype(np.float64)
    for b in range(B):
        for h in range(Hkv):
            ref = O.prefill_scores_from_lse(Qn[b, h * g:(h + 1) * g], Kn[b, h], np64(lse32)[b, h * g:(h + 1) * g])
            assert rel_err(got[b, h], ref) < TOL[dtype], (b, h)
            # element by element: every column is a sum of positive terms, each known to ~1e-5 relative
            assert np.max(np.abs(got[b, h] - ref) / ref) < 1e-4, (b, h)
            assert rel_err(got[b, h], two_pass[b, h]) < 1e-4
    # ragged: queries beyond a sequence's own prompt are not counted
    plen = torch.tensor([P, max(P // 3, 1)], dtype=torch.int32, device=DEV)
    rag = sqa.prefill_scores(Q, K, row_lse=lse32, opts=sqa.batch_opts(prompt_len=plen)).cpu().numpy().astype(np.float64)
    n = int(plen[1])
    ref = O.prefill_scores_from_lse(Qn[1, :g, :n], Kn[1, 0, :n], np64(lse32)[1, :g, :n])
    assert rel_err(rag[1, 0, :n], ref) < TOL[dtype] and np.all(rag[1, 0, n:] == 0.0)


# ---------------------------------------------------------------- decode step, teacher forced

def _unit_inputs(wl, layer, u_dirs, mask):
    K, V = W.prompt_kv(wl, layer, DEV, u_dirs, mask)
    Q = W.prompt_q(wl, layer, DEV, u_dirs)
    q, k, v = W.decode_qkv(wl, layer, DEV, u_dirs, mask)
    return K, V, Q, q, k, v


CASES = [
    # name, dtype, L, Hq, Hkv, D, B, P, S, policy, budgets
    ("h2o_f32_mha", "f32", 2, 2, 2, 64, 1, 40, 12, "h2o", [9, 46]),
    ("h2o_bf16_mha_ragged", "bf16", 2, 3, 3, 128, 2, 150, 10, "h2o", [37, 155]),
    ("h2o_bf16_gqa2", "bf16", 1, 4, 2, 128, 1, 70, 8, "h2o", [21]),
    ("stream_bf16_gqa4", "bf16", 2, 8, 2, 128, 2, 90, 9, "streaming", [13, 95]),
    ("slide_bf16_gqa8", "bf16", 2, 8, 1, 128, 1, 300, 7, "sliding", [67, 303]),
    ("slide_f32_d128", "f32", 1, 2, 2, 128, 1, 33, 6, "sliding", [5]),
    ("stream_f32_d64_gqa2", "f32", 1, 4, 2, 64, 1, 50, 6, "streaming", [11]),
    ("h2o_bf16_d64", "bf16", 1, 2, 2, 64, 1, 80, 6, "h2o", [2]),
    # budgets above the chunk size: units are split over several workgroups
    ("h2o_bf16_split", "bf16", 2, 2, 2, 128, 2, 600, 6, "h2o", [603, 41]),
    ("h2o_f32_split_gqa2", "f32", 1, 4, 2, 64, 1, 420, 5, "h2o", [400]),
    ("stream_bf16_split_gqa4", "bf16", 1, 4, 1, 128, 1, 900, 4, "streaming", [777]),
    # grouped queries in bf16 at D = 128 run on the matrix cores: with H2O logits, ragged tiles, split units
    ("h2o_bf16_gqa8_mfma", "bf16", 2, 16, 2, 128, 2, 200, 8, "h2o", [61, 205]),
    ("stream_bf16_gqa8_mfma_split", "bf16", 1, 8, 1, 128, 1, 900, 4, "streaming", [777]),
    ("h2o_bf16_gqa8_mfma_split", "bf16", 1, 8, 1, 128, 1, 700, 5, "h2o", [650]),
    ("slide_bf16_gqa8_mfma_tiny", "bf16", 1, 16, 2, 128, 1, 40, 6, "sliding", [3]),
    # as many layers in one call as the library takes (SQA_MAX_LAYERS)
    ("h2o_f32_128_layers", "f32", 128, 1, 1, 64, 1, 12, 3, "h2o", [5, 9, 14, 3] * 32),
]


def _random_cases(n, seed=2024):
    """Seeded random shapes: every dtype / head-dim / group size the library has a kernel for, budgets
    below, at and above the prompt length, around multiples of the 64-row tile and of the 256-slot chunk."""
    r = np.random.default_rng(seed)
    out = []
    for i in range(n):
        dtype = ["f32", "bf16"][int(r.integers(2))]
        D = [64, 128][int(r.integers(2))]
        g = [1, 2, 4, 8][int(r.integers(4))]
        Hkv = int(r.integers(1, 4))
        B = int(r.integers(1, 3))
        L = int(r.integers(1, 4))
        P = int(r.choice([3, 17, 63, 64, 65, 130, 255, 256, 257, 400, 513]))
        S = int(r.integers(2, 6))
        policy = ["sliding", "streaming", "h2o"][int(r.integers(3))]
        lo = {"sliding": 1, "streaming": 5, "h2o": 2}[policy]
        budgets = []
        for _ in range(L):
            kind = int(r.integers(4))
            b = [int(r.integers(lo, max(lo + 1, P))), P, P + int(r.integers(1, S + 3)), int(r.integers(lo, lo + 6))][kind]
            budgets.append(max(lo, b))
        out.append(("rand%02d_%s_%s_D%d_g%d" % (i, policy, dtype, D, g), dtype, L, Hkv * g, Hkv, D, B, P, S, policy, budgets))
    return out


# (SQA_RANDOM_CASES=1500 python -m pytest tests/test_gpu_parity.py -m gpu -k teacher_forced  runs a longer campaign)
RANDOM_CASES = _random_cases(int(os.environ.get("SQA_RANDOM_CASES", "28")))


@pytest.mark.parametrize("case", CASES + RANDOM_CASES, ids=[c[0] for c in CASES + RANDOM_CASES])
def test_decode_teacher_forced(sqa, case):
    _teacher_forced(sqa, case, "evict_then_attend")


AE_CASES = [c for c in CASES if c[0] not in ("slide_f32_d128", "stream_f32_d64_gqa2")] + _random_cases(10, seed=77)


@pytest.mark.parametrize("case", AE_CASES, ids=[c[0] for c in AE_CASES])
def test_decode_teacher_forced_attend_then_evict(sqa, case):
    """The other order of a step: attention over all len+1 tokens, accumulation, then the eviction."""
    _teacher_forced(sqa, case, "attend_then_evict")


BLOCKED_CASES = CASES + _random_cases(8, seed=4711)


@pytest.mark.parametrize("order", ["evict_then_attend", "attend_then_evict"])
@pytest.mark.parametrize("case", BLOCKED_CASES, ids=[c[0] for c in BLOCKED_CASES])
def test_decode_teacher_forced_blocked_allocation(sqa, case, order):
    """The same steps with K and V in pools of 16-row blocks that a per-unit table row names, dealt out in a
    seeded random order: no unit is contiguous, neighbouring blocks belong to other units."""
    _teacher_forced(sqa, case, order, blocked=True)


SPARE_CASES = [
    # budgets that are multiples of the 16-row block, caches with more slots than the budget: a full unit's new
    # token under attend-then-evict has index `budget`, the first slot of a block the unit never uses
    ("h2o_bf16_gqa4_mfma_spare", "bf16", 2, 8, 2, 128, 2, 100, 6, "h2o", [64, 32]),
    ("h2o_bf16_mha_spare", "bf16", 1, 2, 2, 128, 2, 100, 6, "h2o", [48]),
    ("slide_bf16_gqa8_mfma_spare", "bf16", 1, 8, 1, 128, 2, 100, 6, "sliding", [80]),
    ("stream_f32_spare", "f32", 1, 2, 2, 64, 1, 60, 6, "streaming", [16]),
]


@pytest.mark.parametrize("blocked", [True, False], ids=["blocked", "dense"])
@pytest.mark.parametrize("order", ["evict_then_attend", "attend_then_evict"])
@pytest.mark.parametrize("case", SPARE_CASES, ids=[c[0] for c in SPARE_CASES])
def test_decode_capacity_above_budget(sqa, case, order, blocked):
    """Caches allocated with 24 more slots per unit than the budget: nothing beyond the budget's slots (and,
    with blocks, beyond the table entries they need) is ever touched."""
    _teacher_forced(sqa, case, order, blocked=blocked, spare_slots=24)


def test_decode_reports_a_block_number_outside_the_pools(sqa):
    """A table entry beyond the pools: the unit is left untouched, its out rows zeroed, SQA_ERR_SHAPE in the
    status word; the other unit of the call steps normally.  Prompt compression reports the same."""
    B, Hkv, D, b, P = 2, 1, 64, 40, 50
    caches = _mk_caches(sqa, [b], [b], B, Hkv, D, "f32", blocked=True)
    K = torch.randn(B, Hkv, P, D, device=DEV); V = torch.randn(B, Hkv, P, D, device=DEV); sc = torch.rand(B, Hkv, P, device=DEV)
    sqa.prefill_compress(K, V, sc, "h2o", 4, caches, 0)
    good = caches.block_table[0].clone()
    before = caches.pos[0][1, 0, :b].sort().values.cpu().tolist()      # (positions are dense: no look-up through the table)
    caches.block_table[0][1, 1] = caches.K[0].shape[0]                 # one past the last block, in unit 1
    q = torch.randn(1, B, Hkv, D, device=DEV); out = torch.full_like(q, 3.0)
    ws = sqa.decode_workspace(caches, Hkv, "h2o")
    sqa.decode_step(q, q, q, P, "h2o", 4, caches, out, ws)
    assert sqa.read_device_status(ws) == 2                             # SQA_ERR_SHAPE
    assert bool((out[0, 1] == 0).all()) and not bool((out[0, 0] == 0).any())
    assert int(caches.lens[0][1, 0]) == b and caches.pos[0][1, 0, :b].sort().values.cpu().tolist() == before
    assert int(caches.pos[0][0, 0].max()) == P                         # unit 0 took the step
    status = torch.zeros(1, dtype=torch.int32, device=DEV)
    sqa.prefill_compress_layers([K], [V], [sc], "h2o", 4, caches, opts=sqa.batch_opts(status=status))
    assert int(status.item()) == 2 and caches.lens[0][:, 0].tolist() == [b, 0]
    caches.block_table[0].copy_(good)


def _teacher_forced(sqa, case, order, blocked=False, spare_slots=0):
    name, dtype, L, Hq, Hkv, D, B, P, S, policy, budgets = case
    ae = order == "attend_then_evict"
    opts = sqa.batch_opts(order=order) if ae else None
    wl = W.scaled(W.WORKLOADS["tiny"], L=L, Hq=Hq, Hkv=Hkv, D=D, B=B, P=P, S=S, dtype=dtype, policy=policy)
    g = Hq // Hkv
    u_dirs, mask = W.unit_dirs(wl), W.hh_mask(wl, DEV)
    inp = [_unit_inputs(wl, l, u_dirs, mask) for l in range(L)]
    caps = [min(b, P + S) + spare_slots for b in budgets]
    caches = _mk_caches(sqa, budgets, caps, B, Hkv, D, dtype, blocked=blocked)
    ws = sqa.decode_workspace(caches, Hq, policy)
    # oracle trajectories (fp32-rounded score storage between steps)
    state = {}
    for l in range(L):
        Kn, Vn, Qn = np64(inp[l][0]), np64(inp[l][1]), np64(inp[l][2])
        for b in range(B):
            for h in range(Hkv):
                s0 = O.prefill_scores(Qn[b, h * g:(h + 1) * g], Kn[b, h]).astype(np.float32).astype(np.float64)
                state[l, b, h] = O.prefill_compress(Kn[b, h], Vn[b, h], s0, budgets[l], policy, wl.n_sink)
    q_all = torch.stack([inp[l][3] for l in range(L)], 1).contiguous()      # [S, L, B, Hq, D]
    k_all = torch.stack([inp[l][4] for l in range(L)], 1).contiguous()
    v_all = torch.stack([inp[l][5] for l in range(L)], 1).contiguous()
    qn, kn, vn = np64(q_all), np64(k_all), np64(v_all)
    out = torch.empty(L, B, Hq, D, dtype=wl.torch_dtype, device=DEV)
    worst, worst_sc = 0.0, 0.0
    mc = uses_matrix_cores(dtype, D, g)
    for t in range(S):
        for key, c in state.items():
            import_state(caches, key[0], key[1], key[2], c)
        sqa.decode_step(q_all[t], k_all[t], v_all[t], P + t, policy, wl.n_sink, caches, out, ws, opts=opts)
        assert sqa.read_device_status(ws) == 0
        o = np64(out)
        for (l, b, h), c in state.items():
            want_out, c2 = O.decode_step(c, qn[t, l, b, h * g:(h + 1) * g], kn[t, l, b, h], vn[t, l, b, h],
                                         P + t, budgets[l], policy, wl.n_sink, order)
            got = export_state(caches, l, b, h)
            worst = max(worst, rel_err(o[l, b, h * g:(h + 1) * g], want_out))
            if ae and policy == "h2o" and got["pos"].tolist() != c2["pos"].tolist():
                _, full = O.decode_step(c, qn[t, l, b, h * g:(h + 1) * g], kn[t, l, b, h], vn[t, l, b, h],
                                        P + t, 1 << 30, policy, wl.n_sink, order)       # nothing evicted: all updated scores
                assert near_tie_swap(got["pos"].tolist(), c2["pos"].tolist(), c, full, budgets[l] - budgets[l] // 2,
                                     mc), (name, t, l, b, h)
                state[l, b, h] = round_scores_f32(c2)
                continue
            assert got["pos"].tolist() == c2["pos"].tolist(), (name, t, l, b, h)
            assert np.array_equal(got["K"], c2["K"]) and np.array_equal(got["V"], c2["V"])
            if policy == "h2o":
                worst_sc = max(worst_sc, check_step_scores(got, c, c2, mc, (name, t, l, b, h)))
            state[l, b, h] = round_scores_f32(c2)
    assert worst < TOL[dtype], (name, worst)
    print("%s %s: worst out error %.2e of %.0e allowed, worst score error %.2f of its bound" % (name, order, worst, TOL[dtype], worst_sc))


def test_decode_tie_breaking_and_leaver_cases(sqa):
    """Hand-built H2O states: all-equal scores (evict the highest position among
    the non-recent, i.e. the ring leaver), leaver better than the worst heavy
    hitter (it moves), and exact ties inside the heavy region."""
    D, b = 64, 8                                # hh 4, recent 4
    r = np.random.default_rng(0)
    for scores in ([0.5] * 8, [0.9, 0.1, 0.1, 0.7, 0.3, 0.2, 0.2, 0.2], [0.9, 0.4, 0.6, 0.7, 0.3, 0.2, 0.2, 0.2],
                   [0.3, 0.3, 0.3, 0.3, 0.3, 0.0, 0.0, 0.0], [0.0] * 8):
        c = {"K": r.standard_normal((8, D)), "V": r.standard_normal((8, D)),
             "pos": np.array([0, 3, 5, 9, 20, 21, 22, 23]), "score": np.array(scores, dtype=np.float64)}
        c["K"] = c["K"].astype(np.float32).astype(np.float64); c["V"] = c["V"].astype(np.float32).astype(np.float64)
        caches = _mk_caches(sqa, [b], [b], 1, 1, D, "f32")
        import_state(caches, 0, 0, 0, c)
        q = torch.randn(1, 1, 1, D, device=DEV); k = torch.randn(1, 1, 1, D, device=DEV); v = torch.randn(1, 1, 1, D, device=DEV)
        out = torch.empty_like(q); ws = sqa.decode_workspace(caches, 1, "h2o")
        sqa.decode_step(q, k, v, 24, "h2o", 4, caches, out, ws)
        want_out, c2 = O.decode_step(c, np64(q)[0, 0], np64(k)[0, 0, 0], np64(v)[0, 0, 0], 24, b, "h2o")
        got = export_state(caches, 0, 0, 0)
        assert got["pos"].tolist() == c2["pos"].tolist(), scores
        assert rel_err(np64(out)[0, 0], want_out) < 1e-5
        check_step_scores(got, c, c2, False, scores)


def test_decode_free_running_tiny(sqa):
    """configs[0] end to end on the GPU alone: probe -> budgets -> prompt scores
    -> compress -> 16 decode steps, against the oracle run on its own in fp64."""
    wl = W.WORKLOADS["tiny"]
    g = wl.g
    u_dirs, mask = W.unit_dirs(wl), W.hh_mask(wl, DEV)
    hs = [W.hidden_states(wl, l, DEV) for l in range(wl.L)]
    h_in = torch.stack([x[0] for x in hs]); h_out = torch.stack([x[1] for x in hs])
    cos = sqa.layer_importance(h_in, h_out).cpu().numpy()
    budgets, _ = sqa.allocate_budgets(cos, wl.total_budget, wl.p)
    # budgets from the GPU's cosines against budgets from the oracle's: comparable because the best split is
    # far ahead of the second best (fp32 noise in the cosines cannot flip it)
    assert clustering_margin(cos) > 1e-6
    assert budgets == O.allocate_budgets(O.layer_importance(np64(h_in), np64(h_out)).astype(np.float32),
                                         wl.total_budget, wl.p)[0]
    caches = _mk_caches(sqa, budgets, budgets, wl.B, wl.Hkv, wl.D, wl.dtype)
    inp = [_unit_inputs(wl, l, u_dirs, mask) for l in range(wl.L)]
    for l in range(wl.L):
        sc = sqa.prefill_scores(inp[l][2], inp[l][0])
        sqa.prefill_compress(inp[l][0], inp[l][1], sc, wl.policy, wl.n_sink, caches, l)
    q_all = torch.stack([inp[l][3] for l in range(wl.L)], 1).contiguous()
    k_all = torch.stack([inp[l][4] for l in range(wl.L)], 1).contiguous()
    v_all = torch.stack([inp[l][5] for l in range(wl.L)], 1).contiguous()
    ws = sqa.decode_workspace(caches, wl.Hq, wl.policy)
    outs = []
    kept = []
    for t in range(wl.S):
        out = torch.empty(wl.L, wl.B, wl.Hq, wl.D, dtype=wl.torch_dtype, device=DEV)
        sqa.decode_step(q_all[t], k_all[t], v_all[t], wl.P + t, wl.policy, wl.n_sink, caches, out, ws)
        outs.append(np64(out))
        kept.append([sqa.kept_idx_sorted(caches, l).cpu().numpy() for l in range(wl.L)])
    assert sqa.read_device_status(ws) == 0
    qn, kn, vn = np64(q_all), np64(k_all), np64(v_all)
    for l in range(wl.L):
        Kn, Vn, Qn = np64(inp[l][0]), np64(inp[l][1]), np64(inp[l][2])
        for h in range(wl.Hkv):
            s0 = O.prefill_scores(Qn[0, h * g:(h + 1) * g], Kn[0, h])
            o_ref, c, states, _ = OP.run_unit(Kn[0, h], Vn[0, h], s0, qn[:, l, 0, h * g:(h + 1) * g], kn[:, l, 0, h],
                                              vn[:, l, 0, h], budgets[l], wl.policy, wl.n_sink, keep_states=True)
            for t in range(wl.S):
                n = len(states[t]["pos"])
                assert kept[t][l][0, h, :n].tolist() == states[t]["pos"].tolist(), (l, h, t)
                assert rel_err(outs[t][l, 0, h * g:(h + 1) * g], o_ref[t]) < 1e-5
            got = export_state(caches, l, 0, h)
            check_scores_after_run(got["score"], c["score"], wl.S, False, (l, h))


def test_decode_free_running_split_units(sqa):
    """Units longer than a chunk, running on their own for many steps: the
    eviction decision carried from step to step and the split-unit merge must
    reproduce the oracle's kept sets and outputs."""
    wl = W.scaled(W.WORKLOADS["tiny"], L=2, Hq=2, Hkv=2, D=64, B=2, P=500, S=40, dtype="f32")
    budgets = [390, 36]
    g = wl.g
    u_dirs, mask = W.unit_dirs(wl), W.hh_mask(wl, DEV)
    inp = [_unit_inputs(wl, l, u_dirs, mask) for l in range(wl.L)]
    caches = _mk_caches(sqa, budgets, budgets, wl.B, wl.Hkv, wl.D, wl.dtype)
    for l in range(wl.L):
        sqa.prefill_compress(inp[l][0], inp[l][1], sqa.prefill_scores(inp[l][2], inp[l][0]), "h2o", 4, caches, l)
    q_all = torch.stack([inp[l][3] for l in range(wl.L)], 1).contiguous()
    k_all = torch.stack([inp[l][4] for l in range(wl.L)], 1).contiguous()
    v_all = torch.stack([inp[l][5] for l in range(wl.L)], 1).contiguous()
    ws = sqa.decode_workspace(caches, wl.Hq, "h2o")
    outs, kept = [], []
    for t in range(wl.S):
        out = torch.empty(wl.L, wl.B, wl.Hq, wl.D, dtype=wl.torch_dtype, device=DEV)
        sqa.decode_step(q_all[t], k_all[t], v_all[t], wl.P + t, "h2o", 4, caches, out, ws)
        outs.append(np64(out))
        kept.append([sqa.kept_idx_sorted(caches, l).cpu().numpy() for l in range(wl.L)])
    assert sqa.read_device_status(ws) == 0
    qn, kn, vn = np64(q_all), np64(k_all), np64(v_all)
    for l in range(wl.L):
        Kn, Vn, Qn = np64(inp[l][0]), np64(inp[l][1]), np64(inp[l][2])
        for b in range(wl.B):
            for h in range(wl.Hkv):
                s0 = O.prefill_scores(Qn[b, h * g:(h + 1) * g], Kn[b, h])
                o_ref, c, states, _ = OP.run_unit(Kn[b, h], Vn[b, h], s0, qn[:, l, b, h * g:(h + 1) * g],
                                                  kn[:, l, b, h], vn[:, l, b, h], budgets[l], "h2o", 4, keep_states=True)
                for t in range(wl.S):
                    n = len(states[t]["pos"])
                    assert kept[t][l][b, h, :n].tolist() == states[t]["pos"].tolist(), (l, b, h, t)
                    assert rel_err(outs[t][l, b, h * g:(h + 1) * g], o_ref[t]) < 1e-5
                got = export_state(caches, l, b, h)
                check_scores_after_run(got["score"], c["score"], wl.S, False, (l, b, h))


@pytest.mark.parametrize("policy,dtype,D,g,order,B,Hkv,L", [
    ("h2o", "bf16", 128, 1, "evict_then_attend", 32, 8, 16),
    ("h2o", "f32", 64, 2, "attend_then_evict", 32, 8, 16),
    ("streaming", "bf16", 128, 4, "evict_then_attend", 32, 8, 16),
    ("sliding", "f32", 128, 1, "attend_then_evict", 32, 8, 16),
    ("h2o", "bf16", 64, 8, "evict_then_attend", 32, 8, 16),
    ("h2o", "bf16", 64, 1, "evict_then_attend", 33, 5, 25),      # 165 units per layer: the last workgroup is partly empty
])
def test_many_short_units_one_wave_per_unit(sqa, policy, dtype, D, g, order, B, Hkv, L):
    """At least 4096 short units in one call: the launch plan gives each wave a unit of its own.  Free
    running from the compressed prompt for 5 steps; a sample of units against the oracle on its own."""
    P, S = 40, 5
    Hq = Hkv * g
    lo = {"sliding": 1, "streaming": 5, "h2o": 2}[policy]
    r = np.random.default_rng(D + g)
    budgets = [int(x) for x in r.choice([lo, 9, 17, 33, 40, 41, 64, 200], size=L)]
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(device="cpu").manual_seed(7)
    mk = lambda *shape: torch.randn(*shape, generator=gen).to(tdt).to(DEV)
    Ks, Vs = [mk(B, Hkv, P, D) for _ in range(L)], [mk(B, Hkv, P, D) for _ in range(L)]
    Ss = [torch.rand(B, Hkv, P, generator=gen).to(DEV) for _ in range(L)]
    q_all, k_all, v_all = mk(S, L, B, Hq, D), mk(S, L, B, Hkv, D), mk(S, L, B, Hkv, D)
    caches = _mk_caches(sqa, budgets, [min(b, P + S) for b in budgets], B, Hkv, D, dtype)
    sqa.prefill_compress_layers(Ks, Vs, Ss if policy == "h2o" else None, policy, 4, caches)
    ws = sqa.decode_workspace(caches, Hq, policy)
    opts = None if order == "evict_then_attend" else sqa.batch_opts(order=order)
    outs, kept = [], []
    for t in range(S):
        out = torch.empty(L, B, Hq, D, dtype=tdt, device=DEV)
        sqa.decode_step(q_all[t], k_all[t], v_all[t], P + t, policy, 4, caches, out, ws, opts=opts)
        outs.append(np64(out))
        kept.append([sqa.kept_idx_sorted(caches, l).cpu().numpy() for l in range(L)])
    assert sqa.read_device_status(ws) == 0
    qn, kn, vn = np64(q_all), np64(k_all), np64(v_all)
    units = [(l, b, h) for l in range(L) for b in range(B) for h in range(Hkv)]
    for l, b, h in units[::89] + units[-3:]:
        o_ref, c, states, _ = OP.run_unit(np64(Ks[l])[b, h], np64(Vs[l])[b, h], np64(Ss[l])[b, h],
                                          qn[:, l, b, h * g:(h + 1) * g], kn[:, l, b, h], vn[:, l, b, h],
                                          budgets[l], policy, 4, keep_states=True, order=order)
        for t in range(S):
            n = len(states[t]["pos"])
            assert kept[t][l][b, h, :n].tolist() == states[t]["pos"].tolist(), (l, b, h, t)
            assert rel_err(outs[t][l, b, h * g:(h + 1) * g], o_ref[t]) < TOL[dtype], (l, b, h, t)
        if policy == "h2o":
            got = export_state(caches, l, b, h)
            check_scores_after_run(got["score"], c["score"], S, uses_matrix_cores(dtype, D, g), (l, b, h))


@pytest.mark.parametrize("g,order", [(4, "evict_then_attend"), (8, "evict_then_attend"), (8, "attend_then_evict")])
def test_many_short_units_grouped_queries_h2o(sqa, g, order):
    """4096 short units with 4 or 8 query heads per KV head under H2O (bf16, D = 128): the matrix-core
    variant with a unit per wave, the step's probabilities kept as bf16 in the workspace.  Teacher forced:
    before every step a sample of units is set to the oracle's state, the step runs for the whole batch and
    the sample is compared."""
    policy, dtype, D, B, Hkv, L, P, S = "h2o", "bf16", 128, 64, 8, 8, 40, 3
    Hq = Hkv * g
    ae = order == "attend_then_evict"
    budgets = [6, 17, 33, 40, 41, 64, 200, 9]
    gen = torch.Generator(device="cpu").manual_seed(70 + g)
    mk = lambda *shape: torch.randn(*shape, generator=gen).to(torch.bfloat16).to(DEV)
    Ks, Vs = [mk(B, Hkv, P, D) for _ in range(L)], [mk(B, Hkv, P, D) for _ in range(L)]
    Ss = [torch.rand(B, Hkv, P, generator=gen).to(DEV) for _ in range(L)]
    q_all, k_all, v_all = mk(S, L, B, Hq, D), mk(S, L, B, Hkv, D), mk(S, L, B, Hkv, D)
    caches = _mk_caches(sqa, budgets, [min(b, P + S) for b in budgets], B, Hkv, D, dtype)
    sqa.prefill_compress_layers(Ks, Vs, Ss, policy, 4, caches)
    ws = sqa.decode_workspace(caches, Hq, policy)
    opts = sqa.batch_opts(order=order) if ae else None
    units = [(l, b, h) for l in range(L) for b in range(B) for h in range(Hkv)]
    sample = units[::97] + units[-2:]
    state = {(l, b, h): O.prefill_compress(np64(Ks[l])[b, h], np64(Vs[l])[b, h], np64(Ss[l])[b, h], budgets[l], policy, 4)
             for l, b, h in sample}
    qn, kn, vn = np64(q_all), np64(k_all), np64(v_all)
    out = torch.empty(L, B, Hq, D, dtype=torch.bfloat16, device=DEV)
    for t in range(S):
        for key, c in state.items():
            import_state(caches, key[0], key[1], key[2], c)
        sqa.decode_step(q_all[t], k_all[t], v_all[t], P + t, policy, 4, caches, out, ws, opts=opts)
        assert sqa.read_device_status(ws) == 0
        o = np64(out)
        for (l, b, h), c in state.items():
            args = (qn[t, l, b, h * g:(h + 1) * g], kn[t, l, b, h], vn[t, l, b, h], P + t)
            want_out, c2 = O.decode_step(c, *args, budgets[l], policy, 4, order)
            got = export_state(caches, l, b, h)
            assert rel_err(o[l, b, h * g:(h + 1) * g], want_out) < TOL[dtype], (t, l, b, h)
            if got["pos"].tolist() != c2["pos"].tolist():           # only a near-tie under attend-then-evict may differ
                assert ae
                _, full = O.decode_step(c, *args, 1 << 30, policy, 4, order)
                assert near_tie_swap(got["pos"].tolist(), c2["pos"].tolist(), c, full, budgets[l] - budgets[l] // 2,
                                     True), (t, l, b, h)
            else:
                assert np.array_equal(got["K"], c2["K"]) and np.array_equal(got["V"], c2["V"])
                check_step_scores(got, c, c2, True, (t, l, b, h))
            state[l, b, h] = round_scores_f32(c2)


@pytest.mark.parametrize("policy", ["sliding", "streaming", "h2o"])
def test_decode_from_an_empty_cache(sqa, policy):
    """No prompt at all: the first step attends to the new token alone (out = v), then the cache
    grows to its budget and starts evicting -- 12 steps with budget 6 against the oracle."""
    D, b, S, Hkv, g = 64, 6, 12, 2, 2
    r = np.random.default_rng(3)
    caches = _mk_caches(sqa, [b], [b], 1, Hkv, D, "f32")
    ws = sqa.decode_workspace(caches, Hkv * g, policy)
    state = {h: O.new_cache(np.zeros((0, D)), np.zeros((0, D))) for h in range(Hkv)}
    for t in range(S):
        q = torch.from_numpy(r.standard_normal((1, 1, Hkv * g, D)).astype(np.float32)).to(DEV)
        k = torch.from_numpy(r.standard_normal((1, 1, Hkv, D)).astype(np.float32)).to(DEV)
        v = torch.from_numpy(r.standard_normal((1, 1, Hkv, D)).astype(np.float32)).to(DEV)
        out = torch.empty_like(q)
        sqa.decode_step(q, k, v, t, policy, 4, caches, out, ws)
        for h in range(Hkv):
            want, state[h] = O.decode_step(state[h], np64(q)[0, 0, h * g:(h + 1) * g], np64(k)[0, 0, h], np64(v)[0, 0, h],
                                           t, b, policy, 4)
            assert rel_err(np64(out)[0, 0, h * g:(h + 1) * g], want) < 1e-5, (t, h)
            got = export_state(caches, 0, 0, h)
            assert got["pos"].tolist() == state[h]["pos"].tolist(), (t, h)
            if t == 0:
                assert np.allclose(np64(out)[0, 0, h * g], np64(v)[0, 0, h], atol=1e-6)
    assert sqa.read_device_status(ws) == 0


def test_decode_one_very_long_unit(sqa):
    """A single unit of 20000 tokens (H2O, bf16): split over many workgroups, logits through the
    workspace, arg-min over 10000 heavy hitters."""
    D, P, b = 128, 20000, 20000
    r = np.random.default_rng(11)
    K = torch.randn(1, 1, P, D, device=DEV).to(torch.bfloat16)
    V = torch.randn(1, 1, P, D, device=DEV).to(torch.bfloat16)
    sc = torch.rand(1, 1, P, device=DEV)
    caches = _mk_caches(sqa, [b], [b], 1, 1, D, "bf16")
    sqa.prefill_compress(K, V, sc, "h2o", 4, caches, 0)
    ws = sqa.decode_workspace(caches, 1, "h2o")
    for t in range(2):
        c = export_state(caches, 0, 0, 0)          # the oracle steps from what the GPU holds (same fp32 scores)
        q = torch.randn(1, 1, 1, D, device=DEV).to(torch.bfloat16)
        k = torch.randn(1, 1, 1, D, device=DEV).to(torch.bfloat16)
        v = torch.randn(1, 1, 1, D, device=DEV).to(torch.bfloat16)
        out = torch.empty_like(q)
        sqa.decode_step(q, k, v, P + t, "h2o", 4, caches, out, ws)
        want, c2 = O.decode_step(c, np64(q)[0, 0], np64(k)[0, 0, 0], np64(v)[0, 0, 0], P + t, b, "h2o")
        got = export_state(caches, 0, 0, 0)
        assert got["pos"].tolist() == c2["pos"].tolist(), t
        assert rel_err(np64(out)[0, 0], want) < 2e-2
        check_step_scores(got, c, c2, False, t)
    assert sqa.read_device_status(ws) == 0


@pytest.mark.parametrize("policy,P,b", [("sliding", 70000, 70010), ("streaming", 70000, 66000), ("h2o", 50000, 40000)])
def test_units_longer_than_any_lds_list(sqa, policy, P, b):
    """Prompt compression and the sorted view for units beyond 32768 and 65536 kept tokens (an uncompressed
    cache of a long context; an H2O budget of 40000): only the tokens chosen by score are listed in LDS,
    the window and the sinks are index arithmetic, and the sorted view ranks from memory."""
    D, S = 64, 2
    gen = torch.Generator(device="cpu").manual_seed(5)
    K = torch.randn(1, 1, P, D, generator=gen).to(DEV); V = torch.randn(1, 1, P, D, generator=gen).to(DEV)
    sc = torch.rand(1, 1, P, generator=gen).to(DEV)
    cap = min(b, P + S)
    caches = _mk_caches(sqa, [b], [cap], 1, 1, D, "f32")
    sqa.prefill_compress(K, V, sc if policy == "h2o" else None, policy, 4, caches, 0)
    c = O.prefill_compress(np64(K)[0, 0], np64(V)[0, 0], np64(sc)[0, 0], b, policy, 4)
    got = export_state(caches, 0, 0, 0)
    assert got["pos"].tolist() == c["pos"].tolist()
    assert np.array_equal(got["K"], c["K"]) and np.array_equal(got["V"], c["V"])
    if policy == "h2o":
        assert np.array_equal(got["score"], c["score"])
    ws = sqa.decode_workspace(caches, 1, policy)
    for t in range(S):
        q = torch.randn(1, 1, 1, D, generator=gen).to(DEV); k = torch.randn(1, 1, 1, D, generator=gen).to(DEV)
        v = torch.randn(1, 1, 1, D, generator=gen).to(DEV)
        out = torch.empty_like(q)
        before = export_state(caches, 0, 0, 0)
        sqa.decode_step(q, k, v, P + t, policy, 4, caches, out, ws)
        want, c2 = O.decode_step(before, np64(q)[0, 0], np64(k)[0, 0, 0], np64(v)[0, 0, 0], P + t, b, policy, 4)
        got = export_state(caches, 0, 0, 0)
        assert got["pos"].tolist() == c2["pos"].tolist(), t
        assert rel_err(np64(out)[0, 0], want) < 1e-5
        if policy == "h2o":
            check_step_scores(got, before, c2, False, t)
    assert sqa.read_device_status(ws) == 0
    n = len(c2["pos"])
    assert sqa.kept_idx_sorted(caches, 0)[0, 0, :n].cpu().tolist() == c2["pos"].tolist()


@pytest.mark.parametrize("order", ["evict_then_attend", "attend_then_evict"])
@pytest.mark.parametrize("dtype,D,g,b", [("f32", 64, 1, 1409), ("f32", 128, 8, 700), ("bf16", 128, 1, 3001), ("bf16", 64, 2, 1290),
                                         ("bf16", 128, 4, 2750), ("bf16", 128, 8, 4100)])
@pytest.mark.parametrize("flat", [False, True], ids=["", "ties"])
def test_a_unit_in_many_pieces(sqa, dtype, D, g, b, order, flat):
    """One unit cut into 4 to 18 pieces (numbers that are and are not multiples of 8, a last piece of few slots):
    outputs, scores and the tokens kept over several steps.  flat: equal keys and scores, so that every heavy
    hitter ties for the lowest score and the highest position has to go."""
    S, P = 3, b + 40
    gen = torch.Generator(device="cpu").manual_seed(b)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    mk = lambda *shape: torch.randn(*shape, generator=gen).to(dt).to(DEV)
    K, V = mk(1, 1, P, D), mk(1, 1, P, D)
    sc = torch.rand(1, 1, P, generator=gen) + 0.5
    if flat:
        K.zero_()
        sc.fill_(1.0)
        sc[0, 0, P - (b - b // 2):] = 2.0            # the recent window: its leaver outlives the worst heavy hitter
    sc = sc.to(DEV)
    caches = _mk_caches(sqa, [b], [b], 1, 1, D, dtype)
    sqa.prefill_compress(K, V, sc, "h2o", 4, caches, 0)
    plan = sqa.decode_plan([b], [b], 1, g, 1, D, dtype, "h2o")
    assert plan["layers"][0]["workgroups_per_unit"] >= 4
    ws, less = sqa.decode_workspace(caches, g, "h2o"), torch.zeros(plan["workspace_bytes"] - 256, dtype=torch.uint8, device=DEV)
    mf = uses_matrix_cores(dtype, D, g)
    for t in range(S):
        q, k, v = mk(1, 1, g, D), mk(1, 1, 1, D), mk(1, 1, 1, D)
        if flat:
            k.zero_()
        before = export_state(caches, 0, 0, 0)
        out = torch.empty_like(q)
        # (in between with less scratch than the cut above needs: fewer pieces, unless there are none fewer)
        w = less if t == 1 and not mf else ws
        sqa.decode_step(q, k, v, P + t, "h2o", 4, caches, out, w, opts=sqa.batch_opts(order=order))
        want, c2 = O.decode_step(oracle_view(before), np64(q)[0, 0], np64(k)[0, 0, 0], np64(v)[0, 0, 0], P + t, b, "h2o", 4, order=order)
        got = export_state(caches, 0, 0, 0)
        assert got["pos"].tolist() == c2["pos"].tolist(), t
        assert rel_err(np64(out)[0, 0], want) < TOL[dtype]
        check_step_scores(got, before, c2, mf, (t,))


@pytest.mark.parametrize("order", ["evict_then_attend", "attend_then_evict"])
def test_fewer_pieces_with_less_scratch_on_the_matrix_cores(sqa, order):
    """16 units in 26 pieces each, and with a workspace that does not hold those in 13: both against the oracle, and the
    same state after every step."""
    B, Hkv, g, D, b, dtype = 8, 2, 8, 128, 8192, "bf16"
    P = b + 20
    gen = torch.Generator(device=DEV).manual_seed(b)
    mk = lambda *shape: torch.randn(*shape, generator=gen, device=DEV).bfloat16()
    K, V, sc = mk(B, Hkv, P, D), mk(B, Hkv, P, D), torch.rand(B, Hkv, P, generator=gen, device=DEV) + 0.5
    caches = [_mk_caches(sqa, [b], [b], B, Hkv, D, dtype) for _ in range(2)]
    for c in caches:
        sqa.prefill_compress(K, V, sc, "h2o", 4, c, 0)
    plan = sqa.decode_plan([b], [b], B, Hkv * g, Hkv, D, dtype, "h2o")
    assert plan["layers"][0]["workgroups_per_unit"] == 26 and uses_matrix_cores(dtype, D, g)
    ws = [torch.zeros(plan["workspace_bytes"] - x, dtype=torch.uint8, device=DEV) for x in (0, 256)]
    for t in range(2):
        q, k, v = mk(1, B, Hkv * g, D), mk(1, B, Hkv, D), mk(1, B, Hkv, D)
        units = [(0, 0), (B - 1, Hkv - 1)]
        outs = []
        for c, w in zip(caches, ws):
            before = [export_state(c, 0, x, h) for x, h in units]
            out = torch.empty_like(q)
            sqa.decode_step(q, k, v, P + t, "h2o", 4, c, out, w, opts=sqa.batch_opts(order=order))
            outs.append(out)
            for (x, h), s0 in zip(units, before):
                want, c2 = O.decode_step(oracle_view(s0), np64(q)[0, x, h * g:(h + 1) * g], np64(k)[0, x, h], np64(v)[0, x, h], P + t, b,
                                         "h2o", 4, order=order)
                got = export_state(c, 0, x, h)
                assert got["pos"].tolist() == c2["pos"].tolist(), (t, x, h)
                assert rel_err(np64(out)[0, x, h * g:(h + 1) * g], want) < TOL[dtype]
                check_step_scores(got, s0, c2, True, (t, x, h))
        assert rel_err(np64(outs[0]), np64(outs[1])) < TOL[dtype]
        assert sqa.read_device_status(ws[0]) == 0 and sqa.read_device_status(ws[1]) == 0


@pytest.mark.parametrize("order", ["evict_then_attend", "attend_then_evict"])
@pytest.mark.parametrize("dtype,D,g,B,b", [("f32", 64, 1, 17, 769), ("f32", 64, 1, 17, 768), ("bf16", 128, 2, 20, 1030)])
def test_long_whole_units_in_a_call_of_some_hundred_workgroups(sqa, dtype, D, g, B, b, order):
    """544 and 640 whole units: the score walk of one over 768 tokens keeps all four waves, of a shorter one does not."""
    Hkv, S, P = 32, 3, b + 20
    gen = torch.Generator(device=DEV).manual_seed(b)
    dt = torch.float32 if dtype == "f32" else torch.bfloat16
    mk = lambda *shape: torch.randn(*shape, generator=gen, device=DEV).to(dt)
    K, V, sc = mk(B, Hkv, P, D), mk(B, Hkv, P, D), torch.rand(B, Hkv, P, generator=gen, device=DEV) + 0.5
    caches = _mk_caches(sqa, [b], [b], B, Hkv, D, dtype)
    sqa.prefill_compress(K, V, sc, "h2o", 4, caches, 0)
    plan = sqa.decode_plan([b], [b], B, Hkv * g, Hkv, D, dtype, "h2o")
    assert 512 < plan["workgroups"] <= 2048 and plan["layers"][0]["workgroups_per_unit"] == 1
    ws = sqa.decode_workspace(caches, Hkv * g, "h2o")
    for t in range(S):
        q, k, v = mk(1, B, Hkv * g, D), mk(1, B, Hkv, D), mk(1, B, Hkv, D)
        units = [(0, 0), (B // 2, 7), (B - 1, Hkv - 1)]
        before = [export_state(caches, 0, x, h) for x, h in units]
        out = torch.empty_like(q)
        sqa.decode_step(q, k, v, P + t, "h2o", 4, caches, out, ws, opts=sqa.batch_opts(order=order))
        for (x, h), c in zip(units, before):
            want, c2 = O.decode_step(oracle_view(c), np64(q)[0, x, h * g:(h + 1) * g], np64(k)[0, x, h], np64(v)[0, x, h], P + t, b,
                                     "h2o", 4, order=order)
            got = export_state(caches, 0, x, h)
            assert got["pos"].tolist() == c2["pos"].tolist(), (t, x, h)
            assert rel_err(np64(out)[0, x, h * g:(h + 1) * g], want) < TOL[dtype]
            check_step_scores(got, c, c2, False, (t, x, h))


def test_decode_is_deterministic_and_per_layer_calls_agree(sqa):
    """Same inputs twice -> identical bytes; one call over all layers == one call per layer (with and without the
    device copy of the layer table), where both give a layer the same cut and waves, as in calls as small as these."""
    wl = W.scaled(W.WORKLOADS["tiny"], L=3, Hq=4, Hkv=2, D=128, B=2, P=320, S=5, dtype="bf16")
    budgets = [30, 323, 17]
    u_dirs, mask = W.unit_dirs(wl), W.hh_mask(wl, DEV)
    inp = [_unit_inputs(wl, l, u_dirs, mask) for l in range(wl.L)]
    q_all = torch.stack([inp[l][3] for l in range(wl.L)], 1).contiguous()
    k_all = torch.stack([inp[l][4] for l in range(wl.L)], 1).contiguous()
    v_all = torch.stack([inp[l][5] for l in range(wl.L)], 1).contiguous()
    results = []
    for mode in ("all", "all", "per_layer", "per_layer_hosttable"):
        caches = _mk_caches(sqa, budgets, budgets, wl.B, wl.Hkv, wl.D, wl.dtype)
        for l in range(wl.L):
            sqa.prefill_compress(inp[l][0], inp[l][1], sqa.prefill_scores(inp[l][2], inp[l][0]), "h2o", 4, caches, l)
        ws = sqa.decode_workspace(caches, wl.Hq, "h2o")
        ws1 = [sqa.decode_workspace(caches, wl.Hq, "h2o", l, 1) for l in range(wl.L)]
        outs = []
        for t in range(wl.S):
            out = torch.empty(wl.L, wl.B, wl.Hq, wl.D, dtype=wl.torch_dtype, device=DEV)
            if mode == "all":
                sqa.decode_step(q_all[t], k_all[t], v_all[t], wl.P + t, "h2o", 4, caches, out, ws)
            else:
                for l in range(wl.L):
                    sqa.decode_step(q_all[t, l], k_all[t, l], v_all[t, l], wl.P + t, "h2o", 4, caches, out[l], ws1[l],
                                    layer0=l, n_layers=1, use_dev_table=(mode == "per_layer"))
            outs.append(out)
        assert sqa.read_device_status(ws) == 0 and all(sqa.read_device_status(w) == 0 for w in ws1)
        results.append((torch.stack(outs).view(torch.int16).cpu(), [s.clone().cpu() for s in caches.score],
                        [p.clone().cpu() for p in caches.pos]))
    for other in results[1:]:
        assert torch.equal(results[0][0], other[0])
        for a, b in zip(results[0][1], other[1]):
            assert torch.equal(a.view(torch.int32), b.view(torch.int32))
        for a, b in zip(results[0][2], other[2]):
            assert torch.equal(a, b)


def test_decode_reports_bad_state_without_touching_the_cache(sqa):
    caches = _mk_caches(sqa, [4], [8], 1, 1, 64, "f32")
    caches.lens[0][0, 0] = 6                      # longer than the budget on entry
    q = torch.randn(1, 1, 1, 64, device=DEV); out = torch.ones_like(q)
    ws = sqa.decode_workspace(caches, 1, "sliding")
    sqa.decode_step(q, q, q, 9, "sliding", 4, caches, out, ws)
    assert sqa.read_device_status(ws) == 8        # SQA_ERR_STATE
    assert int(caches.lens[0][0, 0]) == 6 and float(out.abs().sum()) == 0.0
    sqa.clear_device_status(ws)
    assert sqa.read_device_status(ws) == 0
    caches2 = _mk_caches(sqa, [40], [3], 1, 1, 64, "f32")
    caches2.lens[0][0, 0] = 3                     # no free slot
    ws = sqa.decode_workspace(caches2, 1, "sliding")
    sqa.decode_step(q, q, q, 9, "sliding", 4, caches2, out, ws)
    assert sqa.read_device_status(ws) == 6        # SQA_ERR_CAPACITY


@pytest.mark.parametrize("Hq", [4, 8])
def test_decode_steps_replayed_from_a_hip_graph(sqa, Hq):
    """One launch per layer recorded once into a HIP graph (positions from a device array), replayed
    for every step with eager work and synchronisations between the replays: every replay must leave
    the same bytes as the eager run of the same step.  (8 query heads on 2 KV heads: the matrix-core
    variant, with its direct loads into LDS and its scratch in the workspace.)"""
    from paper_2404_04793_amd.session import Session
    wl = W.scaled(W.WORKLOADS["tiny"], L=4, B=2, P=96, S=10, dtype="bf16", D=128, Hq=Hq, Hkv=2, hidden=256)
    runs = []
    for use_graph in (False, True):
        sess = Session(wl, DEV)
        sess.probe_and_allocate()
        sess.compress_prompt()
        if use_graph:
            sess.capture_step_graph(per_layer=True)
        snaps = []
        for t in range(wl.S):
            if use_graph:
                sess.decode_graph(steps=1, start=t)
                _ = (sess.q[t].float().sum() + 1).item()          # eager work and a sync between replays
            else:
                sess.decode(steps=1, per_layer=True, start=t)
            torch.cuda.synchronize()
            snaps.append((sess.out[t].clone(), [p.clone() for p in sess.caches.pos], [s.clone() for s in sess.caches.score],
                          [s.clone() for s in sess.caches.state]))
        assert all(sqa.read_device_status(w) == 0 for w in sess.dec_ws_layer)
        runs.append(snaps)
    for t, (a, b) in enumerate(zip(*runs)):
        assert torch.equal(a[0].view(torch.int16), b[0].view(torch.int16)), t
        for x, y in zip(a[1] + a[2] + a[3], b[1] + b[2] + b[3]):
            assert torch.equal(x, y), t
