"""8 query heads per KV head in fp32 and in bf16 at D = 64: the products run on the matrix cores with probabilities in 32
bits, tile by tile (32 tokens, 16 in fp32 at D = 128).  Units that end around a tile, a pass of the 4 waves and a piece of a
split unit, in both orders (attend-then-evict has the new token one index beyond the last slot: alone in its tile at multiples
of 16), dense and in blocks, against the oracle; and no value from beyond a unit's end, whatever lies there."""
import pytest
import torch

from tests.test_gpu_stepping import _run_case

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
KINDS = [("bf16", 64), ("f32", 64), ("f32", 128)]


@pytest.fixture(scope="module")
def sqa():
    from paper_2404_04793_amd import binding
    return binding


@pytest.mark.parametrize("blocked", [False, True])
@pytest.mark.parametrize("order", ["evict_then_attend", "attend_then_evict"])
@pytest.mark.parametrize("dtype,D", KINDS)
@pytest.mark.parametrize("policy,budgets", [("h2o", [15, 16, 17, 31, 32, 33]), ("h2o", [63, 64, 65, 127, 128, 129]), ("h2o", [639, 640, 641]),
                                            ("streaming", [16, 32, 33, 128, 129, 640])])
def test_units_around_a_tile(sqa, dtype, D, policy, budgets, order, blocked):
    if policy != "h2o" and (dtype, D) == ("f32", 128):
        pytest.skip("on the vector ALUs")
    _run_case(sqa, ("eight_heads", dtype, 16, 2, D, 2, max(budgets) + 3, 4, policy, budgets, order), stride=1, blocked=blocked,
              need_both_outcomes=False)


@pytest.mark.parametrize("order", ["evict_then_attend", "attend_then_evict"])
@pytest.mark.parametrize("dtype,D", KINDS)
def test_units_that_fill_up(sqa, dtype, D, order):
    _run_case(sqa, ("eight_heads_filling", dtype, 16, 2, D, 2, 30, 6, "h2o", [31, 33, 60, 1000], order), stride=1, need_both_outcomes=False)


@pytest.mark.parametrize("order", ["evict_then_attend", "attend_then_evict"])
@pytest.mark.parametrize("dtype,D", KINDS)
@pytest.mark.parametrize("b,n", [(48, 20), (64, 64), (33, 33), (700, 311)])
def test_nothing_beyond_the_end_of_a_unit_counts(sqa, dtype, D, b, n, order):
    """Slots that hold no token are NaN: rows that a tile reads beyond the unit's tokens must not reach the output."""
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator().manual_seed(b + n)
    mk = lambda *shape: torch.randn(*shape, generator=gen).to(tdt).to(DEV)
    got = []
    for fill in (0.0, float("nan")):
        gen.manual_seed(b + n)
        caches = sqa.LayerCaches([b], [b], 2, 2, D, tdt, DEV, True)
        caches.K[0].fill_(fill); caches.V[0].fill_(fill)
        sqa.prefill_compress_layers([mk(2, 2, n, D)], [mk(2, 2, n, D)], [torch.rand(2, 2, n, generator=gen).to(DEV)], "h2o", 4, caches)
        q, k, v = mk(1, 2, 16, D), mk(1, 2, 2, D), mk(1, 2, 2, D)
        out, ws = torch.empty_like(q), sqa.decode_workspace(caches, 16, "h2o")
        for t in range(3):
            sqa.decode_step(q, k, v, n + t, "h2o", 4, caches, out, ws, opts=sqa.batch_opts(order=order))
        got.append(out.clone())
    assert torch.isfinite(got[1].float()).all() and torch.equal(got[0], got[1])


@pytest.mark.parametrize("order", ["evict_then_attend", "attend_then_evict"])
@pytest.mark.parametrize("dtype,D", KINDS)
def test_scores_use_the_exponents_that_were_summed(sqa, dtype, D, order):
    """A token alone has the probability 1 under each of the 8 heads, however large its logit (here up to 300): the exponential
    that its score adds has to be the one its normaliser holds.  Each is off by at most the reciprocal's and the product's
    rounding, 2^-22 together; a logit rounded in between would be off by 2^-24 of itself."""
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(DEV).manual_seed(D)
    B, H = 16, 4
    mk = lambda *shape: (8 * torch.randn(*shape, generator=gen, device=DEV)).to(tdt)
    caches = sqa.LayerCaches([40], [40], B, H, D, tdt, DEV, True)
    q, k, v = mk(1, B, 8 * H, D), mk(1, B, H, D), mk(1, B, H, D)
    out, ws = torch.empty_like(q), sqa.decode_workspace(caches, 8 * H, "h2o")
    sqa.decode_step(q, k, v, 0, "h2o", 4, caches, out, ws, opts=sqa.batch_opts(order=order))
    assert float((caches.score[0][..., 0].double() - 8).abs().max()) <= 8 * 2.0 ** -22
