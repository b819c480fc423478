"""Every row of the probe counts once, whichever kernel, workgroup and turn it falls to.  Rows that go in and come out as
they are, negated or zero have the cosines 1, -1 and 0, so the sum over a layer's or a sequence's rows is a whole number: one
row lost, counted twice or credited to a neighbour shows in it."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture(scope="module")
def sqa():
    from paper_2404_04793_amd import binding
    return binding


def _rows(L, T, d, dtype, seed):
    """h_in, attn_out, h_out [L, T, d] and the rows' cosines [L, T]: h_out = h_in + attn_out = +-h_in, or both zero."""
    gen = torch.Generator(DEV).manual_seed(seed)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    a = torch.randn(L, T, d, generator=gen, device=DEV).to(tdt)
    a[..., 0] = 1.0                                        # (no zero row by chance)
    kind = torch.randint(0, 5, (L, T), generator=gen, device=DEV)
    a[kind == 4] = 0
    sign = torch.where(kind < 2, 1.0, -1.0).to(tdt).unsqueeze(-1)
    h = a * sign
    return a, h - a, h, torch.where(kind == 4, 0.0, torch.where(kind < 2, 1.0, -1.0)).double()


def _whole(cos, counts, want):
    """The sums that the means stand for; a row is 1.  A mean is rounded to fp32 (2^-24 of it).  The products of a row with
    itself and with its opposite go through the same sums and may round differently (two bf16 products added at once do): over
    a row of up to 1 KiB at most 4 additions in a lane and 6 over the lanes, 10 * 2^-23 of it, 0.31 over 262144 rows if
    all were off in one direction; a row of 8 elements 4, 0.25 over 530000; longer rows are few here (20000 of 264 elements, 14 each: 0.04)."""
    got = cos.double() * counts
    assert float((got - want).abs().max()) < 0.35, (got - want).abs().max()


@pytest.mark.parametrize("dtype,d", [("bf16", 520), ("bf16", 2048), ("f32", 1032), ("bf16", 4096), ("f32", 2056), ("f32", 16384)])
@pytest.mark.parametrize("T", [1, 4, 5, 8, 9, 12, 13])
def test_few_long_rows(sqa, dtype, d, T):
    """One workgroup alone writes the result where its turns are few and short: up to 3 turns, rows of up to 4 KiB, 2 of up to
    8 KiB, one of any."""
    a, r, h, cos = _rows(2, T, d, dtype, T + d)
    want = cos.sum(1)
    _whole(sqa.layer_importance(a, h), T, want)
    out = torch.empty_like(a)
    _whole(sqa.residual_add_importance(a, r, out), T, want)
    assert torch.equal(out, h)


@pytest.mark.parametrize("dtype,d,T", [("bf16", 8, 262143), ("bf16", 8, 262144), ("f32", 8, 262145), ("f32", 128, 294913), ("bf16", 8, 530000),
                                       ("bf16", 264, 262144), ("f32", 136, 262145), ("bf16", 512, 278529)])
def test_many_short_rows(sqa, dtype, d, T):
    """A lane keeps the sums of one row, and when all lanes of a row have one (32 or 64) their cosines are worked out together:
    around and after the 262144 rows at which that comes up inside the loop (1024 workgroups of 4 waves, 8 turns of 8 rows or 16
    of 4), alone and inside the residual add."""
    a, r, h, cos = _rows(1, T, d, dtype, T)
    want = cos.sum(1)
    _whole(sqa.layer_importance(a, h), T, want)
    _whole(sqa.residual_add_importance(a, r, a), T, want)
    assert torch.equal(a, h)


def _lens(name):
    gen = torch.Generator().manual_seed(3)
    return {
        "one long": [1] * 16 + [4096] + [1] * 16,
        "ends on pieces": [0, 32, 16, 4, 1, 0, 0, 64, 8, 3, 128, 0, 31, 33, 0],
        "around 64": [5, 0, 700] + [2] * 60 + [9],         # 64 sequences: one more than a round of the search holds
        "two rounds": torch.randint(0, 9, (1000,), generator=gen).tolist(),
        "three rounds": torch.randint(0, 3, (5000,), generator=gen).tolist(),
        "few rows": [2, 0, 1],
        "few and empty": [0, 3, 0, 0, 5],
        "longer pieces": [0, 3, 30000, 1, 100, 40001, 17, 0],
    }[name]


@pytest.mark.parametrize("dtype,d", [("bf16", 8), ("f32", 64), ("bf16", 512), ("f32", 264)])
@pytest.mark.parametrize("before,after", [(0, 0), (5, 3)])
@pytest.mark.parametrize("name", ["one long", "ends on pieces", "around 64", "two rounds", "three rounds", "few rows",
                                  "few and empty", "longer pieces"])
def test_uneven_sequences(sqa, dtype, d, name, before, after):
    """Rows are shared out in pieces that end where a sequence ends: empty, short and long ones in one batch, rows before the
    first and after the last (which count for none), from one round of the search for a workgroup's sequence to three."""
    lens = _lens(name)
    if name == "longer pieces" and d > 64:
        lens = [n // 4 for n in lens]
    L, T = 2, before + sum(lens) + after
    a, _, h, cos = _rows(L, T, d, dtype, T)
    start = torch.tensor([before] + lens, device=DEV).cumsum(0)
    upto = torch.nn.functional.pad(cos, (1, 0)).cumsum(1)
    want = upto[:, start[1:]] - upto[:, start[:-1]]
    got = sqa.layer_importance_seq(a, h, start.to(torch.int32))
    _whole(got, torch.tensor(lens, device=DEV), want)
    assert bool((got[:, torch.tensor(lens, device=DEV) == 0] == 0).all())
    again = sqa.layer_importance_seq(a, h, start.to(torch.int32))
    assert torch.equal(got, again)
