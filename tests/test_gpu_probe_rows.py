"""Every row of the probe counts once, whichever kernel, workgroup and turn it falls to.  Rows that go in and come out as
they are, negated or zero have the cosines 1, -1 and 0 (zero rows: 0) without rounding, so the sum over a layer's or a
sequence's rows is a whole number: one row lost, counted twice or credited to a neighbour shows in it."""
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
    """The sums that the means stand for.  cos is rounded to fp32 once, at most 2^-24 of |mean| <= 1: 2^-24 of a row per row,
    0.018 for 300000; the cosine of a row alone is off by a few 2^-53."""
    got = cos.double() * counts
    assert float((got - want).abs().max()) < 0.02, (got - want).abs().max()


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
