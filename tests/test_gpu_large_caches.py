"""MHA decode over 7 GiB of K and V and more stores its rows non-temporally, in a kernel of its own.  32 layers of together
exactly 7 GiB in one call against the same steps layer by layer (224 MiB a call, the ordinary kernel, the same split of the
work): outputs, caches and bookkeeping have to be the same bit for bit, while the units fill up and after that."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("dtype,D,policy,order,blocked", [
    ("f32", 128, "h2o", "evict_then_attend", False), ("bf16", 128, "h2o", "attend_then_evict", True),
    ("bf16", 64, "streaming", "evict_then_attend", False), ("f32", 64, "sliding", "attend_then_evict", True)])
def test_one_call_over_large_caches_equals_layer_by_layer(dtype, D, policy, order, blocked):
    from paper_2404_04793_amd import binding as sqa
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    L, H, row = 32, 32, 2 * D * (4 if dtype == "f32" else 2)
    B, budgets = 4096 * 1024 // (H * row), [52, 60] * (L // 2)
    assert sum(budgets) * B * H * row == 7 << 30
    made = [sqa.LayerCaches(budgets, budgets, B, H, D, tdt, DEV, policy == "h2o", blocked=blocked) for _ in range(2)]
    spaces = [sqa.decode_workspace(c, H, policy) for c in made]
    gen = torch.Generator(DEV).manual_seed(D)
    q, k, v = (torch.randn(L, B, H, D, generator=gen, device=DEV).to(tdt) for _ in range(3))
    out = [torch.empty_like(q) for _ in range(2)]
    opts = sqa.batch_opts(order=order)
    for t in range(72):
        # other values each step, without drawing them anew
        qt, kt, vt = (torch.roll(x, t, 1) for x in (q, k, v))
        sqa.decode_step(qt, kt, vt, t, policy, 4, made[0], out[0], spaces[0], opts=opts)
        for l in range(L):
            sqa.decode_step(qt[l:l + 1], kt[l:l + 1], vt[l:l + 1], t, policy, 4, made[1], out[1][l:l + 1], spaces[1], layer0=l, n_layers=1, opts=opts)
        assert torch.equal(*out), t
    for l in range(L):
        for name in ("K", "V", "pos", "state") + (("score",) if policy == "h2o" else ()):
            assert torch.equal(getattr(made[0], name)[l], getattr(made[1], name)[l]), (l, name)
    assert int(made[0].lens[0].min()) == 52 and sqa.read_device_status(spaces[0]) == 0
