"""Slots that hold no token count nothing, whatever lies there: a cache handed over as it was allocated, with NaN in every
slot of K, V and the scores (and any positions), gives the outputs and scores of one filled with zeros, bit for bit, while the units fill up
from nothing and from a prompt, short of their capacity and beyond it.  Every kernel reads rows before it knows the unit's
length, or fills up a tile with them, and counts them with weight 0 -- which is not enough for NaN."""
import pytest
import torch

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
KINDS = [("bf16", 64), ("bf16", 128), ("f32", 64), ("f32", 128)]
# units of a call: few (8 waves each), more than CUs (4 waves), many short ones (a wave each); budget, prompt, slots to spare
CALLS = [(2, 2, [(48, 0, 7), (48, 20, 0), (64, 64, 0), (33, 33, 1), (33, 31, 0), (700, 311, 7)]), (150, 2, [(48, 20, 7), (200, 130, 0), (41, 40, 1)]),
         (700, 4, [(24, 9, 0), (40, 0, 3), (21, 20, 1)])]


@pytest.fixture(scope="module")
def sqa():
    from paper_2404_04793_amd import binding
    return binding


@pytest.mark.parametrize("blocked", [False, True])
@pytest.mark.parametrize("policy", ["h2o", "streaming"])
@pytest.mark.parametrize("order", ["evict_then_attend", "attend_then_evict"])
@pytest.mark.parametrize("g", [1, 2, 4, 8])
@pytest.mark.parametrize("dtype,D", KINDS)
def test_unwritten_slots_count_nothing(sqa, dtype, D, g, order, policy, blocked):
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator(DEV)
    mk = lambda *shape: torch.randn(*shape, generator=gen, device=DEV).to(tdt)
    for B, H, sizes in CALLS:
        for b, n, spare in sizes:
            got = []
            for fill in (0.0, float("nan")):
                gen.manual_seed(b + n)
                caches = sqa.LayerCaches([b], [b + spare], B, H, D, tdt, DEV, True, blocked=blocked)
                for x in (caches.K[0], caches.V[0], caches.score[0]):
                    x.fill_(fill)
                if fill != 0.0:
                    caches.pos[0].fill_(1 << 30)
                if n > 0:
                    scores = torch.rand(B, H, n, generator=gen, device=DEV)
                    sqa.prefill_compress_layers([mk(B, H, n, D)], [mk(B, H, n, D)], [scores], policy, 4, caches)
                q, k, v = mk(1, B, H * g, D), mk(1, B, H, D), mk(1, B, H, D)
                out, ws = torch.empty_like(q), sqa.decode_workspace(caches, H * g, policy)
                outs = []
                for t in range(3):
                    sqa.decode_step(q, k, v, n + t, policy, 4, caches, out, ws, opts=sqa.batch_opts(order=order))
                    outs.append(out.clone())
                assert sqa.read_device_status(ws) == 0
                length = int(caches.lens[0].min())
                assert length == min(n + 3, b) == int(caches.lens[0].max())
                got.append(outs + ([caches.score[0][..., :length].clone()] if policy == "h2o" else []))
            for x, y in zip(*got):
                assert torch.isfinite(y.float()).all(), (B, H, b, n)
                assert torch.equal(x, y), (B, H, b, n)
