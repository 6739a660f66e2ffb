"""Unfiltered layers of 32K to 64K candidates in hc_decode_step with a side stream: the lists by mon_direct's large form beside the
attention pass, at the ends of its range and with more lists than it is used for.  The same bits as with everything on one
stream.  Run with `-m gpu` on an MI355X."""
import pytest
import torch

from paper_2601_13684_amd import binding as hc
from paper_2601_13684_amd import inputs as I
from paper_2601_13684_amd import runtime as R

pytestmark = pytest.mark.gpu
DEV, D, HKV = "cuda:0", 128, 4


def run(made, qs, G, group, side):
    ctx = R.Context(R.make_config(made[0][0]), DEV)
    layers = [R.LayerRuntime(ctx, *m, own_scratch=True) for m in made]
    seen = []
    for q in qs:
        hc.hc_decode_step(ctx.handle, R.make_step_io(layers, q), len(layers), None, side, group)
    torch.cuda.synchronize()
    for x in layers:
        seen += [t.clone() for t in (x.out, x.lse, x.topk_idx, x.base_idx, x.ring, x.inter, x.flag, x.slot_pos, x.arena)]
        x.close()
    ctx.close()
    return seen


# 4 + 7 positions are no candidates: 32,766 (the first the small form has no room for) and 65,533 candidates, one more, and lists of
# thousands; three sequences (18 lists), four (24: not this form)
@pytest.mark.parametrize("G,ctxs,lists", [(4, (32777,), (700, 300)), (4, (65544,), (9000, 3)), (4, (65545,), (700, 300)), (1, (40001,), (4096, 4096)),
                                          (8, (50000,), (700, 300)), (2, (36000, 65544, 1000), (700, 300, 64)), (4, (36000, 20000, 9000, 1000), (700, 300, 64))])
def test_lists_beside_the_attention_pass(G, ctxs, lists):
    print("beside", G, ctxs, lists, flush=True)
    g = torch.Generator(device=DEV)
    g.manual_seed(sum(ctxs) + G)
    made = []
    for _ in range(2):
        heads = [[I.HeadSpec(I.ROLE_FULL)] + [I.HeadSpec(I.ROLE_SATELLITE, rep=0, sink=4, recent=7, budget=11 + r) for r in lists] for _ in ctxs]
        hkv = 1 + len(lists)
        spec = I.LayerSpec(B=len(ctxs), Hq=G * hkv, Hkv=hkv, D=D, ctx=list(ctxs), heads=heads, window=1, window_mode=0)
        data, retrieved, base = I.LayerData(), {}, {}
        for b, n in enumerate(ctxs):
            for h in range(hkv):
                data.K[(b, h)], data.V[(b, h)] = (torch.randn((n, D), generator=g, device=DEV).to(torch.bfloat16) for _ in range(2))
            for h, r in enumerate(lists, 1):
                retrieved[(b, h)] = torch.randperm(n - 11, generator=g, device=DEV)[:r].sort().values.int() + 4
            base[(b, 0)] = retrieved[(b, 1 + lists.index(max(lists)))]
        made.append((spec, data, retrieved, base))
    qs = [torch.randn((2, len(ctxs), G * hkv, D), generator=g, device=DEV).to(torch.bfloat16) for _ in range(3)]
    want, have = run(made, qs, G, 1, None), run(made, qs, G, 1, torch.cuda.Stream())
    for i, (x, y) in enumerate(zip(want, have)):
        assert torch.equal(x, y), i
