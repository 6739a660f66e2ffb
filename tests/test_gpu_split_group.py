"""Layers of a group whose split passes share a launch: the same bits as with a launch for each (groups of one), for layers of
different lengths, with the pivot-logit filter for none, all or some of them, a short layer between long ones, and layers
planned for other numbers of workgroups.  Run with `-m gpu` on an MI355X."""
import pytest
import torch

from paper_2601_13684_amd import binding as hc
from paper_2601_13684_amd import inputs as I
from paper_2601_13684_amd import runtime as R

pytestmark = pytest.mark.gpu
DEV, D, HKV = "cuda:0", 128, 4
CTX = (33000, 40001, 5000, 65600, 12001)         # two full heads each: the third is too short to share a launch


def stack(G, ctxs):
    g = torch.Generator(device=DEV)
    g.manual_seed(7 + G)
    out = []
    for n in ctxs:
        heads = [[I.HeadSpec(I.ROLE_FULL), I.HeadSpec(I.ROLE_FULL), I.HeadSpec(I.ROLE_SATELLITE, rep=0, sink=5, recent=7, budget=612),
                  I.HeadSpec(I.ROLE_SATELLITE, rep=1, sink=5, recent=7, budget=333)]]
        spec = I.LayerSpec(B=1, Hq=G * HKV, Hkv=HKV, D=D, ctx=[n], heads=heads, window=1, window_mode=0)
        data = I.LayerData()
        for h in range(HKV):
            data.K[(0, h)], data.V[(0, h)] = (torch.randn((n, D), generator=g, device=DEV).to(torch.bfloat16) for _ in range(2))
        lists = {h: torch.randperm(n - 12, generator=g, device=DEV)[:spec.r(0, h)].sort().values.int() + 5 for h in (2, 3)}
        out.append((spec, data, {(0, h): x for h, x in lists.items()}, {(0, h - 2): x for h, x in lists.items()}))
    qs = [torch.randn((len(ctxs), 1, G * HKV, D), generator=g, device=DEV).to(torch.bfloat16) for _ in range(3)]
    return out, qs


def run(made, qs, group, monitor=True, splits=None, **filt):
    cfgs = [R.make_config(s, max_ctx=max(CTX)) for s, *_ in made]
    ctx = R.Context(cfgs[0], DEV, **filt)
    layers = []
    for i, m in enumerate(made):
        if splits:
            hc.hc_set_split(ctx.handle, splits[i])
        layers.append(R.LayerRuntime(ctx, *m, own_scratch=True))
    seen = []
    for q in qs:
        hc.hc_decode_step(ctx.handle, R.make_step_io(layers, q, monitor), len(layers), None, None, group)
        seen += [t.clone() for x in layers for t in (x.out, x.lse, x.topk_idx, x.inter, x.flag, x.slot_pos, x.arena)]
        if monitor and not filt:
            seen += [x.rep_logits.clone() for x in layers]
    torch.cuda.synchronize()
    for x in layers:
        x.close()
    ctx.close()
    return seen


def same(a, b):
    assert len(a) == len(b)
    for i, (x, y) in enumerate(zip(a, b)):
        assert torch.equal(x, y), i


@pytest.mark.parametrize("filt", [None, 1, 36000])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_one_launch_like_a_launch_for_each(G, filt):
    print("split passes of a group", G, filt, flush=True)
    made, qs = stack(G, CTX)
    kw = {} if filt is None else dict(filter_margin=1.25, filter_min_candidates=filt)
    want = run(made, qs, 1, **kw)
    same(run(made, qs, len(CTX), **kw), want)


def test_without_the_monitor_and_two_to_a_group():
    made, qs = stack(4, CTX)
    same(run(made, qs, 2, monitor=False), run(made, qs, 1, monitor=False))


def test_layers_planned_for_other_numbers_of_workgroups():
    """hc_set_split between the layers: a launch is as wide as the widest, the others' surplus workgroups do nothing."""
    made, qs = stack(4, (65600, 65600, 65600))
    same(run(made, qs, 3, splits=(3, 2, 1)), run(made, qs, 1, splits=(3, 2, 1)))
