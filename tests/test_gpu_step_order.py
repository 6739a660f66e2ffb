"""hc_decode_step called step after step without a wait in between, the side work on a stream of its own: a layer's attention
must find the slots that the previous step refilled, and the monitor the logits and lse of its own step.  The same steps on
one stream give the same bits.  Run with `-m gpu` on an MI355X."""
import pytest
import torch

from paper_2601_13684_amd import binding as hc
from paper_2601_13684_amd import inputs as I
from paper_2601_13684_amd import runtime as R

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
N_LAYERS, STEPS = 3, 8


def run(ws, qs, tier, group, side):
    """Results of the steps: every step's attention outputs (copied in the main stream's order), the tables at the end, and
    how many retrievals there were.  Every layer has buffers of its own: a group's monitor reads its logits while the next
    group's attention writes."""
    ctx = R.Context(R.make_config(ws[0].spec), DEV)
    layers = [R.LayerRuntime(ctx, w.spec, w.data, *I.initial_lists(w.spec), host_tier=tier, own_scratch=True) for w in ws]
    ios = [R.make_step_io(layers, q) for q in qs]
    seen = []
    torch.cuda.synchronize()
    for io in ios:
        hc.hc_decode_step(ctx.handle, io, N_LAYERS, None, side, group)
        seen.append([t.clone() for x in layers for t in (x.out, x.lse)])
    torch.cuda.synchronize()
    for x in layers:
        seen.append([t.clone() for t in (x.topk_idx, x.base_idx, x.ring, x.inter, x.flag, x.arena)])
    fired = sum(x.monitor_counts(0, p)["triggers"] for x, w in zip(layers, ws) for p in w.spec.reps(0))
    for x in layers:
        x.close()
    ctx.close()
    return seen, fired


@pytest.mark.parametrize("tier", [True, False])
@pytest.mark.parametrize("group", [1, 2])
def test_steps_back_to_back_like_one_stream(tier, group):
    print("steps back to back", tier, group, flush=True)
    ws = [I.make_workload(2, layer=l, N=20000, scale=0.2) for l in range(N_LAYERS)]
    g = torch.Generator().manual_seed(5)
    qs = [torch.randn((N_LAYERS, 1, 32, 128), generator=g).to(torch.bfloat16).to(DEV) for _ in range(STEPS)]      # unrelated: every step refills
    want, fired = run(ws, qs, tier, group, None)
    have, fired_side = run(ws, qs, tier, group, torch.cuda.Stream())
    assert fired == fired_side == N_LAYERS * 2 * STEPS
    for step, (a, b) in enumerate(zip(want, have)):
        for i, (x, y) in enumerate(zip(a, b)):
            assert torch.equal(x, y), (step, i)
