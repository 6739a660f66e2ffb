"""The layers of a hc_decode_step group are combined with one launch: the results are those of the layers one by one, also
where layers share an output buffer (the last one's stay).  Run with `-m gpu` on an MI355X."""
import pytest
import torch

from paper_2601_13684_amd import binding as hc
from paper_2601_13684_amd import inputs as I
from paper_2601_13684_amd import runtime as R

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.mark.parametrize("n,group,shared", [(1, 1, ()), (3, 3, ()), (8, 8, ()), (9, 4, ()), (4, 4, (0, 2)), (5, 5, (1, 2, 4))])
def test_group_like_layer_by_layer(n, group, shared):
    print("combine", n, group, shared, flush=True)
    ws = [I.make_workload(2, layer=l, N=3001 + 64 * 7, scale=0.2) for l in range(n)]
    ctx = R.Context(R.make_config(ws[0].spec), DEV)
    layers = [R.LayerRuntime(ctx, w.spec, w.data, *I.initial_lists(w.spec), host_tier=False) for w in ws]
    q = torch.stack([w.schedule.next() for w in ws]).to(DEV)
    want = []
    for lay, x in zip(layers, q):
        lay.attn(x, monitor=False)
        torch.cuda.synchronize()
        want.append((lay.out.clone(), lay.lse.clone()))
    for lay in layers:
        lay.out.zero_()
        lay.lse.zero_()
    for l in shared[1:]:
        layers[l].out, layers[l].lse = layers[shared[0]].out, layers[shared[0]].lse
    io = R.make_step_io(layers, q, monitor=False)
    hc.hc_decode_step(ctx.handle, io, n, None, None, group)
    torch.cuda.synchronize()
    for l, lay in enumerate(layers):
        k = shared[-1] if l in shared else l
        assert torch.equal(lay.out, want[k][0]) and torch.equal(lay.lse, want[k][1]), l
    for lay in layers:
        lay.close()
    ctx.close()
