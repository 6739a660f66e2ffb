"""The split pass for groups of eight query heads (matrix cores, tiles of 32 rows per wave, 512 staged logits per chunk):
lengths around the edges of tiles, rounds and chunks, the stored pivot logits, and non-finite values.  Run with `-m gpu`
on an MI355X."""
import numpy as np
import pytest
import torch

from oracle import ref
from paper_2601_13684_amd import inputs as I
from paper_2601_13684_amd import runtime as R

import gpu_util as U

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def layer(N, wg=2):
    heads = [I.HeadSpec(I.ROLE_FULL), I.HeadSpec(I.ROLE_SATELLITE, rep=0, sink=0, recent=0, budget=1)]
    spec = I.LayerSpec(B=1, Hq=16, Hkv=2, D=128, ctx=[N], heads=[heads])
    q0 = I.draw_q(spec, N)
    data = I.draw_layer(spec, q0, N + 1, heavy_count=min(3, N), heavy_gain=20.0)
    retrieved, base = I.initial_lists(spec)
    ctx = R.Context(R.make_config(spec), DEV, workgroups_per_cu=wg)
    return spec, data, q0.to(torch.bfloat16), R.LayerRuntime(ctx, spec, data, retrieved, base, host_tier=False), ctx, ref.RefLayer(spec, data, retrieved, base)


# 1 .. 33: one ragged tile; 127 .. 129: a round of four waves; 16 K and 140 K: several chunks of 512 positions per workgroup
@pytest.mark.parametrize("N", [1, 31, 32, 33, 127, 128, 129, 511, 513, 16421, 140001])
def test_lengths_and_stored_logits(N):
    print("group of 8, length", N, flush=True)
    spec, data, q, gpu, ctx, oracle = layer(N)
    for logits in (False, True):
        gpu.out.zero_()
        gpu.attn(q.to(DEV), monitor=logits)
        torch.cuda.synchronize()
        U.check_attention(gpu.out, gpu.lse, oracle.step(q, monitor=False) if not logits else rec, f"N={N}")
        if not logits:
            rec = oracle.step(q, monitor=True)
    got = gpu.rep_logits[0, :N, :].T.cpu().double().numpy()
    # fp32 sums of 128 exact products: at most 128 roundings of 2^-24 of the partial sums, whose size is that of the sum of
    # absolute products, below 12 * 12 * sqrt(128) / sqrt(128) for these inputs
    assert np.abs(got - rec["logits"][(0, 0)]).max() < 2e-5
    assert (gpu.rep_logits[0, N:] == 0).all()
    gpu.close()
    ctx.close()


@pytest.mark.parametrize("value", [float("inf"), float("-inf"), float("nan")])
def test_non_finite_values_stay_in_their_columns(value):
    """One V element is not finite: its column of every head is, every other column is what it was without it (a weight
    is split into parts, and a part that is zero must not turn an infinity of V into something else)."""
    print("group of 8, V element", value, flush=True)
    spec, data, q, gpu, ctx, oracle = layer(3000)
    gpu.attn(q.to(DEV), monitor=False)
    torch.cuda.synchronize()
    want = gpu.out.clone()
    d = gpu.descs[0]
    gpu.arena[d.v_off + 1234 * 128 + 77] = value
    gpu.attn(q.to(DEV), monitor=False)
    torch.cuda.synchronize()
    got = gpu.out
    hit = got[0, :8, 77].cpu().numpy()
    assert np.array_equal(hit, np.full(8, value, np.float32), equal_nan=True)
    rest = torch.ones_like(want, dtype=torch.bool)
    rest[0, :8, 77] = False
    err = (got - want)[rest].abs().max().item()
    assert err <= 1e-5 * want.abs().max().item()           # the same fp32 sums in another order
    gpu.close()
    ctx.close()
