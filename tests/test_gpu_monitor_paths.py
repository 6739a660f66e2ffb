"""The monitor chooses its launches by the number of candidates and by whether it runs beside the attention pass: every
choice, at the sizes where it changes and where its capacity ends, must give the oracle's lists, overlaps and decisions
bit for bit.  Run with `-m gpu` on an MI355X."""
import numpy as np
import pytest
import torch

from paper_2601_13684_amd import binding as hc
from paper_2601_13684_amd import inputs as I
from paper_2601_13684_amd import runtime as R

import test_gpu_parity as T

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def one_pivot(N, rs, sink=5, recent=7):
    heads = [I.HeadSpec(I.ROLE_FULL)] + [I.HeadSpec(I.ROLE_SATELLITE, rep=0, sink=sink, recent=recent, budget=sink + recent + r) for r in rs]
    return I.LayerSpec(B=1, Hq=4 * len(heads), Hkv=len(heads), D=128, ctx=[N], heads=[heads])


# candidates: one workgroup up to 8192, three launches above; 30,000 list entries of 40,000 candidates take six; a range of
# ties and one of two values need the sampled cut; 700,000 candidates need the baseline bitmap in memory
@pytest.mark.parametrize("N,rs,kind", [(8192 + 12, (700, 3), "normal"), (8193 + 12, (700, 3), "normal"), (8193 + 12, (8193, 1), "ties"),
                                       (40000, (30000, 77), "normal"), (90001, (4097, 256), "all_equal"), (90001, (300, 299), "two_values"),
                                       (700000, (2048,), "normal")])
def test_given_scores_across_the_choices(N, rs, kind):
    T.say("monitor paths", N, rs, kind)
    spec = one_pivot(N, rs)
    rng = np.random.default_rng(N)
    s = {"normal": lambda: rng.normal(size=N), "ties": lambda: rng.integers(0, 9, N) / 8.0, "all_equal": lambda: np.full(N, 0.25),
         "two_values": lambda: (rng.random(N) < 0.002) * 1e30}[kind]().astype(np.float32)
    lo, hi = spec.cand_range(0, 0)
    base = {(0, 0): torch.from_numpy(np.sort(rng.choice(np.arange(lo, hi), spec.k_mon(0, 0), replace=False)).astype(np.int32))}
    ctx, gpu, base_all = T.monitor_case(spec, {(0, 0): s}, base)
    T.compare_monitor(spec, gpu, {(0, 0): s}, base_all)
    for call in range(2):                       # what a call leaves behind in the workspace does not reach the next
        gpu.base_idx[0, :len(base_all[(0, 0)])] = base_all[(0, 0)].to(DEV)
        gpu.ring.zero_()
        gpu.monitor(scores_given=True)
        torch.cuda.synchronize()
        T.compare_monitor(spec, gpu, {(0, 0): s}, base_all)
    gpu.close()
    ctx.close()


@pytest.mark.parametrize("N,margin,flat", [(6001, 0.0, False), (20011, 0.0, False), (20011, 1.25, False), (70001, 0.0, True), (70001, 1.25, True)])
def test_beside_the_attention_pass_like_alone(N, margin, flat):
    """The same steps through hc_decode_step with a side stream (the monitor's small workgroups) and through the three
    calls on one stream (its large ones): the tables must be equal bit for bit.  flat: all keys equal, every score a
    tie."""
    T.say("monitor beside attention", N, margin, "flat" if flat else "")
    tables = []
    for beside in (True, False):
        ws = [I.make_workload(2, layer=l, N=N, scale=0.5) for l in range(2)]
        for w in ws if flat else ():
            for k in w.data.K:
                w.data.K[k][:] = w.data.K[k][:1].clone()
        ctx = R.Context(R.make_config(ws[0].spec), DEV, filter_margin=margin)
        lists = [I.initial_lists(w.spec) for w in ws]
        layers = [R.LayerRuntime(ctx, w.spec, w.data, *l, own_scratch=True) for w, l in zip(ws, lists)]
        q = torch.zeros((2, 1, 32, 128), dtype=torch.bfloat16, device=DEV)
        io = R.make_step_io(layers, q)
        side = torch.cuda.Stream()
        seen = []
        for t in range(4):
            q.copy_(torch.stack([w.schedule.next() for w in ws]).to(DEV))
            if beside:
                hc.hc_decode_step(ctx.handle, io, 2, None, side, 1)
            else:
                for lay, x in zip(layers, q):
                    lay.step(x)
            torch.cuda.synchronize()
            seen.append([x.cpu().numpy().copy() for lay in layers for x in (lay.topk_idx, lay.base_idx, lay.ring, lay.inter, lay.flag, lay.slot_pos, lay.out)])
        tables.append(seen)
        for lay in layers:
            lay.close()
        ctx.close()
    for t, (a, b) in enumerate(zip(*tables)):
        for i, (x, y) in enumerate(zip(a, b)):
            np.testing.assert_array_equal(x, y, err_msg=f"step {t} table {i}")
