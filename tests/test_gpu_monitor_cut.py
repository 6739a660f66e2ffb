"""What the monitor cuts a long candidate range down by does not depend on how the scores are distributed: near-equal and equal
scores, lists on both sides of the line between one workgroup per list and the launches of long lists, groups of eight heads,
more kept rows than one workgroup has room for.  Lists, overlaps and decisions bit for bit, and no call several times slower than
one whose scores are spread out.  Run with `-m gpu` on an MI355X."""
import numpy as np
import pytest
import torch

from paper_2601_13684_amd import binding as hc
from paper_2601_13684_amd import inputs as I
from paper_2601_13684_amd import runtime as R

import test_gpu_parity as T
from test_gpu_monitor_paths import one_pivot

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def draw(kind, N, rng):
    if kind == "equal":
        return np.full(N, 1.0 / N, dtype=np.float32)
    if kind == "tied":                               # 40 values, the largest in one place
        return (np.sort(rng.integers(0, 40, N))[::-1] / 40.0 + 1.0).astype(np.float32)
    if kind == "special":                            # NaN, infinities, both zeros among near-equal scores
        s = np.exp(rng.normal(size=N) * 0.02).astype(np.float32)
        s[rng.choice(N, N // 8, replace=False)] = np.nan
        s[rng.choice(N, 300, replace=False)] = np.inf
        s[rng.choice(N, 300, replace=False)] = -np.inf
        s[rng.choice(N, 300, replace=False)] = -0.0
        return s
    return (np.exp(rng.normal(size=N) * {"flat": 0.02, "flatter": 1e-6, "spread": 1.0}[kind]) / N).astype(np.float32)


# 40,000 candidates: 13,000 survivors are expected at a longest list of about 11,300; 131,072: about 10,000.  The odd
# ranges end in the middle of a chunk, of a sample's piece and of four positions.
@pytest.mark.parametrize("N,rs,kind", [(8193 + 12, (1, 8192), "flat"), (8195 + 12, (700, 3), "equal"), (40003, (11000, 77), "flat"), (40003, (11600, 77), "flat"),
                                       (40003, (11600, 77), "equal"), (40003, (11600, 300, 2), "tied"), (90001, (4097, 256, 1), "special"),
                                       (131073, (8192, 4096, 2048), "flatter"), (131073, (8192, 1), "tied"), (131073, (16384, 100), "flat"),
                                       (131073, (16384, 8192, 4096, 2048), "spread"), (131073, (30000, 1), "special"),
                                       (229376, (7872, 3776, 1728, 704), "flat"), (229376, (7872, 704), "equal"), (600011, (20000, 3), "equal")])
def test_given_scores_whatever_their_distribution(N, rs, kind):
    T.say("monitor cut", N, rs, kind)
    spec = one_pivot(N, rs)
    rng = np.random.default_rng(N + len(rs))
    s = draw(kind, N, rng)
    lo, hi = spec.cand_range(0, 0)
    base = {(0, 0): torch.from_numpy(np.sort(rng.choice(np.arange(lo, hi), spec.k_mon(0, 0), replace=False)).astype(np.int32))}
    ctx, gpu, base_all = T.monitor_case(spec, {(0, 0): s}, base)
    s = np.where(np.isnan(s), np.float32(-np.inf), s)       # the oracle takes no NaN; no list here reaches down to them
    T.compare_monitor(spec, gpu, {(0, 0): s}, base_all)
    for call in range(2):                       # what a call leaves behind in the workspace does not reach the next
        gpu.base_idx[0, :len(base_all[(0, 0)])] = base_all[(0, 0)].to(DEV)
        gpu.ring.zero_()
        gpu.monitor(scores_given=True)
        torch.cuda.synchronize()
        T.compare_monitor(spec, gpu, {(0, 0): s}, base_all)
    gpu.close()
    ctx.close()


def test_short_and_long_lists_in_turn():
    """The two ways share a workspace: calls of two layers of one context, one of each kind, in turn."""
    N, rng = 60001, np.random.default_rng(5)
    ctx = None
    cases = []
    for rs in ((3000, 50), (20000, 900)):
        spec = one_pivot(N, rs)
        lo, hi = spec.cand_range(0, 0)
        k = spec.k_mon(0, 0)
        base = torch.from_numpy(np.sort(rng.choice(np.arange(lo, hi), k, replace=False)).astype(np.int32))
        ctx = ctx or R.Context(R.make_config(one_pivot(N, (20000, 900))), DEV)
        kv = torch.zeros((N, 128), dtype=torch.bfloat16)
        data = I.LayerData({(0, h): kv for h in range(spec.Hkv)}, {(0, h): kv for h in range(spec.Hkv)}, {})
        retrieved, _ = I.initial_lists(spec)
        gpu = R.LayerRuntime(ctx, spec, data, retrieved, {(0, 0): base}, host_tier=False, own_scratch=True)
        cases.append((spec, gpu, {(0, 0): base}))
    for kind in ("spread", "flat", "equal", "spread"):
        for spec, gpu, base in cases:
            s = draw(kind, N, rng)
            gpu.scores[0, :N] = torch.from_numpy(s).to(DEV)
            gpu.base_idx[0, :base[(0, 0)].numel()] = base[(0, 0)].to(DEV)
            gpu.ring.zero_()
            gpu.monitor(scores_given=True)
            torch.cuda.synchronize()
            T.compare_monitor(spec, gpu, {(0, 0): s}, base)
    for _, gpu, _ in cases:
        gpu.close()
    ctx.close()


@pytest.mark.parametrize("N,rs", [(20011, (3000, 77)), (40003, (3000, 77)), (229376, (7872, 704))])
def test_a_sample_that_misleads(N, rs):
    """The sampled candidates (one of each of 4,096 equal pieces, at a scattered place) are the best ones of a range of near-equal
    scores: the estimated cut then lets fewer through than the longest list needs, and the whole range is selected from."""
    T.say("monitor cut misled", N, rs)
    spec = one_pivot(N, rs)
    lo, hi = spec.cand_range(0, 0)
    n, i = hi - lo, np.arange(4096, dtype=np.uint64)
    a, b = i * np.uint64(n) // np.uint64(4096), (i + np.uint64(1)) * np.uint64(n) // np.uint64(4096)
    sampled = (a + (((i * np.uint64(2654435761)) & np.uint64(0xffffffff)) * (b - a) >> np.uint64(32))).astype(np.int64)
    rng = np.random.default_rng(N)
    s = (1.0 + 0.01 * rng.random(N)).astype(np.float32)
    s[lo + sampled] += np.float32(0.02)
    t = rs[0] * 4096 / n
    assert t + 5 * np.sqrt(t) + 8 < rs[0]
    base = {(0, 0): torch.from_numpy(np.sort(rng.choice(np.arange(lo, hi), spec.k_mon(0, 0), replace=False)).astype(np.int32))}
    ctx, gpu, base_all = T.monitor_case(spec, {(0, 0): s}, base)
    T.compare_monitor(spec, gpu, {(0, 0): s}, base_all)
    gpu.close()
    ctx.close()


@pytest.mark.parametrize("rs", [(3000, 77), (11600, 77)])
def test_captured_call_replays_like_eager(rs):
    """One captured call, replayed over scores of every kind with eager work and an eager call between the replays."""
    N, rng = 40003, np.random.default_rng(8)
    T.say("monitor cut captured", rs)
    spec = one_pivot(N, rs)
    lo, hi = spec.cand_range(0, 0)
    base = {(0, 0): torch.from_numpy(np.sort(rng.choice(np.arange(lo, hi), spec.k_mon(0, 0), replace=False)).astype(np.int32))}
    ctx, gpu, base_all = T.monitor_case(spec, {(0, 0): draw("spread", N, rng)}, base)
    cap = torch.cuda.Stream()
    cap.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(cap):
        with torch.cuda.graph(graph, stream=cap):
            gpu.monitor(scores_given=True)
    torch.cuda.synchronize()
    junk = torch.zeros((1 << 20,), device=DEV)
    for kind in ("spread", "flat", "equal", "tied", "spread"):
        s = draw(kind, N, rng)
        for call in (graph.replay, graph.replay, lambda: gpu.monitor(scores_given=True)):
            gpu.scores[0, :N] = torch.from_numpy(s).to(DEV)
            gpu.base_idx[0, :len(base_all[(0, 0)])] = base_all[(0, 0)].to(DEV)
            gpu.ring.zero_()
            junk.add_(1.0)
            torch.cuda.synchronize()
            call()
            torch.cuda.synchronize()
            T.compare_monitor(spec, gpu, {(0, 0): s}, base_all)
    gpu.close()
    ctx.close()


def stack_spec(N, budgets, G):
    heads = [I.HeadSpec(I.ROLE_FULL), I.HeadSpec(I.ROLE_FULL)] + [I.HeadSpec(I.ROLE_SATELLITE, rep=j % 2, sink=5, recent=7, budget=12 + r) for j, r in enumerate(budgets)]
    return I.LayerSpec(B=1, Hq=G * len(heads), Hkv=len(heads), D=128, ctx=[N], heads=[heads])


# unrelated queries at every step: a set filter's check fails or more rows than expected are kept, and the launches
# that stand by decide
@pytest.mark.parametrize("N,budgets,G,margin,scale", [(30011, (700, 3000), 8, 0.0, 1.0), (30011, (9000, 3000), 8, 0.0, 0.02), (30011, (700, 3000), 8, 1.25, 1.0),
                                                      (30011, (13000, 3000), 4, 0.0, 0.02), (40011, (3000, 500), 4, 1.25, 1.0),
                                                      (40011, (3000, 500), 4, 1.25, 0.02), (70001, (16000, 2000), 4, 1.25, 1.0),
                                                      (70001, (16000, 2000), 4, 1.25, 0.02), (40011, (15000, 500), 2, 1.25, 1.0)])
def test_beside_the_attention_pass_like_alone(N, budgets, G, margin, scale):
    """Steps through hc_decode_step with a side stream and through the three calls on one stream without the filter: equal bits."""
    T.say("monitor cut beside attention", N, budgets, G, margin, scale)
    specs = [stack_spec(N, budgets, G) for _ in range(2)]
    datas = [I.draw_layer(s, I.draw_q(s, 3 + l, DEV), 11 + l, DEV) for l, s in enumerate(specs)]
    g = torch.Generator(device=DEV)
    g.manual_seed(N)
    qs = [(torch.randn((2, 1, specs[0].Hq, 128), generator=g, device=DEV) * scale).to(torch.bfloat16) for _ in range(4)]
    tables, fell = [], 0
    for beside in (True, False):
        ctx = R.Context(R.make_config(specs[0]), DEV, filter_margin=margin if beside else 0.0)
        layers = [R.LayerRuntime(ctx, s, d, *I.initial_lists(s), host_tier=False, own_scratch=True) for s, d in zip(specs, datas)]
        side = torch.cuda.Stream()
        seen = []
        for q in qs:
            if beside:
                hc.hc_decode_step(ctx.handle, R.make_step_io(layers, q), 2, None, side, 1)
            else:
                for lay, x in zip(layers, q):
                    lay.step(x)
            torch.cuda.synchronize()
            seen.append([x.cpu().numpy().copy() for lay in layers for x in (lay.topk_idx, lay.base_idx, lay.ring, lay.inter, lay.flag, lay.out)])
        if beside:
            fell = sum(lay.monitor_counts(0, h)["fallbacks"] for lay in layers for h in range(2))
        tables.append(seen)
        for lay in layers:
            lay.close()
        ctx.close()
    assert not margin or budgets[0] > 10000 or fell > 0      # (the longer lists keep enough rows to be decided over them)
    for t, (a, b) in enumerate(zip(*tables)):
        for i, (x, y) in enumerate(zip(a, b)):
            np.testing.assert_array_equal(x, y, err_msg=f"step {t} table {i}")


def test_time_does_not_depend_on_the_distribution():
    """229,376 candidates, lists of 7,872 and shorter: near-equal and equal scores take at most three times what spread-out ones
    take (measured: 1.5 and 1.9 times; 10 and 12 times when the range was not cut down)."""
    N = 229376
    spec = one_pivot(N, (7872, 3776, 1728))
    us = {}
    for kind in ("spread", "flat", "equal"):
        ctx, gpu, _ = T.monitor_case(spec, {(0, 0): draw(kind, N, np.random.default_rng(1))}, I.initial_lists(spec)[1])
        best = []
        for _ in range(5):
            a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            a.record()
            for _ in range(20):
                gpu.monitor(scores_given=True)
            b.record()
            torch.cuda.synchronize()
            best.append(a.elapsed_time(b) / 20 * 1e3)
        us[kind] = min(best)
        gpu.close()
        ctx.close()
    T.say("monitor time by distribution", {k: round(v, 1) for k, v in us.items()})
    assert us["flat"] < 3 * us["spread"] and us["equal"] < 3 * us["spread"], us
