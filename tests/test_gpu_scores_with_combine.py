"""hc_decode_step makes the scores of unfiltered layers of a middle length with the combine pass: the same bits as by hc_decode_attn,
hc_rep_topk_drift and hc_gather_retrieve one after the other.  Run with `-m gpu` on an MI355X."""
import pytest
import torch

from paper_2601_13684_amd import binding as hc
from paper_2601_13684_amd import inputs as I
from paper_2601_13684_amd import runtime as R

pytestmark = pytest.mark.gpu
DEV, D = "cuda:0", 128


def make(G, ctxs, n_full, lists, agg, window=1, window_mode=0, layers=2, seed=0):
    g = torch.Generator(device=DEV)
    g.manual_seed(sum(ctxs) + G + seed)
    hkv, made = n_full + len(lists), []
    for _ in range(layers):
        heads = [[I.HeadSpec(I.ROLE_FULL) for _ in range(n_full)] +
                 [I.HeadSpec(I.ROLE_SATELLITE, rep=j % n_full, sink=3, recent=6, budget=9 + r) for j, r in enumerate(lists)] for _ in ctxs]
        spec = I.LayerSpec(B=len(ctxs), Hq=G * hkv, Hkv=hkv, D=D, ctx=list(ctxs), heads=heads, window=window, window_mode=window_mode, agg=agg)
        data, retrieved, base = I.LayerData(), {}, {}
        for b, n in enumerate(ctxs):
            for h in range(hkv):
                data.K[(b, h)], data.V[(b, h)] = (torch.randn((n, D), generator=g, device=DEV).to(torch.bfloat16) for _ in range(2))
            for j, r in enumerate(lists):
                retrieved[(b, n_full + j)] = torch.randperm(n - 9, generator=g, device=DEV)[:r].sort().values.int() + 3
            for p in range(n_full):
                k = spec.k_mon(b, p)
                base[(b, p)] = torch.randperm(n - 9, generator=g, device=DEV)[:k].sort().values.int() + 3
        made.append((spec, data, retrieved, base))
    qs = [torch.randn((layers, len(ctxs), G * hkv, D), generator=g, device=DEV).to(torch.bfloat16) for _ in range(3)]
    return made, qs


def run(made, qs, how, group=1, side=None, **kw):
    ctx = R.Context(R.make_config(made[0][0]), DEV, **kw)
    layers = [R.LayerRuntime(ctx, *m, own_scratch=True) for m in made]
    seen = []
    for q in qs:
        if how == "step":
            hc.hc_decode_step(ctx.handle, R.make_step_io(layers, q), len(layers), None, side, group)
        else:
            for x, one in zip(layers, q):
                x.attn(one)
            for x in layers:
                x.monitor()
                x.gather()
        torch.cuda.synchronize()
        for x in layers:
            seen += [t.clone() for t in (x.out, x.lse, x.topk_idx, x.base_idx, x.ring, x.inter, x.flag, x.slot_pos, x.arena)]
            for b in range(x.spec.B):
                for p in x.spec.reps(b):
                    lo, hi = x.spec.cand_range(b, p)
                    seen.append(x.scores[x.rep_slot(b, p), lo:hi].clone())
    for x in layers:
        x.close()
    ctx.close()
    return seen


def same(a, b):
    assert len(a) == len(b)
    for i, (x, y) in enumerate(zip(a, b)):
        assert torch.equal(x, y), i


# 9 positions are no candidates.  8,193 candidates, the first range with a histogram; one full head with hundreds of partial results; 65,533 alone; a batch
# with a short sequence; mean logits; lists that one launch does not write at a time
@pytest.mark.parametrize("G,ctxs,n_full,lists,agg", [(4, (8202,), 2, (300, 64), I.AGG_PROB), (4, (16384,), 1, (512,), I.AGG_PROB), (1, (40000,), 1, (700,), I.AGG_PROB),
                                                     (2, (33001, 700, 9001), 2, (300, 64), I.AGG_PROB), (8, (30003,), 2, (2000, 64), I.AGG_PROB), (4, (65542,), 1, (1000, 64), I.AGG_PROB),
                                                     (4, (20001,), 2, (300, 64), I.AGG_LOGIT), (8, (12001, 9000), 1, (300,), I.AGG_LOGIT), (4, (32777,), 1, (16500,), I.AGG_PROB)])
def test_a_step_like_the_three_calls(G, ctxs, n_full, lists, agg):
    print("scores with the combine pass", G, ctxs, lists, agg, flush=True)
    made, qs = make(G, ctxs, n_full, lists, agg)
    want = run(made, qs, "calls")
    same(run(made, qs, "step"), want)
    same(run(made, qs, "step", group=2), want)
    same(run(made, qs, "step", side=torch.cuda.Stream()), want)


def test_more_lists_than_one_launch_takes():
    """Beside the attention pass, eight pivots of three lists each and a range that needs the large form: by survivors."""
    made, qs = make(4, (36000,) + (9000,) * 7, 1, (300, 64, 33), I.AGG_PROB)
    same(run(made, qs, "step", side=torch.cuda.Stream()), run(made, qs, "calls"))


def test_layers_of_a_group_that_filter_and_that_do_not():
    """The filter is on for contexts from 30,000 candidates: one layer's scores come with the combine pass, the other's from the kept rows."""
    short, qs = make(4, (20001,), 1, (300,), I.AGG_PROB, layers=1)
    long, _ = make(4, (40001,), 1, (300,), I.AGG_PROB, layers=1)
    both = [long[0], short[0]]
    qs = [torch.cat([q, q.flip(-1)]) for q in qs]
    kw = dict(filter_margin=1.25, filter_min_candidates=30000)
    a, b = run(both, qs, "step", group=2, **kw), run(both, qs, "calls", **kw)
    n = len(a) // (2 * len(qs))
    for i, (x, y) in enumerate(zip(a, b)):
        if i % n < 9 or (i // n) % 2:                # (a filtered layer's scores are of rows, not of positions)
            assert torch.equal(x, y), i


def test_layers_that_share_a_buffer_of_scores():
    """On one stream, logits their own: their scores are made behind the other's selection, as ever."""
    made, qs = make(4, (20001,), 1, (300,), I.AGG_PROB)
    want = run(made, qs, "calls")
    ctx = R.Context(R.make_config(made[0][0]), DEV)
    layers = [R.LayerRuntime(ctx, *m, own_scratch=True) for m in made]
    layers[1].scores = layers[0].scores
    for q in qs:
        hc.hc_decode_step(ctx.handle, R.make_step_io(layers, q), 2, None, None, 1)
    torch.cuda.synchronize()
    per = len(want) // len(qs) // 2
    for l, x in enumerate(layers):
        for i, t in enumerate((x.out, x.lse, x.topk_idx, x.base_idx, x.ring, x.inter, x.flag, x.slot_pos, x.arena)):
            assert torch.equal(t, want[-2 * per + l * per + i]), (l, i)
        x.close()
    ctx.close()


def touched(x):
    """Where the layer's scores may have been written: its pivots' candidates."""
    m = torch.zeros_like(x.scores, dtype=torch.bool)
    for b in range(x.spec.B):
        for p in x.spec.reps(b):
            lo, hi = x.spec.cand_range(b, p)
            m[x.rep_slot(b, p), lo:hi] = True
    return m


# one workgroup per list, its small and its large form, and the lists by survivors (36,000: more than 20 lists); ranges that begin
# and end beside a multiple of four positions
@pytest.mark.parametrize("ctxs,lists,layers,group", [((20001,), (300, 64), 4, 2), ((40002,), (300, 64), 4, 2), ((36003,) + (9000,) * 7, (300, 64, 33), 2, 1),
                                                     ((9003, 16387, 700), (300,), 4, 2)])
def test_a_reader_on_the_side_stream(ctxs, lists, layers, group):
    """What is put on the side stream between two steps finds the scores of the step before it, however late it runs, and two calls that
    share their layers' buffers of scores do not get in each other's way.  Nothing but candidates is written."""
    made, qs = make(4, ctxs, 1, lists, I.AGG_PROB, layers=layers)
    ctx = R.Context(R.make_config(made[0][0]), DEV)

    def stack():
        xs = [R.LayerRuntime(ctx, *m, own_scratch=True) for m in made]
        for x in xs:
            x.scores.fill_(-7.0)
        return xs

    apart, cut = stack(), stack()
    for a, b in zip(cut[:layers // 2], cut[layers // 2:]):
        b.scores = a.scores
    side = torch.cuda.Stream()
    want, have, last = [], [], []
    for q in qs:
        for x, one in zip(apart, q):
            x.attn(one)
            x.monitor()
            x.gather()
        torch.cuda.synchronize()
        want += [x.scores.clone() for x in apart]
        last = [t.clone() for x in apart for t in (x.out, x.lse, x.topk_idx, x.base_idx, x.inter, x.flag, x.slot_pos, x.arena)]
    for x, w in zip(apart, want[-layers:]):
        assert (w[~touched(x)] == -7.0).all()
    again = stack()
    torch.cuda.synchronize()
    for q in qs:
        hc.hc_decode_step(ctx.handle, R.make_step_io(again, q), layers, None, side, group)
        with torch.cuda.stream(side):
            torch.cuda._sleep(2_000_000)             # later than the next step's attention
            have += [x.scores.clone() for x in again]
    torch.cuda.synchronize()
    same(have, want)
    same([t for x in again for t in (x.out, x.lse, x.topk_idx, x.base_idx, x.inter, x.flag, x.slot_pos, x.arena)], last)
    half = layers // 2
    for q in qs:
        io = R.make_step_io(cut, q)
        parts = [(type(io[0]) * half)(*io[i * half:(i + 1) * half]) for i in range(2)]
        for p in parts:
            hc.hc_decode_step(ctx.handle, p, half, None, side, max(1, group // 2))
    torch.cuda.synchronize()
    same([t for x in cut for t in (x.out, x.lse, x.topk_idx, x.base_idx, x.inter, x.flag, x.slot_pos, x.arena)], last)
    for x in apart + cut + again:
        x.close()
    ctx.close()


def run_on(made, qs, tokens, how, side=None, group=1, room=64):
    """As `run`, every step appending its token (tokens: [steps, layers, 2, B, Hkv, D], or None) and with a re-scored window where the layers have one."""
    spec = made[0][0]
    grow = 0 if tokens is None else room
    ctx = R.Context(R.make_config(spec, max_ctx=(max(spec.ctx) + grow + 63) // 64 * 64), DEV)
    layers = [R.LayerRuntime(ctx, *m, own_scratch=True, growth=grow) for m in made]
    seen, counts = [], []
    for t, q in enumerate(qs):
        if how == "step":
            io = R.make_step_io(layers, q)
            for l in range(len(layers) if grow else 0):
                io[l].k_new, io[l].v_new = (x.data_ptr() for x in tokens[t, l])
            hc.hc_decode_step(ctx.handle, io, len(layers), None, side, group)
        else:
            for l, (x, one) in enumerate(zip(layers, q)):
                if grow:
                    x.append(tokens[t, l, 0], tokens[t, l, 1])
                x.attn(one)
                if x.q_window is not None:
                    x.rescore(one)
                x.monitor()
                x.gather()
        torch.cuda.synchronize()
        for x in layers:
            seen += [y.clone() for y in (x.out, x.lse, x.topk_idx, x.base_idx, x.ring, x.inter, x.flag, x.slot_pos, x.arena)]
            for b in range(x.spec.B):
                for p in x.spec.reps(b):
                    lo, hi = x.spec.cand_range(b, p)
                    seen.append(x.scores[x.rep_slot(b, p), lo:hi + (t + 1 if grow else 0)].clone())
                    counts.append(x.monitor_counts(b, p)["tests"])
    for x in layers:
        x.close()
    ctx.close()
    return seen, counts


def drawn_tokens(spec, steps, layers, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return torch.randn((steps, layers, 2, spec.B, spec.Hkv, D), generator=g, device=DEV).to(torch.bfloat16)


# windows of four steps, twice over and one step more; with a fixed context and a growing one; two pivots, and a batch with a sequence that is short
@pytest.mark.parametrize("G,ctxs,n_full,lists", [(4, (20001,), 2, (300, 64)), (2, (12000, 9000, 700), 1, (300,)), (8, (33000,), 1, (2000,))])
@pytest.mark.parametrize("grow", [False, True])
def test_a_step_with_a_rescored_window_like_the_calls(G, ctxs, n_full, lists, grow):
    """The combine pass keeps the step's queries and scores, and the re-scoring passes come between it and the selection that reads its histogram."""
    print("scores with the combine pass, re-scored window", G, ctxs, lists, grow, flush=True)
    made, _ = make(G, ctxs, n_full, lists, I.AGG_PROB, window=4, window_mode=2, layers=4)
    g = torch.Generator(device=DEV)
    g.manual_seed(11 + G)
    spec = made[0][0]
    qs = [torch.randn((4, spec.B, spec.Hq, D), generator=g, device=DEV).to(torch.bfloat16) for _ in range(9)]
    tokens = drawn_tokens(spec, len(qs), 4, 12 + G) if grow else None
    want, counts = run_on(made, qs, tokens, "calls")
    assert max(counts) == 2                          # windows tested
    for side, group in ((torch.cuda.Stream(), 2), (None, 2), (torch.cuda.Stream(), 1), (None, 4)):
        have, n = run_on(made, qs, tokens, "step", side, group)
        same(have, want)
        assert n == counts


# 9 positions are no candidates: 8,190 to 8,196 of them, the line being at 8,192, and 65,530 to 65,536, the line at 65,533; two layers, one of which
# crosses it two steps later
@pytest.mark.parametrize("first,lists", [(8198, (300, 64)), (65538, (700, 300))])
def test_layers_that_grow_into_and_out_of_the_range(first, lists):
    print("scores with the combine pass, growing from", first, flush=True)
    long, _ = make(4, (first,), 1, lists, I.AGG_PROB, layers=1)
    short, _ = make(4, (first - 2,), 1, lists, I.AGG_PROB, layers=1, seed=5)
    made = [long[0], short[0]]
    g = torch.Generator(device=DEV)
    g.manual_seed(first)
    spec = made[0][0]
    qs = [torch.randn((2, 1, spec.Hq, D), generator=g, device=DEV).to(torch.bfloat16) for _ in range(9)]
    tokens = drawn_tokens(spec, len(qs), 2, first + 1)
    want, _ = run_on(made, qs, tokens, "calls")
    for side, group in ((torch.cuda.Stream(), 1), (None, 1), (None, 2)):
        same(run_on(made, qs, tokens, "step", side, group)[0], want)
