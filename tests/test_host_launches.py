"""The launches that the host side makes, and what it does when one fails, on a stand-in for the HIP runtime (fake_hip.cpp) in a
process of its own.  No GPU needed."""
import os
import subprocess
import sys
import textwrap

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    so = str(tmp_path_factory.mktemp("fake_hip") / "libfakehip.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", "-Wno-deprecated-declarations",
                    os.path.join(HERE, "fake_hip.cpp"), "-o", so], check=True)
    return so


PROLOGUE = '''
import ctypes as C, sys, types
torch = types.ModuleType("torch")            # the binding only needs the name: its pointers are plain addresses here
torch.Tensor = type("Tensor", (), {})
torch.cuda = types.SimpleNamespace(Stream=type("Stream", (), {}), Event=type("Event", (), {}))
sys.modules["torch"] = torch
sys.path.insert(0, ROOT)
fake = C.CDLL(FAKE, mode=C.RTLD_GLOBAL)
fake.fake_log.restype = C.c_char_p
from paper_2601_13684_amd import binding as hc
L = hc.lib()
def log():
    return [l.split() for l in fake.fake_log().decode().splitlines()]
def layer(ctx, N, r, n=4):
    """One pivot and n - 1 satellites of r retrieved slots."""
    descs = (hc.hc_head_desc * n)()
    for h in range(n):
        ln = N if h == 0 else 12 + r
        descs[h] = hc.hc_head_desc(k_off=h * (1 << 26), v_off=h * (1 << 26) + (1 << 25), tier_off=h * (1 << 27), ctx=N, len=ln, role=0 if h == 0 else 1,
                                   rep=-1 if h == 0 else 0, sink=0 if h == 0 else 5, recent=0 if h == 0 else 7, k_mon=0, cap=0)
    out = C.c_void_p()
    assert L.hc_layer_create(ctx, descs, C.byref(out)) == 0, L.hc_last_error(ctx)
    return out.value
def context(N, r, G=4, n=4):
    cfg = hc.hc_config(B=1, Hq=G * n, Hkv=n, D=128, max_ctx=(N + 63) // 64 * 64, max_k=r, window=1, metric=0, tau_num=1, tau_den=2, agg=0, window_mode=0)
    out = C.c_void_p()
    assert L.hc_create(C.byref(cfg), C.byref(out)) == 0
    return out.value
def io_of(layers):
    """Addresses that nothing reads: a launch is only written down."""
    arr = (hc.hc_layer_io * len(layers))()
    for i, l in enumerate(layers):
        a = lambda k: (1 << 40) + (i << 34) + (k << 28)
        arr[i] = hc.hc_layer_io(layer=l, kv_arena=a(0), host_tier=a(1), q=a(2), out=a(3), lse=a(4), rep_logits=a(5), scores=a(6), topk_idx=a(7), base_idx=a(8),
                                ring=a(9), inter=a(10), flag=a(11), slot_pos=a(12))
    return arr
'''


def run(fake, body):
    code = f"ROOT, FAKE = {ROOT!r}, {fake!r}\n" + PROLOGUE + textwrap.dedent(body)
    r = subprocess.run([sys.executable, "-c", code], stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True, timeout=120)
    assert r.returncode == 0, r.stdout
    return r.stdout


def test_a_failed_launch_leaves_the_layers_before_it_combined(fake):
    """Four layers in one group, the third one's split pass fails: the first two are combined, in one launch, and nothing of the
    group follows."""
    run(fake, """
        ctx = context(5000, 300)
        layers = [layer(ctx, 5000, 300) for _ in range(4)]
        fake.fake_reset(3)
        assert L.hc_decode_step(ctx, io_of(layers), 4, 4, None, None) == hc.HC_EHIP
        names = [(l[0], int(l[3])) for l in log()]
        assert [n for n, z in names if "attn_split" in n] == [names[0][0]] * 2, names
        assert len(names) == 3 and "attn_combine" in names[2][0] and names[2][1] == 2, names
        fake.fake_reset(0)
        assert L.hc_decode_step(ctx, io_of(layers), 4, 4, None, None) == 0
        names = [(l[0], int(l[3])) for l in log()]
        assert sum("attn_split" in n for n, z in names) == 4 and [z for n, z in names if "attn_combine" in n] == [4], names
    """)


def test_the_gather_shape_goes_back_to_automatic(fake):
    """A set launch shape holds alone and on the side stream; with 0 workgroups each has its own default again."""
    run(fake, """
        ctx = context(30000, 6000)
        layers = [layer(ctx, 30000, 6000) for _ in range(2)]
        def grids():
            fake.fake_reset(0)
            assert L.hc_decode_step(ctx, io_of(layers), 2, 1, None, C.c_void_p(77)) == 0
            assert L.hc_decode_step(ctx, io_of(layers[:1]), 1, 1, None, None) == 0
            return [int(l[1]) for l in log() if "gather" in l[0]]
        first = grids()
        assert first == [48, 48, 96], first
        assert L.hc_set_gather_shape(ctx, 30, 64) == 0 and grids() == [30, 30, 30]
        assert L.hc_set_gather_shape(ctx, 0, 256) == 0 and grids() == first
        assert L.hc_set_gather_shape(ctx, -1, 256) == hc.HC_EINVAL and L.hc_set_gather_shape(ctx, 4097, 256) == hc.HC_EINVAL
    """)


@pytest.mark.parametrize("G,N", [(4, 306816), (8, 224896)])
def test_the_longest_context_whose_refill_is_planned_by_bitmaps(fake, G, N):
    """Beside the attention pass: bitmaps of 75 KB (groups of eight heads: 55 KB) with their masks, next to which the satellites' first
    rows still find room."""
    run(fake, f"""
        names = []
        def long_layer(ctx, N):
            descs = (hc.hc_head_desc * 4)()
            for h in range(4):
                descs[h] = hc.hc_head_desc(k_off=h * (1 << 28), v_off=h * (1 << 28) + (1 << 27), tier_off=h * (1 << 28), ctx=N, len=N if h == 0 else 312,
                                           role=0 if h == 0 else 1, rep=-1 if h == 0 else 0, sink=0 if h == 0 else 5, recent=0 if h == 0 else 7, k_mon=0, cap=0)
            out = C.c_void_p()
            assert L.hc_layer_create(ctx, descs, C.byref(out)) == 0, L.hc_last_error(ctx)
            return out.value
        for n in ({N}, {N} + 8192):
            ctx = context(n, 300, G={G})
            layers = [long_layer(ctx, n) for _ in range(2)]
            fake.fake_reset(0)
            assert L.hc_decode_step(ctx, io_of(layers), 2, 1, None, C.c_void_p(77)) == 0
            names.append([l[0] for l in log() if "gather" in l[0]])
        assert all("plan_bitmap" in x for x in names[0]) and len(names[0]) == 2, names
        assert not any("plan_bitmap" in x for x in names[1]) and len(names[1]) == 4, names
    """)


@pytest.mark.parametrize("r,kernel", [(300, "mon_selectILi512ELi1E"), (4096, "mon_selectILi512ELi1E"), (4097, "mon_directILi512ELi1E"), (9000, "mon_directILi512ELi1E")])
def test_what_selects_among_the_kept_rows_beside_the_attention_pass(fake, r, kernel):
    """Once the filter is set: mon_select for lists of up to 4,096, mon_direct for longer ones; alone mon_direct for both."""
    run(fake, f"""
        ctx = context(70000, {r})
        assert L.hc_set_logit_filter(ctx, C.c_float(1.25), 0) == 0
        layers = [layer(ctx, 70000, {r}) for _ in range(2)]
        for side in (77, 77, None):
            fake.fake_reset(0)
            assert L.hc_decode_step(ctx, io_of(layers), 2, 1, None, C.c_void_p(side)) == 0
            names = [l[0] for l in log() if "mon_" in l[0] and "ELi3" not in l[0]]
            if side is None:
                assert sum("mon_directILi1024ELi1E" in n for n in names) == 2, names
        fake.fake_reset(0)
        assert L.hc_decode_step(ctx, io_of(layers), 2, 1, None, C.c_void_p(77)) == 0
        names = [l[0] for l in log() if "mon_" in l[0]]
        assert sum("{kernel}" in n for n in names) == 2 and len(names) == 6, names
    """)


def test_workgroups_of_a_refill_beside_the_attention_pass(fake):
    """48 where few satellites or many layers share a launch, 96 for groups of up to four layers with more than 24 satellites."""
    run(fake, """
        def gathers(n_heads, group, layers_n):
            ctx = context(30000, 600, n=n_heads)
            layers = [layer(ctx, 30000, 600, n=n_heads) for _ in range(layers_n)]
            fake.fake_reset(0)
            assert L.hc_decode_step(ctx, io_of(layers), layers_n, group, None, C.c_void_p(77)) == 0
            return [int(l[1]) for l in log() if "gather" in l[0]]
        assert gathers(13, 2, 4) == [48, 48]          # 24 satellites
        assert gathers(14, 2, 4) == [96, 96]          # 26
        assert gathers(8, 4, 8) == [96, 96]           # 28
        assert gathers(8, 5, 10) == [48, 48]          # 35 in a group of five
    """)


def test_long_layers_of_a_group_share_a_launch_of_the_split_pass(fake):
    """Layers whose pass fills the GPU: one launch for the group; a short layer between them, or buffers that two of them share, part
    it; with timing events set every layer has its own; if the shared launch fails, the layers before it are combined."""
    run(fake, """
        ctx = context(70000, 300)
        long = [layer(ctx, 70000, 300) for _ in range(4)]
        short = layer(ctx, 5000, 300)
        def splits(layers, io=None):
            fake.fake_reset(0)
            assert L.hc_decode_step(ctx, io or io_of(layers), len(layers), 8, None, None) == 0
            return [int(l[2]) for l in log() if "attn_split" in l[0]], [int(l[3]) for l in log() if "attn_combine" in l[0]]
        assert splits(long) == ([4], [4])
        assert splits(long[:1]) == ([1], [1])
        assert splits(long[:2] + [short] + long[2:]) == ([2, 1, 2], [5])
        io = io_of(long)
        io[2].out = io[1].out
        assert splits(long, io) == ([2, 2], [2, 2])
        ev = (C.c_void_p * 4)(1, 2, 3, 4)
        assert L.hc_set_timing_events(ctx, ev, ev, 4) == 0
        assert splits(long) == ([1, 1, 1, 1], [4])
        assert splits(long) == ([4], [4])
        fake.fake_reset(3)                           # the third launch: the two long layers behind the short one
        assert L.hc_decode_step(ctx, io_of(long[:2] + [short] + long[2:]), 5, 8, None, None) == hc.HC_EHIP
        names = [(l[0], int(l[2]), int(l[3])) for l in log()]
        assert [y for n, y, z in names if "attn_split" in n] == [2, 1] and "attn_combine" in names[2][0] and names[2][2] == 3 and len(names) == 3, names
    """)


def test_a_short_pass_of_a_group_of_eight_is_not_tuned(fake):
    """Its plan has no weights to measure, whatever its number of workgroups and their length (one to a compute unit, of up to 31
    granules): hc_layer_tune leaves it as it is."""
    run(fake, """
        seen = 0
        for N in range(137000, 138000, 100):
            ctx = context(N, 300, G=8)
            x = layer(ctx, N, 300)
            nb = L.hc_layer_num_workgroups(x)
            assert nb <= 256
            if nb % 16 == 0 and N // 32 >= 16 * nb:
                seen += 1
                before = [C.c_float(0) for _ in range(16)]
                fake.fake_reset(0)
                assert L.hc_layer_tune(ctx, x, C.c_void_p(1 << 40), C.c_void_p(1 << 41), C.c_void_p(1 << 42), C.c_void_p(1 << 43), None, 2, None) == 0
                assert log() == []
        assert seen
    """)


@pytest.mark.parametrize("N,n,kernel", [(32777, 4, "mon_directILi512ELi0E"), (32778, 4, "mon_directILi1024ELi0E"), (65545, 4, "mon_directILi1024ELi0E"),
                                        (65600, 4, "mon_selectILi512ELi2E")])
def test_what_selects_among_long_ranges_beside_the_attention_pass(fake, N, n, kernel):
    """Unfiltered, few lists: mon_direct's small form up to 32,765 candidates (N - 12), its large one up to 65,533."""
    run(fake, f"""
        ctx = context({N}, 300, n={n})
        layers = [layer(ctx, {N}, 300, n={n}) for _ in range(2)]
        fake.fake_reset(0)
        assert L.hc_decode_step(ctx, io_of(layers), 2, 1, None, C.c_void_p(77)) == 0
        names = [l[0] for l in log() if "mon_" in l[0]]
        assert sum("{kernel}" in n for n in names) == 2, names
    """)


@pytest.mark.parametrize("N,kernel,scored", [(8204, "mon_directILi1024ELi3E", False), (8205, "mon_directILi1024ELi0E", True),
                                             (65545, "mon_directILi1024ELi0E", True), (65546, "mon_selectILi1024ELi2E", False)])
def test_which_steps_score_with_the_combine_pass(fake, N, kernel, scored):
    """Ranges that mon_direct takes from a histogram: no launch of mon_score_hist, and none where it makes the scores itself or takes more."""
    run(fake, f"""
        ctx = context({N}, 300)
        layers = [layer(ctx, {N}, 300) for _ in range(2)]
        for t in range(2):
            fake.fake_reset(0)
            assert L.hc_decode_step(ctx, io_of(layers), 2, 2, None, None) == 0
            names = [l[0] for l in log()]
            assert sum("attn_combine_score" in n for n in names) == {int(scored)} and sum("attn_combine" in n for n in names) == 1, names
            assert sum("{kernel}" in n for n in names) == 1, names
            assert sum("mon_score_hist" in n for n in names) == {int(not scored and "select" in kernel)}, names
    """)


def test_a_step_that_failed_does_not_count_scores_twice(fake):
    """The selection's launch fails: the layers' histograms are not known to be clear, so the steps that follow do without them."""
    run(fake, """
        ctx = context(20000, 300)
        layers = [layer(ctx, 20000, 300) for _ in range(2)]
        def names():
            return [l[0] for l in log()]
        fake.fake_reset(0)
        assert L.hc_decode_step(ctx, io_of(layers), 2, 2, None, None) == 0
        first = names()
        at = [i for i, n in enumerate(first) if "mon_direct" in n][0]
        assert any("attn_combine_score" in n for n in first[:at])
        fake.fake_reset(at + 1 - sum("mon_prep" in n for n in first))
        assert L.hc_decode_step(ctx, io_of(layers), 2, 2, None, None) == hc.HC_EHIP and any("attn_combine_score" in n for n in names()) and not any("mon_direct" in n for n in names())
        fake.fake_reset(0)
        assert L.hc_decode_step(ctx, io_of(layers), 2, 2, None, None) == 0
        assert not any("attn_combine_score" in n for n in names()) and any("mon_score_hist" in n for n in names()), names()
    """)


def test_a_step_that_failed_costs_one_step_its_scores_with_the_combine_pass(fake):
    """One of two groups' selection fails: at the next step its layers' histograms are cleared, ahead of everything that could use them, from the
    one after that on both groups score with the combine pass again."""
    run(fake, """
        ctx = context(20000, 300)
        layers = [layer(ctx, 20000, 300) for _ in range(4)]
        def step(fail=0):
            fake.fake_reset(fail)
            st = L.hc_decode_step(ctx, io_of(layers), 4, 2, None, C.c_void_p(77))
            return st, [l[0] for l in log()], [int(l[-1]) for l in log()]
        st, good, _ = step()
        assert st == 0 and sum("attn_combine_score" in n for n in good) == 2
        at = [i for i, n in enumerate(good) if "mon_direct" in n][0]
        assert step(at + 1 - sum("mon_prep" in n for n in good[:at]))[0] == hc.HC_EHIP
        st, names, streams = step()
        assert st == 0, names
        clears = [i for i, n in enumerate(names) if "mon_prep" in n and streams[i] == 0]       # (on the side stream: the workspaces')
        assert clears and clears[0] < min(i for i, n in enumerate(names) if "attn_combine" in n), names
        for _ in range(2):
            st, names, _ = step()
            assert st == 0 and sum("attn_combine_score" in n for n in names) == 2 and not any("mon_score_hist" in n or "mon_prep" in n for n in names), names
    """)


def first_argument_sizes():
    """Bytes of every kernel's first argument, from the library's own metadata."""
    import msgpack
    from test_kernel_resources import LIB, code_objects, notes
    with open(LIB, "rb") as f:
        blob = f.read()
    return {k[".name"]: k[".args"][0][".size"] for obj in code_objects(blob) for desc in notes(obj) for k in msgpack.unpackb(desc)["amdhsa.kernels"] if k[".args"]}


@pytest.mark.parametrize("N,L,group,kernel", [(20000, 4, 2, "mon_directILi512ELi0E"), (40000, 4, 2, "mon_directILi1024ELi0E"), (36000, 16, 8, "mon_compact"),
                                              (5000, 4, 2, "mon_directILi512ELi3E"), (70000, 4, 2, "mon_compact")])
def test_the_scores_buffer_is_the_side_streams(fake, N, L, group, kernel):
    """Nothing on the main stream is given the caller's scores, whatever makes them: what else a caller puts on the side stream to read them, or
    another call's side work that uses the buffer, is in order with the side work alone."""
    run(fake, f"""
        for name, size in {first_argument_sizes()!r}.items():
            fake.fake_first_size(name.encode(), size)
        def layer3():
            descs = (hc.hc_head_desc * 4)()
            for h, ln in enumerate(({N}, 312, 212, 112)):
                descs[h] = hc.hc_head_desc(k_off=h * (1 << 26), v_off=h * (1 << 26) + (1 << 25), tier_off=h * (1 << 27), ctx={N}, len=ln, role=int(h > 0),
                                           rep=-1 if h == 0 else 0, sink=5 * (h > 0), recent=7 * (h > 0), k_mon=0, cap=0)
            out = C.c_void_p()
            assert L.hc_layer_create(ctx, descs, C.byref(out)) == 0, L.hc_last_error(ctx)
            return out.value
        ctx = context({N}, 300)
        io = io_of([layer3() for _ in range({L})])
        fake.fake_reset(0)
        assert L.hc_decode_step(ctx, io, {L}, {group}, None, C.c_void_p(77)) == 0
        assert any("{kernel}" in l[0] for l in log()), log()
        reads = {{0: 0, 77: 0}}
        for i, l in enumerate(log()):
            words = (C.c_uint64 * 1024)()
            n = fake.fake_first_arg(C.c_long(i), words)
            assert n > 0
            reads[int(l[-1])] += sum(x.scores == w for w in words[:n // 8] for x in io)
        assert reads[0] == 0 and reads[77] > 0, reads
    """)


@pytest.mark.parametrize("agg", [0, 1])
@pytest.mark.parametrize("side", [None, 77])
def test_a_histogram_is_made_of_the_digits_that_are_read(fake, agg, side):
    """Over drawn stacks of middle lengths: the digits of the combine pass's histogram are those of what selects from it, mon_direct's (1, 2 for mean
    logits) or the keys' (0)."""
    run(fake, f"""
        import random, re
        rng = random.Random(5)
        seen = set()
        for _ in range(120):
            N, n, G, B = rng.randint(8000, 70000), rng.choice([2, 4, 8]), rng.choice([1, 2, 4, 8]), rng.choice([1, 1, 2, 4])
            r = rng.choice([64, 700, 4000, 8000])
            cfg = hc.hc_config(B=B, Hq=G * n, Hkv=n, D=128, max_ctx=(N + 63) // 64 * 64, max_k=r, window=1, metric=0, tau_num=1, tau_den=2, agg={agg}, window_mode=0)
            ctx = C.c_void_p()
            assert L.hc_create(C.byref(cfg), C.byref(ctx)) == 0
            layers = []
            for _ in range(rng.choice([2, 4])):
                descs = (hc.hc_head_desc * (B * n))()
                for i in range(B * n):
                    h, c = i % n, N if i < n else min(N, 9000)
                    descs[i] = hc.hc_head_desc(k_off=i * (1 << 26), v_off=i * (1 << 26) + (1 << 25), tier_off=i * (1 << 27), ctx=c, len=c if h == 0 else 12 + max(1, r - 7 * (h - 1)),
                                               role=int(h > 0), rep=-1 if h == 0 else 0, sink=5 * (h > 0), recent=7 * (h > 0), k_mon=0, cap=0)
                out = C.c_void_p()
                assert L.hc_layer_create(ctx, descs, C.byref(out)) == 0, L.hc_last_error(ctx)
                layers.append(out.value)
            fake.fake_reset(0)
            assert L.hc_decode_step(ctx, io_of(layers), len(layers), rng.choice([1, 2]), None, C.c_void_p({side})) == 0, L.hc_last_error(ctx)
            names = [l[0] for l in log()]
            made = [int(re.search("attn_combine_score_kernelILi.ELi(.)E", x)[1]) for x in names if "attn_combine_score" in x]
            if made:
                direct, select = sum(bool(re.search("mon_directILi[0-9]+ELi0E", x)) for x in names), sum(bool(re.search("mon_selectILi[0-9]+ELi2E", x)) for x in names)
                assert sum(x == 0 for x in made) == select and sum(x == {1 + agg} for x in made) == direct and select + direct == len(made), (N, G, B, names)
                assert not any("mon_score_hist" in x for x in names)
                seen |= set(made)
            for x in layers:
                assert L.hc_layer_destroy(C.c_void_p(x)) == 0
            assert L.hc_destroy(ctx) == 0
        assert seen == ({{0, {1 + agg}}} if {side} else {{{1 + agg}}}), seen
    """)
