"""How the rows of a short pass are dealt to the workgroups of the split pass (host only): no workgroup crosses from one head to
the next, every row is covered, nobody's share is longer than it has to be, and as many partial results fit as before."""
import random

import pytest

from paper_2601_13684_amd import binding as hc
from paper_2601_13684_amd import inputs as I
from paper_2601_13684_amd import runtime as R

SHORT_SHARE = 16


def describe(ctxs, budgets, n_full, group, cus, wg):
    heads = [[I.HeadSpec(I.ROLE_FULL)] * n_full + [I.HeadSpec(I.ROLE_ANCHOR, sink=1, recent=0, budget=min(b, n)) for b in budgets] for n in ctxs]
    hkv = n_full + len(budgets)
    spec = I.LayerSpec(B=len(ctxs), Hq=group * hkv, Hkv=hkv, D=128, ctx=list(ctxs), heads=heads)
    descs, _, _ = R.make_descs(spec)
    info = hc.hc_plan_describe(R.make_config(spec), descs, compute_units=cus, workgroups_per_cu=wg)
    assert info.rows_covered == info.total_rows == sum(d.len for d in descs)
    return info, [-(-d.len // 32) for d in descs]


def fewest(units, most):
    share = 1
    while sum(-(-u // share) for u in units) > most:
        share += 1
    return share


def check(info, units, group, cus, wg):
    limit = min(cus * wg, max(hc.HC_STATIC_MAX_PARTIALS, sum(units) // 4))
    if len(units) > limit or sum(units) < 8 or sum(units) >= SHORT_SHARE * cus * wg:
        return False
    assert info.n_partials == info.n_workgroups <= limit
    two = fewest(units, limit)
    one = fewest(units, min(cus, limit)) if len(units) <= cus else None
    share = one if one is not None and (group >= 8 or one <= two + 2) else two
    assert info.max_rows_per_workgroup <= 32 * share
    if share == one:
        assert info.n_workgroups <= cus
    return True


@pytest.mark.parametrize("group", [1, 4, 8])
@pytest.mark.parametrize("ctxs", [(256,), (1000,), (4096,), (8193,), (16384,), (32768,), (70000,), (8192, 5000, 6000, 12000), (33,) * 60])
def test_workgroups_of_a_short_pass_keep_to_one_head(ctxs, group):
    info, units = describe(ctxs, (512, 700, 33, 1, 600, 512), 2, group, 256, 2)
    assert check(info, units, group, 256, 2)


def test_drawn_layers_and_devices():
    rng = random.Random(3)
    short = 0
    for _ in range(300):
        cus, wg = rng.choice([(1, 1), (8, 2), (38, 2), (64, 4), (256, 1), (256, 2), (304, 2)])
        ctxs = [rng.randint(2, rng.choice([64, 2000, 40000])) for _ in range(rng.randint(1, 20))]
        group = rng.choice([1, 2, 4, 8])
        info, units = describe(ctxs, [rng.randint(2, 900) for _ in range(rng.randint(1, 7))], rng.randint(1, 2), group, cus, wg)
        assert 1 <= info.n_workgroups <= cus * wg
        short += check(info, units, group, cus, wg)
    assert short > 50


def test_partial_results_of_a_wide_split_still_fit_the_fixed_scratch():
    """hc_set_split(16): a layer of 3,000 granules had 750 workgroups; one to a granule would be more than hc_decode_attn_static takes."""
    info, units = describe((40000, 30000), (512,) * 6, 1, 4, 256, 16)
    assert sum(units) > 2300 and info.n_partials == info.n_workgroups <= hc.HC_STATIC_MAX_PARTIALS
