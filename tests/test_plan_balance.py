"""CPU tests of the planner's load balance: units cut only where the
workgroups' loads need it, uneven groups spread over XCDs."""
import numpy as np
import pytest

import paper_2606_02964_amd as msa
from test_abi_host import _descriptors, check_plan, host_plan

#: the cost of an item beside its key steps, as the planner counts it
ITEM_STEPS = 4.0


def _loads(plan, slots):
    info = plan.info()
    row_pos, work, merge = msa.msa_plan_export(plan)
    cost = (work[:, 5] - work[:, 4] + 63) // 64 + ITEM_STEPS
    return info, row_pos, work, merge, np.bincount(work[:, 7], weights=cost, minlength=slots)


CASES = [
    # contexts, segments, Hq, Hkv, d, most a workgroup may hold over the mean
    ([10240], [[(0, 5056), (10112, 128)]], 32, 8, 128, 1.12),          # long causal units, a group per XCD
    ([10129 - 37 * b for b in range(9)], None, 8, 2, 128, 1.06),       # 18 even groups on 8 XCDs
    ([28861], [[(7215, 304), (28253, 608)]], 8, 2, 128, 1.20),         # few units, each far longer than the mean
    ([10336, 10299, 10262], None, 16, 16, 64, 1.06),                   # 48 groups
    ([4643, 900, 2100, 333, 1800, 4000], [[(4000, 643)], [(899, 1)], [(2000, 100)], [(332, 1)], [(1, 1799)],
                                          [(3999, 1)]], 64, 8, 128, 1.35),
]


def _inst(lens, segs, hq, hkv, d):
    inst = _descriptors(lens, segs, hq, hkv, d)
    inst.total_q = int(inst.seg_len.sum())
    inst.segments = lambda b: segs[b]
    return inst


@pytest.mark.parametrize("lens,segs,hq,hkv,d,most", CASES)
def test_workgroup_loads_are_even(lens, segs, hq, hkv, d, most):
    inst = _inst(lens, segs or [[(0, n)] for n in lens], hq, hkv, d)
    plan = host_plan(msa, inst)
    slots = 256 if plan.info()["tile_rows"] == 256 else 512
    info, row_pos, work, merge, load = _loads(plan, slots)
    check_plan(inst, row_pos, work, merge, info, hq // hkv)
    assert load.max() <= most * load.sum() / slots


@pytest.mark.parametrize("tile", [msa.MSA_PLAN_TILE_ROWS_128, msa.MSA_PLAN_TILE_ROWS_256])
@pytest.mark.parametrize("tokens", [2000, 4096, 8000, 8200, 12000])
def test_partials_of_cut_units_fit_the_noalloc_workspace(tokens, tile):
    """One sequence of 131072 keys whose units number about one to two per
    workgroup: every partial of the cuts fits the 64 MiB workspace of the
    call that allocates nothing."""
    L = 131072
    inst = _inst([L], [[(L - tokens, tokens)]], 8, 2, 128)
    info = host_plan(msa, inst, flags=tile).info()
    assert info["workspace_bytes"] <= msa.MSA_NOALLOC_WORKSPACE_BYTES


def test_short_units_are_not_cut():
    """Units of up to 1024 keys stay whole however few there are, and
    MSA_PLAN_NO_AUTO_SPLIT keeps every unit whole."""
    inst = _descriptors([1024], [[(448, 576)]], 32, 8, 128)
    assert host_plan(msa, inst).info()["num_merge"] == 0
    long = _descriptors([30000], [[(29000, 1000)]], 32, 8, 128)
    assert host_plan(msa, long).info()["num_merge"] > 0
    assert host_plan(msa, long, flags=msa.MSA_PLAN_NO_AUTO_SPLIT).info()["num_merge"] == 0


@pytest.mark.parametrize("lens,segs,hq,hkv,d,items", [
    ([512], [[(128, 64), (384, 64)]], 4, 4, 64, True),
    ([1000, 300], [[(900, 100)], [(0, 5), (299, 1)]], 8, 2, 128, True),
    ([700], [[(700 - 248, 248)]], 32, 8, 128, True),      # 31 x 8 items of 8 tokens
    ([700], [[(700 - 249, 249)]], 32, 8, 128, False),     # 32 x 8: no longer fewer than CUs
    ([6000], [[(5900, 60)]], 8, 2, 128, True),            # split, a CU for each piece
    ([28861], [[(7215, 304), (28253, 608)]], 8, 2, 128, False),
])
def test_few_tiles_run_as_32_row_items(lens, segs, hq, hkv, d, items):
    """128-row plans of few short tiles: items of up to 32 rows, one per CU at most."""
    inst = _inst(lens, segs, hq, hkv, d)
    G = hq // hkv
    plan = host_plan(msa, inst)
    info = plan.info()
    row_pos, work, merge = msa.msa_plan_export(plan)
    check_plan(inst, row_pos, work, merge, info, G)
    assert info["tile_rows"] == 128
    assert ((work[:, 3] * G).max() <= 32) == items
    assert not items or len(work) <= 256
    forced = host_plan(msa, inst, flags=msa.MSA_PLAN_TILE_ROWS_128)
    assert (msa.msa_plan_export(forced)[1][:, 3] * G).max() > 32


@pytest.mark.parametrize("lens,segs,hq,hkv,d,rows", [
    ([10240], [[(0, 5056), (10112, 128)]], 32, 8, 128, 256),   # 109 key steps per workgroup slot
    ([8000], [[(0, 3850), (7700, 300)]], 32, 8, 128, 128),     # 75
    ([30000], [[(7500, 300), (29400, 600)]], 32, 8, 128, 256),  # few tiles, each long
    ([6468, 6431], None, 16, 16, 64, 128),                      # 160 of the shorter 64-wide steps
    ([16000] * 8 + [12000] * 40, [[(15000, 1000)]] * 8 + [[(11999, 1)]] * 40, 32, 8, 128, 128),  # much decoding
    ([16000] * 8 + [12000] * 4, [[(15000, 1000)]] * 8 + [[(11999, 1)]] * 4, 32, 8, 128, 256),    # little
])
def test_tile_width_by_steps_and_fill(lens, segs, hq, hkv, d, rows):
    inst = _inst(lens, segs or [[(0, n)] for n in lens], hq, hkv, d)
    plan = host_plan(msa, inst)
    check_plan(inst, *msa.msa_plan_export(plan), plan.info(), hq // hkv)
    assert plan.info()["tile_rows"] == rows


@pytest.mark.parametrize("lens,segs,hq,hkv,d,split", [
    ([2048], [[(1948, 100)]], 32, 8, 128, 64),
    ([8192], [[(8064, 128)]], 8, 2, 128, 64),
    ([512], [[(128, 64), (384, 64)]], 4, 4, 64, 192),
    ([3001, 60], [[(0, 40), (2950, 51)], [(9, 51)]], 7, 7, 128, 320),
])
def test_forced_split_of_few_tiles_keeps_whole_tiles(lens, segs, hq, hkv, d, split):
    """A forced split length cuts 128-row tiles, not 32-row items of them: the
    plan and its workspace are those of forced 128-row tiles."""
    inst = _inst(lens, segs, hq, hkv, d)
    auto = host_plan(msa, inst, kv_split_tokens=split)
    forced = host_plan(msa, inst, kv_split_tokens=split, flags=msa.MSA_PLAN_TILE_ROWS_128)
    check_plan(inst, *msa.msa_plan_export(auto), auto.info(), hq // hkv)
    assert auto.info() == forced.info()
    for a, b in zip(msa.msa_plan_export(auto), msa.msa_plan_export(forced)):
        assert np.array_equal(a, b)


LONG = ([10240], [[(0, 5056), (10112, 128)]], 32, 8, 128)  # 109 key steps per workgroup slot
MUCH_DECODING = ([16000] * 8 + [12000] * 40, [[(15000, 1000)]] * 8 + [[(11999, 1)]] * 40, 32, 8, 128)


@pytest.mark.parametrize("layout,rows", [(LONG, 128), (MUCH_DECODING, 256)])
@pytest.mark.parametrize("opts", [dict(q_tile_tokens=32), dict(kv_split_tokens=4096),
                                  dict(q_tile_tokens=20, kv_split_tokens=1024)])
def test_tile_width_with_given_tokens(layout, rows, opts):
    """Options whose accepted values or partials depend on the tile width:
    wide from 1024 tiles and 384 key steps per slot, however full."""
    inst = _inst(*layout)
    plan = host_plan(msa, inst, **opts)
    check_plan(inst, *msa.msa_plan_export(plan), plan.info(), 4)
    assert plan.info()["tile_rows"] == rows


def test_q_tile_tokens_of_wide_tiles():
    """64 tokens of 4 heads need 256-row tiles."""
    assert host_plan(msa, _inst(*MUCH_DECODING), q_tile_tokens=64).info()["tile_rows"] == 256
    with pytest.raises(msa.MsaError) as e:
        host_plan(msa, _inst(*LONG), q_tile_tokens=64)
    assert e.value.status == msa.MSA_ERR_INVALID_ARG


@pytest.mark.parametrize("lens,merges", [
    ([786, 779] + [720] * 8, False),   # cutting 786 keys leaves the 720
    ([1024] * 2 + [513] * 6, False),
    ([1024] * 2 + [512] * 6, True),
    ([1000] * 4, True),
    ([1100] + [700] * 8, True),        # rows past 1024 keys
])
def test_decode_rows_are_cut_only_if_the_longest_chain_falls(lens, merges):
    """Rows of up to 1024 keys: cut only where the longest item left is 512
    keys shorter, which is what the merge launch costs."""
    inst = _inst(lens, [[(n - 1, 1)] for n in lens], 28, 4, 128)
    plan = host_plan(msa, inst)
    check_plan(inst, *msa.msa_plan_export(plan), plan.info(), 7)
    assert plan.info()["tile_rows"] == 32 and (plan.info()["num_merge"] > 0) == merges


@pytest.mark.parametrize("new,hq,hkv,flags,rows", [
    (1900, 8, 2, 0, 256),
    (1900, 8, 2, msa.MSA_PLAN_NO_AUTO_SPLIT, 128),   # 120 narrow units
    (3600, 8, 2, msa.MSA_PLAN_NO_AUTO_SPLIT, 128),   # 226
    (3600, 16, 2, msa.MSA_PLAN_NO_AUTO_SPLIT, 256),  # 450
])
def test_uncut_units_widen_past_one_per_cu(new, hq, hkv, flags, rows):
    inst = _inst([30000], [[(30000 - new, new)]], hq, hkv, 128)
    plan = host_plan(msa, inst, flags=flags)
    check_plan(inst, *msa.msa_plan_export(plan), plan.info(), hq // hkv)
    assert plan.info()["tile_rows"] == rows
