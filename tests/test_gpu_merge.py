"""GPU test of the split merge: every row chunk of a split tile, and split
counts around the merge kernel's batch of 8 pieces."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2606_02964_amd as msa
import workloads
from gpu_helpers import DeviceInstance, check_o, run


@pytest.mark.parametrize("tile", [msa.MSA_PLAN_TILE_ROWS_32, msa.MSA_PLAN_TILE_ROWS_128,
                                  msa.MSA_PLAN_TILE_ROWS_256])
@pytest.mark.parametrize("hq,hkv,d", [(4, 2, 128), (3, 1, 64)])
@pytest.mark.parametrize("pieces", [2, 7, 8, 9, 17])
def test_merge_split_counts(oracle_lib, pieces, hq, hkv, d, tile):
    """The last 70 tokens of one sequence cut into `pieces` key ranges: tiles
    of full and partial height, rows that end in the last piece."""
    L = 64 * pieces - 5
    n = min(70, L)
    inst = workloads.make_layout(300 + pieces, [L, 40], [[(L - n, n)], [(39, 1)]], hq, hkv, d)
    ro, rl = oracle_lib.forward(inst)
    o, lse, plan = run(DeviceInstance(inst), kv_split_tokens=64, flags=tile)
    assert plan.info()["max_splits"] == pieces
    check_o(o.float().cpu().numpy(), ro, lse.cpu().numpy(), rl)


@pytest.mark.parametrize("hq,hkv,d", [(8, 2, 128), (4, 4, 64)])
def test_units_cut_to_even_out_workgroups(oracle_lib, hq, hkv, d):
    """An automatic plan whose long units are cut at uneven places, some more
    than once, beside whole units; every row of one head per KV head."""
    L = 6011
    inst = workloads.make_layout(77, [L, 900], [[(100, 300), (L - 500, 500)], [(0, 900)]], hq, hkv, d)
    heads_of = np.arange(0, hq, hq // hkv, dtype=np.int32)
    rows = np.repeat(np.arange(inst.total_q, dtype=np.int64), heads_of.size)
    heads = np.tile(heads_of, inst.total_q)
    ro, rl = oracle_lib.forward(inst, rows=rows, heads=heads)
    o, lse, plan = run(DeviceInstance(inst))
    info = plan.info()
    assert 0 < info["num_merge"] < info["num_tiles"] and info["max_splits"] > 2
    check_o(o.float().cpu().numpy()[rows, heads], ro, lse.cpu().numpy()[rows, heads], rl)
