"""GPU test of the attention kernels' step bookkeeping: runs of key steps that
end at and around the 64-step windows of preloaded block ids, with whole and
partial last steps and last blocks."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2606_02964_amd as msa
import workloads
from gpu_helpers import DeviceInstance, check_o, run


@pytest.mark.parametrize("precise", [0, msa.MSA_PLAN_PRECISE_WEIGHTS])
@pytest.mark.parametrize("tile", [msa.MSA_PLAN_TILE_ROWS_32, msa.MSA_PLAN_TILE_ROWS_128,
                                  msa.MSA_PLAN_TILE_ROWS_256])
@pytest.mark.parametrize("hq,hkv,d", [(8, 2, 128), (3, 1, 64)])
@pytest.mark.parametrize("L", [64 * 2, 64 * 3, 64 * 3 + 1, 64 * 4 + 5, 64 * 5, 64 * 64 - 1, 64 * 64, 64 * 64 + 33, 64 * 65 + 16, 64 * 67,
                               64 * 128 + 49, 64 * 131])
def test_id_windows_and_last_steps(oracle_lib, L, hq, hkv, d, tile, precise):
    """Unsplit items of up to L keys: as many rows at the end of the context
    as a 256-row tile holds (all eight waves compute, four of them copy), and
    a few in the middle that share their tile."""
    n = 256 // (hq // hkv)
    mid = min(L // 2, L - n - 8)
    inst = workloads.make_layout(500 + L, [L], [[(mid, 5), (L - n, n)]], hq, hkv, d, keep_logical=False)
    ro, rl = oracle_lib.forward(inst)
    o, lse, plan = run(DeviceInstance(inst), flags=tile | precise | msa.MSA_PLAN_NO_AUTO_SPLIT)
    if tile == msa.MSA_PLAN_TILE_ROWS_256:
        work = msa.msa_plan_export(plan)[1]
        assert (work[:, 3] * (hq // hkv)).max() > 224  # the last wave has rows
    check_o(o.float().cpu().numpy(), ro, lse.cpu().numpy(), rl)


@pytest.mark.parametrize("precise", [0, msa.MSA_PLAN_PRECISE_WEIGHTS])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("L", [64 * 63 + 9, 64 * 66 + 21, 64 * 67, 64 * 131 + 49])
def test_id_windows_of_full_128_row_tiles(oracle_lib, L, d, precise):
    """272 full 128-row tiles, more than one per CU: no helper
    waves, so every wave both copies and computes, past 64 and 128 key steps;
    every row of one head per KV head."""
    hq, hkv, seqs, n = 8, 2, 17, 256
    inst = workloads.make_layout(700 + L, [L] * seqs, [[(L - n, n)]] * seqs, hq, hkv, d, keep_logical=False)
    rows = np.repeat(np.arange(inst.total_q, dtype=np.int64), hkv)
    heads = np.tile(np.arange(0, hq, hq // hkv, dtype=np.int32) + 1, inst.total_q)
    ro, rl = oracle_lib.forward(inst, rows=rows, heads=heads)
    o, lse, plan = run(DeviceInstance(inst), flags=msa.MSA_PLAN_TILE_ROWS_128 | msa.MSA_PLAN_NO_AUTO_SPLIT | precise)
    assert plan.info()["num_workgroups"] > 256 and (msa.msa_plan_export(plan)[1][:, 3] == 32).all()
    check_o(o.float().cpu().numpy()[rows, heads], ro, lse.cpu().numpy()[rows, heads], rl)


@pytest.mark.parametrize("seqs", [32, 33])
def test_workgroups_at_and_past_one_per_cu(oracle_lib, seqs):
    """128-row tiles in 256 workgroups (one per CU, with copying helper waves)
    and in 264 (without): every row with the oracle, and bit for bit with
    256-row tiles."""
    L = 64 * 66 + 21
    segs = [[(L - 3, 3)] if b % 4 else [(L - 60, 2), (L - 30, 30)] for b in range(seqs)]
    inst = workloads.make_layout(91, [L] * seqs, segs, 16, 8, 64, keep_logical=False)
    ro, rl = oracle_lib.forward(inst)
    flags = msa.MSA_PLAN_TILE_ROWS_128 | msa.MSA_PLAN_NO_AUTO_SPLIT
    o, lse, plan = run(DeviceInstance(inst), flags=flags)
    assert (plan.info()["num_workgroups"] <= 256) == (seqs == 32)
    check_o(o.float().cpu().numpy(), ro, lse.cpu().numpy(), rl)
    o2, _, wide = run(DeviceInstance(inst), flags=msa.MSA_PLAN_TILE_ROWS_256 | msa.MSA_PLAN_NO_AUTO_SPLIT)
    assert wide.info()["tile_rows"] == 256 and torch.equal(o2.view(torch.int16), o.view(torch.int16))
