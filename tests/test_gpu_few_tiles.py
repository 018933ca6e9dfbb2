"""GPU test of 128-row plans whose few tiles run as 32-row items: whole, split
with workspace slots of 128 rows, with ragged ends and with precise weights."""
import pytest
import torch

pytestmark = pytest.mark.gpu
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

import paper_2606_02964_amd as msa
import workloads
from gpu_helpers import DeviceInstance, check_o, run


@pytest.mark.parametrize("precise", [0, msa.MSA_PLAN_PRECISE_WEIGHTS])
@pytest.mark.parametrize("hq,hkv,d", [(4, 4, 64), (8, 2, 128), (5, 1, 128), (32, 1, 64)])
@pytest.mark.parametrize("lens,segs", [
    ([70, 33], [[(0, 70)], [(31, 2)]]),
    ([777], [[(100, 17), (300, 1), (740, 37)]]),
    ([769], [[(700, 69)]]),
    ([3001], [[(0, 40), (2950, 51)]]),
])
def test_few_tiles(oracle_lib, lens, segs, hq, hkv, d, precise):
    inst = workloads.make_layout(600 + sum(lens), lens, segs, hq, hkv, d, keep_logical=False)
    ro, rl = oracle_lib.forward(inst)
    o, lse, plan = run(DeviceInstance(inst), flags=precise)
    info = plan.info()
    assert info["tile_rows"] in (32, 128)
    assert (info["num_merge"] > 0) == (max(lens) > 768)
    check_o(o.float().cpu().numpy(), ro, lse.cpu().numpy(), rl)
