"""The merge of a pair that many workgroups share: on both sides of the 16 partials taken in one go, of the 64 from which on 32 loads
are in flight, at whole batches of 32 loads and whole chunks of 128 scales and one beyond, up to one partial per workgroup of the
grid.  The lengths are found from the plan of the shares, which says how many partials a pair of so many rows has."""
import numpy as np
import pytest
import torch

import paper_2510_08525_amd as rl
from harness import Case

pytestmark = pytest.mark.gpu

TILED, ROWS = (rl.RLKV_BF16, rl.RLKV_KERNEL_MFMA), (rl.RLKV_F32, rl.RLKV_KERNEL_VALU)
ALLOWANCE = 32                         # tokens of growth a list is planned for


def length_with(partials, n_wg):
    """Tokens of one pair whose list (rounds of 128 rows, planned with room for 32 more) has this many partials."""
    for rounds in range(1, 4 * n_wg):
        _, _, _, count = rl.rlkv_plan_shares([rounds], n_wg)
        if count[0] == partials:
            return rounds * 128 - ALLOWANCE
    raise AssertionError(f"no list of one pair has {partials} partials on {n_wg} workgroups")


@pytest.mark.parametrize("gate", [None, 0.3], ids=["plain", "blending"])
@pytest.mark.parametrize("partials,kind,Hq", [(16, TILED, 4), (17, TILED, 4), (64, TILED, 4), (65, TILED, 2), (96, TILED, 4), (128, TILED, 16),
                                              (129, TILED, 2), (256, TILED, 4), (16, ROWS, 2), (65, ROWS, 2), (128, ROWS, 4), (129, ROWS, 2)],
                         ids=lambda x: str(x) if isinstance(x, int) else ("tiled" if x is TILED else "rows"))
def test_one_pair_over_many_workgroups(gpu_device, partials, kind, Hq, gate):
    n = length_with(partials, torch.cuda.get_device_properties(0).multi_processor_count)
    c = Case(Hq=Hq, Hkv=1, B=1, S=16, R=112, dtype=kind[0], kernel=kind[1], mask=[1], cap=n + 2 * ALLOWANCE, seed=12)
    g = None
    if gate is not None:
        g = np.asarray([gate], dtype=np.float32)
        c.cache.set_gates(g)
    while c.n[0] < n:
        c.append([min(4096, n - int(c.n[0]))])
    c.check_decode(0, "decode", gates=g)
    c.check_decode(1, "fused step", fused=True, gates=g)
    c.close()
