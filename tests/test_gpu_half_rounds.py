"""Short fp32 lists go out in half rounds, one per workgroup: on both sides of the lines (a pair of 32 half rounds, as many half rounds
as the grid has workgroups), whole and broken batches of 16 rows, and the merge of 31 to 33 partials, which it takes in one go up to 32."""
import numpy as np
import pytest
import torch

import paper_2510_08525_amd as rl
from harness import Case

pytestmark = pytest.mark.gpu

ROOM = 32                         # tokens of growth a list is planned for


def run(lengths, Hq, Hkv, mask, dtype, kernel, gate):
    c = Case(Hq=Hq, Hkv=Hkv, B=len(lengths), S=16, R=112, dtype=dtype, kernel=kernel, mask=mask, cap=max(lengths) + 2 * ROOM, seed=21,
             arena_fill=0xFF)
    g = None
    if gate is not None:
        g = np.asarray([gate if f else 1.0 for f in mask], dtype=np.float32)
        c.cache.set_gates(g)
    while (c.n < np.asarray(lengths)).any():
        c.append([int(min(2048, n - x)) for n, x in zip(lengths, c.n)])
    c.check_decode(0, "decode", gates=g)
    c.check_decode(1, "fused step", fused=True, gates=g)
    c.close()


@pytest.mark.parametrize("gate", [None, 0.3], ids=["plain", "blending"])
@pytest.mark.parametrize("Hq", [1, 4, 7, 16])
@pytest.mark.parametrize("n", [130, 64 * 31 - ROOM, 64 * 32 - ROOM, 64 * 32 - ROOM + 1, 1001])
def test_one_pair(gpu_device, n, Hq, gate):
    run([n], Hq, 1, [1], rl.RLKV_F32, rl.RLKV_KERNEL_VALU, gate)


@pytest.mark.parametrize("extra", [0, 1])
def test_as_many_half_rounds_as_workgroups(gpu_device, extra):
    n_wg = torch.cuda.get_device_properties(0).multi_processor_count
    # pairs of 8 half rounds each, the last one a row short of a ninth or one beyond
    pairs = n_wg // 8
    run([64 * 8 - ROOM] * (pairs - 1) + [64 * 8 - ROOM + extra], 2, 1, [1], rl.RLKV_F32, rl.RLKV_KERNEL_VALU, None)


@pytest.mark.parametrize("gate", [None, 0.3], ids=["plain", "blending"])
@pytest.mark.parametrize("partials", [31, 32, 33])
def test_merge_of_about_32_partials(gpu_device, partials, gate):
    n_wg = torch.cuda.get_device_properties(0).multi_processor_count
    for rounds in range(17, 4 * n_wg):
        if rl.rlkv_plan_shares([rounds], n_wg)[3][0] == partials:
            break
    else:
        pytest.skip(f"no list of one pair has {partials} partials on {n_wg} workgroups")
    run([rounds * 128 - ROOM], 4, 1, [1], rl.RLKV_BF16, rl.RLKV_KERNEL_MFMA, gate)
