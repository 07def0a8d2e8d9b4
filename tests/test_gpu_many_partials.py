"""The merge of a pair that many workgroups share: 17 and more partials, around the batches of 32 loads and chunks of 128
scales of the merge kernel, up to one partial per workgroup of the grid."""
import numpy as np
import pytest

import paper_2510_08525_amd as rl
from harness import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,kernel,Hq,gate,n", [
    (rl.RLKV_BF16, rl.RLKV_KERNEL_MFMA, 4, None, 17 * 128),
    (rl.RLKV_BF16, rl.RLKV_KERNEL_MFMA, 4, 0.3, 33 * 128 + 5),
    (rl.RLKV_BF16, rl.RLKV_KERNEL_MFMA, 16, None, 128 * 128),
    (rl.RLKV_BF16, rl.RLKV_KERNEL_MFMA, 2, None, 300 * 128 + 1),
    (rl.RLKV_F32, rl.RLKV_KERNEL_VALU, 4, None, 64 * 128 - 3),
    (rl.RLKV_F32, rl.RLKV_KERNEL_VALU, 2, 0.6, 129 * 128),
], ids=lambda x: str(x))
def test_one_pair_over_many_workgroups(gpu_device, dtype, kernel, Hq, gate, n):
    c = Case(Hq=Hq, Hkv=1, B=1, S=16, R=112, dtype=dtype, kernel=kernel, mask=[1], cap=n + 4, seed=12)
    g = None
    if gate is not None:
        g = np.asarray([gate], dtype=np.float32)
        c.cache.set_gates(g)
    for _ in range(0, n - 1000, 4096):
        c.append([min(4096, n - 1000 - int(c.n[0]))])
    c.append([n - int(c.n[0])])
    c.check_decode(0, "decode", gates=g)
    c.check_decode(1, "fused step", fused=True, gates=g)
    c.close()
