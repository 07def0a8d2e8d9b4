"""Row-major kernel at groups of one and two heads (vector ALU) and of three (matrix cores): batches of 16 rows whole and broken, one to
all eight wavefronts with rows, shares and whole pairs, decode calls and steps, blending heads, large scores, against the oracle."""
import numpy as np
import pytest

import paper_2510_08525_amd as rl
from harness import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [rl.RLKV_F32, rl.RLKV_BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("gate", [None, 0.3], ids=["plain", "blending"])
@pytest.mark.parametrize("group", [1, 2, 3])
@pytest.mark.parametrize("lengths", [[1, 2], [15, 16], [17, 31], [32, 33], [63, 129], [300, 96], [1100, 520], [2500, 900]], ids=str)
def test_against_the_oracle(gpu_device, lengths, group, gate, dtype):
    c = Case(Hq=3 * group, Hkv=3, B=2, S=9, R=61, dtype=dtype, kernel=rl.RLKV_KERNEL_VALU, mask=[1, 0, 1], cap=max(lengths) + 8, seed=31,
             arena_fill=0xFF)
    g = None
    if gate is not None:
        g = np.asarray([gate, 1.0, 0.8], np.float32)
        c.cache.set_gates(g)
    while (c.n < np.asarray(lengths)).any():
        c.append([int(min(2048, n - x)) for n, x in zip(lengths, c.n)])
    c.check_decode(0, "decode", gates=g)
    for t in range(1, 4):
        c.check_decode(t, "step", fused=True, gates=g)
    c.close()


@pytest.mark.parametrize("dtype", [rl.RLKV_F32, rl.RLKV_BF16], ids=["f32", "bf16"])
@pytest.mark.parametrize("group", [1, 2])
@pytest.mark.parametrize("scale", [1e8, -1e9, 1e30])
def test_large_scores(gpu_device, group, scale, dtype):
    c = Case(Hq=2 * group, Hkv=2, B=2, S=4, R=28, dtype=dtype, kernel=rl.RLKV_KERNEL_VALU, mask=[1, 0], cap=1000, seed=12, scale=scale)
    c.append([900, 17])
    c.check_decode(0, "decode")
    c.check_decode(1, "step", fused=True)
    c.close()
