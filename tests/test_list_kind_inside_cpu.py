"""The kind of list a layer gets where shares are merged inside the attention launch, without a GPU: the measured side on both sides of
each line, and the older rule where the merge is a launch."""
import numpy as np
import pytest

import paper_2510_08525_amd as rl

MFMA, VALU, BF16, F32 = rl.RLKV_KERNEL_MFMA, rl.RLKV_KERNEL_VALU, rl.RLKV_BF16, rl.RLKV_F32


def kind(kernel, dtype, q_heads, kv_heads, n_full, batch, n, gated=0, step=0, fn="rlkv_plan_list_kind"):
    n = np.full(batch, n, np.int32)
    return getattr(rl.load_library(), fn)(kernel, dtype, q_heads // kv_heads, gated, step, 256, kv_heads, n_full, 320, batch, n.ctypes.data, None)


# (q heads, KV heads, full heads, sequences, gated, tokens of whole pairs, tokens of shares)
@pytest.mark.parametrize("Hq,Hkv,full,B,gated,yes,no", [
    (32, 8, 4, 1, 0, 352, 353), (28, 4, 2, 1, 0, 300, 400), (28, 4, 2, 8, 0, 300, 480), (8, 8, 4, 4, 0, 300, 400), (16, 1, 1, 4, 0, 300, 400),
    (28, 4, 4, 4, 1, 256, 257), (32, 8, 8, 1, 1, 256, 257), (32, 8, 4, 16, 0, 350, 800), (8, 8, 4, 16, 0, 300, 800),
], ids=lambda x: str(x))
@pytest.mark.parametrize("step", [0, 1], ids=["decode", "step"])
def test_lines(Hq, Hkv, full, B, gated, yes, no, step):
    assert kind(MFMA, BF16, Hq, Hkv, full, B, yes, gated, step) == 1
    assert kind(MFMA, BF16, Hq, Hkv, full, B, no, gated, step) == 0


def test_elsewhere_as_with_a_merge_launch():
    for n in (100, 130, 260, 400, 1000, 2000):
        for dtype in (BF16, F32):
            assert kind(VALU, dtype, 32, 8, 4, 2, n) == kind(VALU, dtype, 32, 8, 4, 2, n, fn="rlkv_plan_list_whole")
        assert kind(MFMA, BF16, 64, 4, 4, 32, n) == kind(MFMA, BF16, 64, 4, 4, 32, n, fn="rlkv_plan_list_whole")
    assert kind(MFMA, BF16, 32, 8, 4, 1, 17 * 128) == 0 and kind(MFMA, BF16, 32, 8, 9, 1, 100) == -1
